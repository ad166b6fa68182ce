// The block kernel on 4-bit weights with zero points.
#include "rtn_linear_block.h"

namespace rtn {
template hipError_t launch_block<4, true>(const BlockGroup& g, int ng, int mb, unsigned grid, hipStream_t st);
}
