// The block kernel on 8-bit weights.
#include "rtn_linear_block.h"

namespace rtn {
template hipError_t launch_block<8, false>(const BlockGroup& g, int ng, int mb, unsigned grid, hipStream_t st);
}
