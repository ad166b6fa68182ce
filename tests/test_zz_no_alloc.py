"""rtn_linear_noalloc (the entry point for callers that cannot allocate: split-K partial sums in the library's fixed
device array) against rtn_linear with a caller's workspace, through the C ABI: same plan, so the outputs must be
bit-identical.  Two calls in a row, the second on a smaller problem, so stale partial sums of the first call would
show; plans with a K split across workgroups are forced by the shapes chosen (long K, few output columns)."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


def _run_pair(rtn, synth, M, N, K, bits, g, seed):
    dev = "cuda:0"
    W = synth.normal_weight(N, K, 0.02, seed, dev)
    A = synth.activation(M, K, 100 + seed, dev)
    qw, sc = rtn.rtn_quantize(W, bits, g)
    ws = torch.empty(max(256, rtn.rtn_workspace_nbytes(M, N, K, bits, g)), dtype=torch.uint8, device=dev)
    ref = torch.empty((M, N), dtype=torch.float16, device=dev)
    got = torch.full((M, N), float("nan"), dtype=torch.float16, device=dev)
    lib = rtn._lib
    st = torch.cuda.current_stream().cuda_stream
    assert lib.rtn_linear(A.data_ptr(), M, qw.data_ptr(), sc.data_ptr(), N, K, bits, g, ref.data_ptr(), ws.data_ptr(),
                          ws.numel(), st) == 0
    assert lib.rtn_linear_noalloc(A.data_ptr(), M, qw.data_ptr(), sc.data_ptr(), N, K, bits, g, got.data_ptr(), st) == 0
    torch.cuda.synchronize()
    plan = rtn.rtn_linear_query(M, N, K, bits, g)
    return torch.equal(ref, got), plan


def _first_that_splits(rtn, candidates):
    for M, N, K, bits, g in candidates:
        if rtn.rtn_linear_query(M, N, K, bits, g)["split_k"] > 1:
            return M, N, K, bits, g
    pytest.fail(f"none of {candidates} has an automatic plan with a K split across workgroups: update the list")


def test_noalloc_matches_rtn_linear_on_two_calls_in_a_row(rtn):
    from paper_2505_15909_amd import synth
    # first call: a long-K projection at 16 rows whose automatic plan splits K across workgroups (partials in scratch)
    big = _first_that_splits(rtn, [(16, 4096, 14336, 4, 128), (16, 8192, 28672, 4, 128), (16, 16384, 53248, 4, 128)])
    same, _ = _run_pair(rtn, synth, *big, seed=1)
    assert same
    # second call, smaller (fewer rows, fewer output columns), also with a K split: stale partials of the first call
    # would show
    small = _first_that_splits(rtn, [(8, 4096, 14336, 4, 128), (4, 2048, 28672, 4, 128), (8, 4096, 14336, 8, 0),
                                     (8, 2048, 53248, 4, 128)])
    assert small[0] * small[1] < big[0] * big[1]
    same, _ = _run_pair(rtn, synth, *small, seed=2)
    assert same
    # and one without a K split, and an 8-bit one above 16 rows (wide kernel)
    same, _ = _run_pair(rtn, synth, 1, 2048, 2048, 4, 128, seed=3)
    assert same
    same, _ = _run_pair(rtn, synth, 40, 1024, 8192, 8, 0, seed=4)
    assert same


@pytest.mark.parametrize("M,N,K,bits,g", [(1011, 4608, 5120, 4, 128), (2252, 2176, 5632, 8, 128), (2048, 10240, 8192, 4, 128)])
def test_noalloc_runs_within_the_fixed_array_from_144_tiles(rtn, M, N, K, bits, g):
    """Problems whose preferred plan wants more than the fixed array, but whose tiles fill the compute units: the plan for 16 MiB,
    bit for bit that of rtn_linear with such a workspace, and right (columns from both ends and between, against the oracle).
    The last one goes out as two launches."""
    import numpy as np
    from oracle import rtn_oracle as O
    from paper_2505_15909_amd import synth
    from tests import helpers as H
    dev = "cuda:0"
    assert rtn.rtn_workspace_nbytes(M, N, K, bits, g) > 16 << 20 and -(-M // 128) * -(-N // 256) >= 144
    qw, sc = rtn.rtn_quantize(synth.normal_weight(N, K, 0.02, 7, dev), bits, g)
    A = synth.activation(M, K, 107, dev)
    got = torch.full((M, N), float("nan"), dtype=torch.float16, device=dev)
    rtn.rtn_linear_noalloc(A, qw, sc, bits, g, got)
    want = rtn.rtn_linear(A, qw, sc, bits, g, workspace=torch.empty(16 << 20, dtype=torch.uint8, device=dev))
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    cols = np.r_[0:16, N // 2:N // 2 + 16, N - 16:N]
    codes = rtn.rtn_unpack(qw, N, K, bits)[torch.from_numpy(cols).to(dev)].cpu().numpy()
    ref = O.rtn_linear(A.cpu().numpy(), codes, sc.cpu().numpy()[cols], g)
    H.assert_linear_close(got.cpu().numpy()[:, cols], ref, f"noalloc M={M} N={N} K={K}")


def test_noalloc_rejects_what_the_fixed_array_cannot_hold(rtn):
    lib = rtn._lib
    # 256 rows on the 405B-shaped down projection: the plan's partial sums exceed 16 MiB.  Operands of full size, so that
    # an accepted call would find its memory
    M, N, K = 256, 16384, 53248
    assert rtn.rtn_workspace_nbytes(M, N, K, 4, 128) > 16 << 20
    big = {n: torch.zeros(b, dtype=torch.uint8, device="cuda:0") for n, b in
           (("A", M * K * 2), ("q", N * K // 2), ("s", N * (K // 128) * 2), ("C", M * N * 2))}
    assert lib.rtn_linear_noalloc(big["A"].data_ptr(), M, big["q"].data_ptr(), big["s"].data_ptr(), N, K, 4, 128,
                                  big["C"].data_ptr(), None) == 6
    t = torch.empty(4096, dtype=torch.uint8, device="cuda:0")
    p = t.data_ptr()
    assert lib.rtn_linear_noalloc(None, 1, p, p, 64, 512, 4, 128, p, None) == 1
    assert lib.rtn_linear_noalloc(p, 1, p, p, 64, 500, 4, 128, p, None) == 4
