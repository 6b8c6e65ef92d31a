"""Every tile of the batched kernel in every layout, with more K panels than the
branch-free loop needs (four whole ones) and fewer, whole and ragged, and with
edges that leave some or most waves of the tile outside C.

Integer operands (|x| <= 8) are exact in every kind and all sums stay below 2^24,
so the result must equal the oracle bit for bit."""
import numpy as np
import pytest
import torch

from helpers import PATH_ID, Problem

pytestmark = pytest.mark.gpu
VARIANTS = [("fp32", 3), ("fp32", 0)] + [(p, c) for p in ("bf16x3", "bf16", "fp16") for c in (4, 5, 2)]
SIZES = [(1, 1), (31, 129), (33, 64), (63, 97), (65, 31), (96, 96), (127, 33), (129, 257), (200, 65), (260, 130)]


@pytest.mark.parametrize("path,cfg", VARIANTS)
@pytest.mark.parametrize("tA,tB", [("N", "N"), ("N", "T"), ("T", "N"), ("T", "T")])
@pytest.mark.parametrize("strided", [False, True])
def test_every_tile_and_layout(gpu, path, cfg, tA, tB, strided):
    from paper_2305_18236_amd import _native
    probs = []
    for K in (1, 33, 127, 128, 160, 161, 500):
        for i, (M, N) in enumerate(SIZES):
            ld = dict(lda=(M if tA == "T" else K) + 1, ldb=(K if tB == "T" else N) + 3, ldc=N + 2) if strided else {}
            probs.append(Problem(M, N, K, tA, tB, alpha=2.0, beta=-1.0, seed=100 * K + i, dist="integers",
                                 **ld).to_device(gpu))
    arr = (_native.mg_problem * len(probs))(*[
        _native.mg_problem(p.tA.encode(), p.tB.encode(), p.M, p.N, p.K, p.alpha, p.beta, p.dA.data_ptr(), p.lda,
                           p.dB.data_ptr(), p.ldb, p.dC.data_ptr(), p.ldc) for p in probs])
    pid = PATH_ID[path]
    ws = torch.empty(_native.mg_gemm_batched_workspace_size(pid, len(probs)), dtype=torch.uint8, device=gpu)
    _native.check(_native.mg_force_config(pid, cfg), "mg_force_config")
    try:
        st, bad = _native.mg_gemm_batched(pid, len(probs), arr, ws.data_ptr(), ws.numel(),
                                          torch.cuda.current_stream().cuda_stream)
    finally:
        _native.mg_force_config(pid, -1)
    assert st == 0, (_native.status_string(st), bad)
    for p in probs:
        ref, _ = p.oracle()
        np.testing.assert_array_equal(p.result(), ref.reshape(p.M, p.N), err_msg=f"{p.M} x {p.N} x {p.K}")
        assert p.padding_untouched()
