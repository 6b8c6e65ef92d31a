"""FP32 tiles of 32 rows or columns (configurations 21-23), the FP8 tiles for few
rows (configurations 12-14), the plans of small
and skinny outputs, and odd row strides at every edge of a tile and a K panel.

Integer operands (|x| <= 8): every partial sum stays below 2^24, so FP32 is
exact in any order and the result must equal the oracle bit for bit."""
import numpy as np
import pytest

from helpers import Problem, tolerance
import oracle

pytestmark = pytest.mark.gpu
LAYOUTS = [("N", "N"), ("N", "T"), ("T", "N"), ("T", "T")]


def run_exact(gpu, M, N, K, tA, tB, path="fp32", **kw):
    from paper_2305_18236_amd import _native
    p = Problem(M, N, K, tA, tB, alpha=2.0, beta=-1.0, seed=M + 7 * N + 13 * K, dist="integers", **kw).to_device(gpu)
    _native.check(p.run(path), "mg_gemm")
    ref, _ = p.oracle()
    np.testing.assert_array_equal(p.result(), ref.reshape(M, N))
    assert p.padding_untouched()


@pytest.mark.parametrize("cfg", [21, 22, 23])
@pytest.mark.parametrize("tA,tB", LAYOUTS)
@pytest.mark.parametrize("K", [1, 32, 33, 127, 128, 160, 1000])
def test_32_row_tiles_every_panel_count(gpu, cfg, tA, tB, K):
    from paper_2305_18236_amd import _native
    _native.check(_native.mg_force_config(0, cfg), "mg_force_config")
    try:
        run_exact(gpu, 33, 95, K, tA, tB)
        run_exact(gpu, 64, 64, K, tA, tB, ldc=67)
    finally:
        _native.mg_force_config(0, -1)


@pytest.mark.parametrize("tA,tB", LAYOUTS)
@pytest.mark.parametrize("M,N,K", [(1, 1, 5000), (1, 1030, 257), (31, 1029, 2047), (32, 1024, 1024), (33, 2050, 515),
                                   (255, 1027, 300), (1031, 3, 700), (2053, 31, 1025), (500, 511, 130),
                                   (17, 384, 384)])
def test_small_and_skinny_plans(gpu, tA, tB, M, N, K):
    run_exact(gpu, M, N, K, tA, tB)
    p = Problem(M, N, K, tA, tB, seed=5).to_device(gpu)
    assert p.run("fp32", use_workspace=False) == 0
    ref, D = p.oracle()
    err = oracle.normalized_error(p.result(), ref.reshape(M, N), D.reshape(M, N))
    assert err <= tolerance("fp32", K)


@pytest.mark.parametrize("path", ["fp32", "bf16x3", "bf16", "fp16"])
@pytest.mark.parametrize("tA,tB", LAYOUTS)
@pytest.mark.parametrize("M,N,K", [(257, 259, 95), (130, 515, 97), (65, 66, 513), (513, 641, 127), (6, 5, 70)])
def test_odd_strides_and_edges(gpu, path, tA, tB, M, N, K):
    """Row strides one, two and three past a multiple of 4, and edges inside
    a 4-element chunk, with NaN-free padding between the rows never stored."""
    a, b = (M if tA == "T" else K), (K if tB == "T" else N)
    run_exact(gpu, M, N, K, tA, tB, path, lda=a + 1, ldb=b + 2, ldc=N + 3)


@pytest.mark.parametrize("cfg,waves", [(12, 8), (13, 4), (14, 4)])
@pytest.mark.parametrize("panels", [1, 2, 3, 4, 5, 59, 60, 61, 64])
def test_fp8_skinny_tiles_every_ring_state(gpu, cfg, waves, panels):
    """FP8 tiles whose waves take their own K panels: every count of panels
    around the ring's fill and around the 60 panels whose scales a wave holds,
    with whole and ragged last rows of panels, exact on integers."""
    from paper_2305_18236_amd import _native
    _native.check(_native.mg_force_config(3, cfg), "mg_force_config")
    try:
        for K in {128 * waves * panels, 128 * waves * (panels - 1) + 130}:
            run_exact(gpu, 33, 70, K, "N", "T", "fp8", ldc=71)
    finally:
        _native.mg_force_config(3, -1)


@pytest.mark.parametrize("M,N,K", [(1, 1024, 1000), (32, 1030, 4096), (64, 1024, 2500), (65, 2049, 1024),
                                   (200, 1024, 300), (256, 1500, 2048), (384, 384, 4096)])
def test_fp8_few_rows(gpu, M, N, K):
    run_exact(gpu, M, N, K, "N", "T", "fp8")
    run_exact(gpu, M, N, K, "T", "N", "fp8")
