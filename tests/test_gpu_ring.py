"""Direct-copy tiles through the ring of LDS stages (at most one workgroup per
compute unit): every count of K panels around the ring's fill and drain, whole
and ragged, exact on integers and bit-identical to the two-buffer form.

Integer operands (|x| <= 8) are exact in bf16, binary16, E4M3 and int8 and every
partial sum stays below 2^24, so the result must equal the oracle bit for bit."""
import numpy as np
import pytest

from helpers import PATH_ID, Problem

pytestmark = pytest.mark.gpu


def run(path, p, cfg, splits=1):
    from paper_2305_18236_amd import _native
    pid = PATH_ID[path]
    _native.check(_native.mg_force_config(pid, cfg), "mg_force_config")
    _native.check(_native.mg_force_splits(pid, splits), "mg_force_splits")
    try:
        p.reset_c()
        _native.check(p.run(path), "mg_gemm")
        return p.result()
    finally:
        _native.mg_force_config(pid, -1)
        _native.mg_force_splits(pid, -1)


@pytest.mark.parametrize("path", ["bf16", "fp16", "bf16x3"])
@pytest.mark.parametrize("panels", [1, 2, 3, 4, 5, 8, 9, 10, 11, 13, 14, 18])
def test_sixteen_bit_ring(gpu, path, panels):
    depth = 32 if path == "bf16x3" else 64
    for K in (depth * panels, depth * panels - 7):
        if K < 32:
            continue
        p = Problem(515, 640, K, "N", "N", 2.0, -1.0, seed=K, dist="integers", ldc=641).to_device(gpu)
        ref, _ = p.oracle()
        np.testing.assert_array_equal(run(path, p, 10), ref.reshape(p.M, p.N))
        assert p.padding_untouched()


@pytest.mark.parametrize("path", ["bf16", "fp16", "bf16x3"])
@pytest.mark.parametrize("splits", [1, 3])
def test_sixteen_bit_ring_equals_two_buffers(gpu, path, splits):
    for tA, tB in (("N", "N"), ("T", "T")):
        p = Problem(600, 700, 1111, tA, tB, 1.5, 0.5, seed=3).to_device(gpu)
        np.testing.assert_array_equal(run(path, p, 10, splits), run(path, p, 7, splits))


@pytest.mark.parametrize("panels", [1, 2, 3, 4, 5, 8, 9, 10, 11, 13, 14, 64, 65])
def test_fp8_ring(gpu, panels):
    for K in (128 * panels, 128 * panels - 31):
        p = Problem(130, 257, K, "N", "T", 2.0, -1.0, seed=K, dist="integers", ldc=259).to_device(gpu)
        ref, _ = p.oracle()
        np.testing.assert_array_equal(run("fp8", p, 10), ref.reshape(p.M, p.N))
        assert p.padding_untouched()


@pytest.mark.parametrize("cfg,waves", [(6, 1), (8, 8), (9, 4), (10, 4)])
@pytest.mark.parametrize("turns", [1, 2, 3, 4, 5, 8, 9, 13, 59, 60, 61])
def test_i8_ring_and_streams(gpu, cfg, waves, turns):
    """INT8: the ring (6) and the tiles whose waves stream their own panels."""
    import torch
    import oracle
    from paper_2305_18236_amd import _native, gemm_i8
    rng = np.random.default_rng(turns)
    _native.check(_native.mg_force_config(5, cfg), "mg_force_config")
    try:
        for K in (128 * waves * turns, max(128 * waves * (turns - 1), 0) + 77):
            M, N = 70, 133
            a = rng.integers(-128, 128, (M, K)).astype(np.int8)
            b = rng.integers(-128, 128, (K, N)).astype(np.int8)
            c0 = rng.integers(-1000, 1000, (M, N)).astype(np.int32)
            C = torch.from_numpy(c0.copy()).to(gpu)
            gemm_i8(torch.from_numpy(a).to(gpu), torch.from_numpy(b).to(gpu), C, alpha=3, beta=-2)
            want = 3 * (a.astype(np.int64) @ b.astype(np.int64)) - 2 * c0.astype(np.int64)
            np.testing.assert_array_equal(C.cpu().numpy(), want.astype(np.uint64).astype(np.uint32).view(np.int32))
    finally:
        _native.mg_force_config(5, -1)
