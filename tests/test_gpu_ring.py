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
