"""A plan picked by a time model lets no accumulator sum a longer chain of
products than the plan of the tile ladder, which it replaces: rounding error
against 64 bits grows with that chain.  The ladder's plans of the shapes below
are written out (configuration and K ranges); each had a chain 1.1 to 11 times
as long under the time models alone."""
import pytest

GROUPS = {15: 2, 16: 2, 21: 4, 22: 4, 23: 8}   # FP32 configurations whose waves share out the K panels

FP32 = [(8116, 116, 5609, 17, 8), (4838, 200, 4725, 17, 13), (6183, 122, 6053, 17, 10), (3302, 168, 4356, 15, 3),
        (7233, 81, 2905, 17, 8), (165, 4167, 1978, 12, 6), (249, 7605, 5879, 17, 8), (200, 8192, 8192, 17, 8),
        (148, 2135, 8122, 15, 4), (169, 5369, 5826, 17, 12), (54, 262, 50, 15, 1), (120, 24, 51, 15, 1)]

BF16X3 = [(1078, 1786, 5662, 1, 7), (1410, 1197, 5451, 1, 8), (2148, 1204, 2010, 1, 4), (1680, 1243, 1371, 1, 4),
          (940, 2043, 3981, 1, 8), (1973, 916, 3946, 1, 8), (1301, 741, 3618, 1, 10), (731, 2322, 892, 2, 2),
          (712, 755, 5494, 1, 15), (2353, 475, 2141, 1, 6)]


def chain(native, path, cfg, splits, K):
    bk = native.mg_config_info(path, cfg)["bk"]
    k = K if splits < 2 else -(-(-(-K // splits)) // 128) * 128
    groups = GROUPS.get(cfg, 1) if path == 0 else 1
    return -(-(-(-k // bk)) // groups) * bk


@pytest.fixture()
def native():
    from paper_2305_18236_amd import _native
    _native.lib()
    _native.mg_load_tuning(None)   # the built-in rule alone
    yield _native
    _native._load_default_tuning(_native.lib())


@pytest.mark.parametrize("path,M,N,K,cfg,splits", [(0, *s) for s in FP32] + [(1, *s) for s in BF16X3])
def test_chain_is_no_longer_than_the_ladders(native, path, M, N, K, cfg, splits):
    st, c, s, _ = native.mg_gemm_plan(path, M, N, K, native.mg_gemm_workspace_size(path, "N", "N", M, N, K))
    assert st == 0
    assert chain(native, path, c, s, K) <= chain(native, path, cfg, splits, K), (c, s)


def rms_error(gemm, A, B, path):
    C = gemm(A, B, path=path).double()
    ref = A.double() @ B.double()
    return ((C - ref).norm() / ref.norm()).item()


@pytest.mark.gpu
@pytest.mark.parametrize("path,name,allowed,M,N,K,cfg,splits", [(0, "fp32", 1.05, *s) for s in FP32[:9]] +
                         [(1, "bf16x3", 1.001, *s) for s in BF16X3[:7]])
def test_error_is_no_larger_than_the_ladders(gpu, native, path, name, allowed, M, N, K, cfg, splits):
    """RMS error on uniform inputs.  With chains of L products and P partial
    sums its square goes as L / 4 + P / 2, so up to eight more partials beside
    chains of 384 and more add 2 % at most; 5 % allows for the sample too
    (under the longer chains the ratio was 1.2 to 2.0).  bf16x3's error of
    3.8e-6 is mostly its split, the same in both; sixteen partials add 1e-7 in
    square, 0.04 % (the longer chains 0.2 to 0.8 %)."""
    import torch
    from paper_2305_18236_amd import gemm
    gen = torch.Generator(device=gpu).manual_seed(M)
    A = torch.rand((M, K), device=gpu, generator=gen) * 2 - 1
    B = torch.rand((K, N), device=gpu, generator=gen) * 2 - 1
    now = rms_error(gemm, A, B, name)
    try:
        native.check(native.mg_force_config(path, cfg), "mg_force_config")
        native.check(native.mg_force_splits(path, splits), "mg_force_splits")
        ladder = rms_error(gemm, A, B, name)
    finally:
        native.mg_force_config(path, -1)
        native.mg_force_splits(path, -1)
    assert now <= allowed * ladder, (now, ladder)
