"""16-bit plans of few tiles follow the workspace they get: without room for the
pre-packed planes they are weighed by what the tiles cost when they convert in
the kernel."""
import pytest

# (path, M, N, K); each ran 15 to 60 % slower on the 128 x 128 tile (10) that was
# planned for planes than on 64 x 64 tiles (4)
SHAPES = [(1, 1470, 1147, 2573), (1, 665, 966, 909), (1, 707, 1212, 3895), (1, 618, 1464, 3037), (1, 1542, 617, 1941),
          (2, 1380, 605, 3416), (2, 907, 518, 2241), (2, 696, 1831, 3879), (4, 1012, 720, 2442), (4, 2421, 611, 3783)]


@pytest.fixture()
def native():
    from paper_2305_18236_amd import _native
    _native.lib()
    _native.mg_load_tuning(None)   # the built-in rule alone
    yield _native
    _native._load_default_tuning(_native.lib())


@pytest.mark.parametrize("path,M,N,K", SHAPES)
def test_without_workspace(native, path, M, N, K):
    assert native.mg_gemm_plan(path, M, N, K, 0) == (0, 4, 1, 0)


@pytest.mark.parametrize("path,M,N,K", SHAPES)
def test_planes_without_partials(native, path, M, N, K):
    """A workspace for the planes alone still has them used."""
    rows = -(-M // 256) * 256 + -(-N // 256) * 256
    planes = rows * (-(-K // 128) * 128) * (4 if path == 1 else 2)
    st, cfg, splits, packed = native.mg_gemm_plan(path, M, N, K, planes)
    assert (st, splits) == (0, 1)
    assert packed == 1 or cfg == 4
    assert native.mg_gemm_plan(path, M, N, K, planes - 1) == (0, 4, 1, 0)
