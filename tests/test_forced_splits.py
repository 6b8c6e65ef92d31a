"""A configuration that the caller forces or a table names is cut into the K
ranges that its own tiles ask for, not into those that the rule's time models
would give it."""
import pytest

# path, configuration, M, N, K, K ranges
SHAPES = [(0, 3, 2791, 108, 3281, 7), (0, 12, 4980, 17, 1829, 3), (0, 15, 104, 596, 2518, 7), (1, 4, 784, 2094, 1423, 1),
          (1, 4, 700, 650, 500, 1), (1, 2, 2889, 495, 2268, 2), (2, 9, 426, 2652, 2482, 3), (2, 4, 506, 596, 5567, 3),
          (4, 4, 488, 1692, 774, 1), (4, 10, 832, 580, 2004, 6)]


@pytest.fixture()
def native():
    from paper_2305_18236_amd import _native
    _native.lib()
    _native.mg_load_tuning(None)
    yield _native
    for path in (0, 1, 2, 4):
        _native.mg_force_config(path, -1)
    _native._load_default_tuning(_native.lib())


@pytest.mark.parametrize("path,cfg,M,N,K,splits", SHAPES)
def test_forced_configuration(native, path, cfg, M, N, K, splits):
    assert native.mg_force_config(path, cfg) == 0
    assert native.mg_split_count(path, M, N, K) == splits


@pytest.mark.parametrize("path,cfg,M,N,K,splits", SHAPES[:6])
def test_configuration_of_a_table_bucket(native, tmp_path, path, cfg, M, N, K, splits):
    from paper_2305_18236_amd.autotune import bucket
    table = tmp_path / "t.txt"
    table.write_text(f"{path} {bucket(M)} {bucket(N)} {bucket(K)} {cfg} s\n")
    assert native.mg_load_tuning(str(table)) == 0
    assert native.mg_tuned_config(path, M, N, K) == cfg
    assert native.mg_split_count(path, M, N, K) == splits
