"""mg_batched_config names the tile that the batched launch runs."""
import pytest

TILE = {0: {3: (64, 128), 0: (128, 128)}, 1: {4: (64, 64), 5: (128, 64), 2: (128, 128)}}
TILE[2] = TILE[4] = TILE[1]


@pytest.fixture()
def native():
    from paper_2305_18236_amd import _native
    _native.lib()
    _native.mg_load_tuning(None)   # the built-in rule alone
    yield _native
    _native._load_default_tuning(_native.lib())


@pytest.mark.parametrize("path,shape,cfg", [(0, (256, 256, 256), 3), (0, (33, 70, 5000), 3), (0, (8192, 8192, 64), 0),
                                            (1, (64, 64, 64), 4), (2, (300, 200, 1000), 4), (4, (8192, 4096, 32), 2)])
def test_query_answers_for_a_batch_of_one(native, path, shape, cfg):
    assert native.mg_batched_config(path, *shape) == cfg


@pytest.mark.gpu
@pytest.mark.parametrize("path", [0, 1, 2, 4])
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (256, 256, 256), (700, 900, 40), (1000, 1500, 33), (2048, 1024, 32),
                                   (2500, 2100, 48), (5000, 3000, 32), (1, 1, 1)])
def test_launch_runs_the_tile_the_query_names(gpu, native, path, M, N, K):
    """The launch has a workgroup per tile, up to the GPU's slots."""
    import torch
    A, B, C = (torch.ones(s, device=gpu) for s in ((M, K), (K, N), (M, N)))
    arr = (native.mg_problem * 1)(native.mg_problem(b"N", b"N", M, N, K, 1.0, 0.0, A.data_ptr(), K, B.data_ptr(), N,
                                                    C.data_ptr(), N))
    ws = torch.empty(native.mg_gemm_batched_workspace_size(path, 1), dtype=torch.uint8, device=gpu)
    slots = native.mg_batched_slots(path)
    stamps = torch.zeros(2 * slots, dtype=torch.int64, device=gpu)
    st, _, grid = native.mg_gemm_batched_timed(path, 1, arr, ws.data_ptr(), ws.numel(),
                                               torch.cuda.current_stream().cuda_stream, stamps.data_ptr(), 2 * slots)
    assert st == 0
    bm, bn = TILE[path][native.mg_batched_config(path, M, N, K)]
    assert grid == min(-(-M // bm) * -(-N // bn), slots)
    assert torch.equal(C, torch.full_like(C, K))
