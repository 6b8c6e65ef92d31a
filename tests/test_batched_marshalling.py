"""gemm_batched's packed problem descriptors against the ctypes structure
filled through operand_layout and output_ld, over every layout it accepts
(CPU: the library call itself is replaced)."""
import ctypes
import itertools

import pytest
import torch

import paper_2305_18236_amd as pkg
from paper_2305_18236_amd import _native


def views(r, c):
    """The ways an r x c operand can be stored."""
    yield torch.zeros(r, c)
    yield torch.zeros(r, c + 3)[:, :c]
    yield torch.zeros(c, r).t()
    yield torch.zeros(c, r + 2)[:, :r].t()


@pytest.fixture()
def captured(monkeypatch):
    got = []

    def fake(path, count, arr, ws, nbytes, stream):
        got.append(bytes(ctypes.string_at(arr, count * ctypes.sizeof(_native.mg_problem))))
        return 0, -1

    monkeypatch.setattr(_native, "mg_gemm_batched", fake)
    monkeypatch.setattr(pkg, "_stream_ptr", lambda dev: 0)
    return got


@pytest.mark.parametrize("M,N,K", [(4, 5, 6), (1, 5, 6), (4, 1, 6), (4, 5, 1), (1, 1, 1), (0, 5, 6), (4, 0, 6), (4, 5, 0)])
def test_descriptors_equal_the_general_marshalling(captured, M, N, K):
    probs = []
    for A, B, C in itertools.product(views(M, K), views(K, N), list(views(M, N))[:2]):
        probs.append((A, B, C, 1.5, -0.5))
    probs.append((probs[0][0], probs[0][1], probs[0][2], 2, torch.tensor(0.25)))
    pkg.gemm_batched(probs)
    want = (_native.mg_problem * len(probs))()
    for i, (A, B, C, alpha, beta) in enumerate(probs):
        tA, lda = pkg.operand_layout(A)
        tB, ldb = pkg.operand_layout(B)
        want[i] = _native.mg_problem(tA.encode(), tB.encode(), M, N, K, float(alpha), float(beta), A.data_ptr(), lda,
                                     B.data_ptr(), ldb, C.data_ptr(), pkg.output_ld(C))
    for i in range(len(probs)):
        a = _native.mg_problem.from_buffer_copy(captured[0], i * ctypes.sizeof(_native.mg_problem))
        for name, _ in _native.mg_problem._fields_:
            assert getattr(a, name) == getattr(want[i], name), (i, name)


def test_what_was_refused_stays_refused(captured):
    a, b, c = torch.zeros(4, 6), torch.zeros(6, 5), torch.zeros(4, 5)
    with pytest.raises(TypeError):
        pkg.gemm_batched([(a.double(), b, c, 1.0, 0.0)])
    for bad in ((a, torch.zeros(7, 5), c), (a, b, torch.zeros(5, 4).t()), (a, b, torch.zeros(1, 5).expand(4, 5)),
                (torch.zeros(4, 1).expand(4, 6), b, c), (torch.zeros(4, 12)[:, ::2], b, c), (a, b, torch.zeros(4, 6))):
        with pytest.raises(ValueError):
            pkg.gemm_batched([bad + (1.0, 0.0)])
    assert not captured
