"""Index algebra of the panel loads at the edges of a matrix (CPU model).

The FP32 and 16-bit tiles read whole 4-element chunks at clamped offsets where
a panel overhangs the matrix in m or n, and edge_load / edge_fix where it
overhangs in K; the packs read 4 floats or 16 bytes the same way.  Modelled
here address by address: no read leaves the stored matrix, every element that
can reach a stored output is the right one, and everything beyond K reads 0.
"""
import itertools

import numpy as np
import pytest


def edge(mem, ld, gr, gc, R, Cn, W):
    """edge_load then edge_fix: W values of stored row gr from column gc."""
    p = min(gr, R - 1) * ld
    if Cn >= W:
        at = p + min(gc, Cn - W)
        idx = np.arange(at, at + W)
    else:
        idx = p + np.minimum(gc + np.arange(W), Cn - 1)
    assert idx.min() >= 0 and idx.max() <= (R - 1) * ld + Cn - 1
    w = mem[idx]
    left = max(0, min(W, Cn - gc))
    keep = left if gr < R else 0
    sh = W - left if Cn >= W else 0
    if sh < W:                       # a chunk wholly outside is cleared by `keep`
        w = np.concatenate([w[sh:], np.zeros(sh, mem.dtype)])
    return np.where(np.arange(W) < keep, w, 0)


@pytest.mark.parametrize("W", [4, 16])
def test_edge_fetch_reads_the_matrix_and_zero_outside(W):
    for R, Cn, pad in itertools.product((1, 2, 5), (1, 3, 4, 5, 15, 16, 17, 33), (0, 1, 3)):
        ld = Cn + pad
        mem = np.arange(1, (R - 1) * ld + Cn + 1, dtype=np.int64)
        for gr, gc in itertools.product(range(R + 2), range(0, Cn + 2 * W, W)):
            want = [mem[gr * ld + gc + e] if gr < R and gc + e < Cn else 0 for e in range(W)]
            assert edge(mem, ld, gr, gc, R, Cn, W).tolist() == want


@pytest.mark.parametrize("kmajor", [False, True])
@pytest.mark.parametrize("B,BK", [(32, 32), (64, 32), (128, 16)])
def test_panel_loads_stay_inside_and_deliver_every_stored_element(kmajor, B, BK):
    for MN, K, pad in itertools.product((1, 3, 4, 5, 31, 64, 65, 130), (1, 15, 32, 33, 64), (0, 1, 2)):
        R, Cn = (K, MN) if kmajor else (MN, K)
        ld = Cn + pad
        mem = np.arange(1, (R - 1) * ld + Cn + 1, dtype=np.int64)
        SR, SC = (BK, B) if kmajor else (B, BK)
        for mn0, k0 in itertools.product(range(0, MN, B), range(0, K, BK)):
            r0, c0 = (k0, mn0) if kmajor else (mn0, k0)
            whole = r0 + SR + (c0 + SC > Cn and Cn % 4 != 0) <= R if kmajor else c0 + SC <= Cn
            fast = Cn >= 4 and whole
            last = min(SC - 4, (Cn - 1 - c0) & ~3) if kmajor else min(SR - 1, R - 1 - r0)
            for r, c in itertools.product(range(SR), range(0, SC, 4)):
                if fast:
                    at = (r0 + r) * ld + c0 + min(c, last) if kmajor else (r0 + min(r, last)) * ld + c0 + c
                    assert at >= 0 and at + 3 <= (R - 1) * ld + Cn - 1
                    got = mem[at:at + 4]
                else:
                    got = edge(mem, ld, r0 + r, c0 + c, R, Cn, 4)
                for e in range(4):
                    gr, gc = r0 + r, c0 + c + e
                    mn, k = (gc, gr) if kmajor else (gr, gc)
                    if mn < MN and k < K:
                        assert got[e] == mem[gr * ld + gc]
                    elif k >= K:
                        assert not fast and got[e] == 0
