"""CPU model of which reference density the step kernel decodes each pulled
population with (FP16 storage with a per-node reference, LBM_F16R, bitmap
index): the halves of the 8-byte windows as they are picked, bit by bit,
against the neighbour table.

The reference array holds each node's own number here, so a pick is right
when it yields the source node of the table, or the node itself at a wall.
The array is preceded by two foreign entries, where the window of r0 = 0
starts.  Rows of one and two voxels are the ones whose wrapped sources lie
inside the window, beside or on r0."""
import numpy as np
import pytest

import paper_1902_11193_amd as P
from lbm_inputs import random_mask

ROW = (0, 0, 0, 1, 2, 3, 4, 1, 2, 2, 1, 3, 4, 4, 3, 5, 6, 7, 8)
WHICH = (0, -1, 1, 0, 0, 0, 0, -1, 1, -1, 1, -1, 1, -1, 1, 0, 0, 0, 0)


def direction(row, which):
    return next(i for i in range(1, 19) if ROW[i] == row and WHICH[i] == which)


def picked(t, b, xw, wb, lo, hi, wrap):
    """finish_refs: t, lo, hi and wrap by row."""
    two, nxt = [], []
    for r in range(9):
        sh = (t[r] << 3) & 31
        two.append(((hi[r] << 32 | lo[r]) >> sh) & 0xffffffff)
        if r <= 4:
            v = hi[r] >> sh
            nxt.append(two[r] >> 16 if r >= 1 and not (b >> r) & 1 else v)
    own = two[0] >> 16
    own2 = own | (two[0] & 0xffff0000)
    v = [0] + [nxt[ROW[i]] if WHICH[i] > 0 else two[ROW[i]] for i in range(1, 19)]
    for r in range(5):
        if xw & 1:
            v[direction(r, -1)] = wrap[r]
        if xw & 2:
            v[direction(r, 1)] = wrap[r]
    out = [own]
    for i in range(1, 19):
        s = own2 if (wb >> i) & 1 else v[i]
        out.append((s >> 16 if WHICH[i] == 0 else s) & 0xffff)
    return out


def row_nodes(mask):
    """r0 of every voxel: the fluid voxels of its row before it, counted from the row's first node."""
    nz, ny, nx = mask.shape
    order = P.lbm_node_order(mask)
    node = -np.ones(mask.size, np.int64)
    node[order] = np.arange(len(order))
    node = node.reshape(mask.shape)
    r0 = np.zeros(mask.shape, np.int64)
    for z in range(nz):
        for y in range(ny):
            fl = np.flatnonzero(mask[z, y] == 0)
            if len(fl):
                before = np.concatenate(([0], np.cumsum(mask[z, y] == 0)[:-1]))
                r0[z, y] = node[z, y, fl[0]] + before
    return order, r0


@pytest.mark.parametrize("nx", [1, 2, 3, 4, 19])
@pytest.mark.parametrize("ny,nz,solid,seed", [(6, 5, 0.0, 1), (2, 2, 0.0, 2), (1, 1, 0.0, 3), (6, 5, 0.35, 4),
                                              (7, 4, 0.6, 5)])
def test_every_population_takes_its_source_nodes_reference(nx, ny, nz, solid, seed):
    mask = random_mask((nz, ny, nx), solid, seed) if solid else np.zeros((nz, ny, nx), np.uint8)
    order, r0 = row_nodes(mask)
    nf = len(order)
    if nf == 0:
        pytest.skip("no fluid voxel")
    refs = np.concatenate(([60001, 60002], np.arange(nf), [60003] * 4)).tolist()   # entry m at [m + 2]
    table = P.lbm_neighbor_table(mask)
    c = P.lbm_velocities()
    # velocity of a direction that pulls from row R, per row
    dy = [-int(c[ROW.index(r)][1]) if r else 0 for r in range(9)]
    dz = [-int(c[ROW.index(r)][2]) if r else 0 for r in range(9)]
    for n in range(nf):
        v = int(order[n])
        x, y, z = v % nx, (v // nx) % ny, v // (nx * ny)
        rows = [((z + dz[r]) % nz, (y + dy[r]) % ny) for r in range(9)]
        t = [2 * int(r0[q][x]) + 2 for q in rows]
        b = sum((mask[rows[r]][x] == 0) << r for r in range(1, 5))
        at = [(tr & ~3) // 2 for tr in t]                    # window's first entry, from entry -2
        lo = [refs[a] | refs[a + 1] << 16 for a in at]
        hi = [refs[a + 2] | refs[a + 3] << 16 for a in at]
        xw = (x == 0) | (x == nx - 1) << 1
        src = [n] + [int(table[i - 1, n]) for i in range(1, 19)]
        wb = sum((src[i] < 0) << i for i in range(1, 19))
        # found from the gather offset (issue_refs); not loaded at a wall
        wrap = [max(src[direction(r, -1 if xw & 1 else 1)], 0) for r in range(5)]
        want = [m if m >= 0 else n for m in src]
        assert picked(t, b, xw, wb, lo, hi, wrap) == want, (n, x, y, z)
