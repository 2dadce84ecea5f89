"""Several steps in one launch (small images) against one launch a step: the
same state and per-step history bit for bit, at the edges of the chunk count
(one node, one chunk and one node more, the largest count that takes this
path and one chunk beyond it), for step counts that end in either buffer and
need more than one launch; with the blocks' meeting cut short, so that one
block does all the work; and with contexts on several streams at once that
do not fit the GPU together.  The single-step launches are held to the
oracle by the parity tests."""
import threading

import numpy as np
import pytest
import torch

import paper_1902_11193_amd as P
from gpu_helpers import banner, random_state

pytestmark = pytest.mark.gpu

G = (1e-5, 2e-6, -1e-6)
SYNC_BYTES = 65792      # the barrier memory, before the reduction scratch at the workspace's end


def image(nodes, shape, seed=3):
    """An image of exactly `nodes` fluid voxels at random places."""
    m = np.ones(int(np.prod(shape)), np.uint8)
    m[np.random.default_rng(seed).permutation(m.size)[:nodes]] = 0
    return m.reshape(shape)


def solver(mask, graphs=True, storage="f32", index="bitmap", boundary="", seed=4):
    g = (0.0, 0.0, 0.0) if boundary == "pressure" else G
    s = P.Solver(mask, 0.9, 3 / 16, "E", g, storage, index)
    s.set_graphs(graphs)
    if boundary == "mirror_fullway":
        s.set_symmetry(True, True)
        s.set_wall("fullway")
    elif boundary == "pressure":
        s.set_pressure(1.001, 0.999)
    s.set_state(random_state(s.n_fluid, seed))
    return s


def same(a, b, done):
    assert np.array_equal(a.get_state(), b.get_state())
    assert np.array_equal(a.history(done), b.history(done))


@pytest.mark.parametrize("nodes,shape,storage,index,boundary", [
    (1, (2, 3, 4), "f32", "bitmap", ""),
    (256, (7, 9, 11), "f16", "bitmap", ""),
    (257, (7, 9, 11), "bf16", "table", ""),
    (257, (7, 9, 11), "f16r", "table", ""),
    (5000, (20, 21, 22), "f16r", "bitmap", ""),
    (5000, (20, 21, 22), "f32", "bitmap", "mirror_fullway"),
    (5000, (20, 21, 22), "f32", "bitmap", "pressure"),
    (65 * 256, (30, 31, 32), "f32", "table", ""),
    (896 * 256, (64, 63, 65), "f32", "bitmap", ""),
    (896 * 256 + 1, (64, 63, 65), "f32", "bitmap", ""),
])
def test_steps_in_one_launch_equal_single_launches(nodes, shape, storage, index, boundary):
    banner(f"steps in one launch: {nodes} nodes {shape} {storage} {index} {boundary}")
    mask = image(nodes, shape)
    a, b = (solver(mask, g, storage, index, boundary) for g in (True, False))
    done = 0
    for n in (4, 1, 37, 2, 130):
        a.step(n)
        b.step(n)
        done += n
        same(a, b, done)
    a.close()
    b.close()


@pytest.mark.parametrize("boundary", ["", "mirror_fullway"])
def test_one_block_takes_over_when_the_others_do_not_come(boundary):
    banner(f"meeting cut short {boundary}")
    mask = image(9000, (25, 26, 27))
    a, b = (solver(mask, g, boundary=boundary) for g in (True, False))
    at = a.workspace.numel() - P.LBM_REDUCTION_BYTES - SYNC_BYTES
    a.workspace[at + 8:at + 12].view(torch.int32).fill_(1)     # 10 ns
    done = 0
    for n in (5, 8):
        a.step(n)
        b.step(n)
        done += n
        same(a, b, done)
    a.close()
    b.close()


def test_adjoint_equals_single_launches():
    banner("adjoint, steps in one launch")
    mask = image(6000, (22, 23, 24))
    r = []
    for g in (True, False):
        s = solver(mask, g)
        r.append(s.adjoint(47, 9))
        s.close()
    assert r[0]["k"] == r[1]["k"] and r[0]["dk_dtau"] == r[1]["dk_dtau"] and r[0]["dk_dLambda"] == r[1]["dk_dLambda"]
    assert torch.equal(r[0]["dk_dg"], r[1]["dk_dg"])


def test_contexts_on_several_streams():
    """Three streams, contexts of 600 chunks (no two fit the GPU together) and of 40."""
    banner("three streams")
    masks = [image(n, (64, 63, 65), k) for k, n in enumerate((600 * 256, 600 * 256 - 7, 40 * 256))]
    want = []
    for m in masks:
        s = solver(m, False)
        s.step(160)
        want.append((s.get_state(), s.history(160)))
        s.close()
    got = [None] * 3

    def work(k):
        torch.cuda.set_device(0)
        with torch.cuda.stream(torch.cuda.Stream()):
            s = solver(masks[k])
            for _ in range(8):
                s.step(20)
            got[k] = (s.get_state(), s.history(160))
            s.close()

    th = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for w, g in zip(want, got):
        assert np.array_equal(w[0], g[0]) and np.array_equal(w[1], g[1])
