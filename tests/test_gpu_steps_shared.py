"""Several steps in one launch where its blocks do not all get room in time:
the launch closes its count and the blocks share the chunk-steps.  Forced from
the host through the meeting time's word, or by kernels of another stream that
hold the GPU; results are those of single launches, bit for bit, and the work is
shared: such a launch may not take a hundred times longer."""
import time

import numpy as np
import pytest
import torch

import paper_1902_11193_amd as P
from gpu_helpers import banner, random_state

pytestmark = pytest.mark.gpu

G = (1e-5, 2e-6, -1e-6)
SYNC_BYTES = 65792      # the barrier memory, before the reduction scratch at the workspace's end


def image(nodes, shape, seed=3):
    m = np.ones(int(np.prod(shape)), np.uint8)
    m[np.random.default_rng(seed).permutation(m.size)[:nodes]] = 0
    return m.reshape(shape)


def solver(mask, graphs, storage="f32", index="bitmap", boundary=""):
    g = (0.0, 0.0, 0.0) if boundary == "pressure" else G
    s = P.Solver(mask, 0.9, 3 / 16, "E", g, storage, index)
    s.set_graphs(graphs)
    if boundary == "mirror_fullway":
        s.set_symmetry(True, True)
        s.set_wall("fullway")
    elif boundary == "pressure":
        s.set_pressure(1.001, 0.999)
    s.set_state(random_state(s.n_fluid, 4))
    return s


def words(s):
    at = s.workspace.numel() - P.LBM_REDUCTION_BYTES - SYNC_BYTES
    return s.workspace[at:at + SYNC_BYTES].view(torch.int32)


MEET, BLOCKS = 2, 64


def closed(s):
    """Launches whose blocks did not all meet: the second word behind the ring."""
    return int(s.workspace[-33024 + 32768:].view(torch.int32)[1])


@pytest.mark.parametrize("nodes,shape,storage,index,boundary", [
    (1, (2, 3, 4), "f32", "bitmap", ""),
    (300, (7, 9, 11), "f16", "table", ""),
    (64 * 256, (30, 31, 32), "bf16", "bitmap", ""),
    (5000, (20, 21, 22), "f16r", "bitmap", ""),
    (5000, (20, 21, 22), "f16r", "table", ""),
    (9000, (25, 26, 27), "f32", "bitmap", "mirror_fullway"),
    (9000, (25, 26, 27), "f32", "bitmap", "pressure"),
    (896 * 256, (64, 63, 65), "f32", "bitmap", ""),
])
def test_closed_counts_equal_single_launches(nodes, shape, storage, index, boundary):
    banner(f"closed count: {nodes} nodes {shape} {storage} {index} {boundary}")
    mask = image(nodes, shape)
    a, b = (solver(mask, g, storage, index, boundary) for g in (True, False))
    w = words(a)
    chunks = -(-nodes // 256)
    done = told = 0
    for n, meet in ((5, -1), (12, 0), (16, -1), (17, 1)):     # closed, open, closed, 10 ns
        w[MEET] = meet
        a.step(n)
        b.step(n)
        done += n
        told += n + 1
        assert np.array_equal(a.get_state(), b.get_state()), n
        # the words of every chunk, whoever stepped it, and the counts back at zero
        assert (w[BLOCKS::16][:chunks] == told).all() and w[0] == 0 and w[1] == 0 and w[4] == 0 and w[16] == 0
    assert 2 <= closed(a) <= 3
    assert np.array_equal(a.history(done), b.history(done))   # (which has the next calls take single steps)
    a.close()
    b.close()


def test_closed_counts_in_the_adjoint():
    banner("closed count, adjoint")
    mask = image(6000, (22, 23, 24))
    r = []
    for meet in (0, -1):
        s = solver(mask, True)
        words(s)[MEET] = meet
        r.append(s.adjoint(60, 20))
        assert closed(s) == (0 if meet == 0 else 5)    # 2 forward, 1 kept, 2 recomputed segments
        s.close()
    assert r[0]["k"] == r[1]["k"] and r[0]["dk_dtau"] == r[1]["dk_dtau"] and r[0]["dk_dLambda"] == r[1]["dk_dLambda"]
    assert torch.equal(r[0]["dk_dg"], r[1]["dk_dg"])


def test_blocks_share_the_work_of_a_closed_count():
    banner("closed count, time")
    s = solver(image(800 * 256, (64, 63, 65)), True)
    t = {}
    for meet in (0, -1):
        words(s)[MEET] = meet
        s.step(20)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(5):
            s.step(20)
        torch.cuda.synchronize()
        t[meet] = time.perf_counter() - t0
    print(f"100 steps of 800 chunks: open {1e3 * t[0]:.2f} ms, closed {1e3 * t[-1]:.2f} ms")
    assert t[-1] < 30 * t[0]     # one block alone: 800 times the work of a block
    s.close()


def test_beside_kernels_of_another_stream():
    """Large elementwise kernels on a second stream take every compute unit in turn."""
    banner("beside other kernels")
    mask = image(800 * 256, (64, 63, 65))
    b = solver(mask, False)
    b.step(300)
    want = b.get_state(), b.history(300)
    b.close()
    s = solver(mask, True)
    x = torch.zeros(1 << 28, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        for _ in range(60):
            x.add_(1.0)
    s.step(300)
    assert np.array_equal(s.get_state(), want[0]) and np.array_equal(s.history(300), want[1])
    torch.cuda.synchronize()
    print(f"counts closed: {closed(s)} of {-(-300 // 20)} launches")
    assert float(x[0]) == 60.0 and float(x[-1]) == 60.0
    s.close()
