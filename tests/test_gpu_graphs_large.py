"""Captured-graph replay on images of more than 896 chunks, which take one step
a launch: replays give the state and history of plain launches bit for bit, in
every storage, across settings changes that drop the graphs and through
lbm_setup_static, with the program's own reads and single steps in between.
No launch of several steps takes part: its finished-steps words stay at zero."""
import numpy as np
import pytest
import torch

import paper_1902_11193_amd as P
from gpu_helpers import banner, random_state

pytestmark = pytest.mark.gpu

G = (1e-5, 2e-6, 0.0)
SHAPE = (63, 64, 65)
SYNC_BYTES = 65792      # the barrier memory, before the reduction scratch at the workspace's end


def image(nodes=897 * 256 + 3):
    m = np.ones(int(np.prod(SHAPE)), np.uint8)
    m[np.random.default_rng(3).permutation(m.size)[:nodes]] = 0
    return m.reshape(SHAPE)


def pair(storage, static=False):
    mask = image()
    a = P.Solver(mask, 0.9, 3 / 16, "E", G, storage, "bitmap", static_scratch=static)
    b = P.Solver(mask, 0.9, 3 / 16, "E", G, storage, "bitmap")
    b.set_graphs(False)
    f0 = random_state(a.n_fluid, 4)
    a.set_state(f0)
    b.set_state(f0)
    return a, b


def same(a, b, done):
    assert np.array_equal(a.get_state(), b.get_state()), done
    assert np.array_equal(a.history(done), b.history(done)), done


def no_several(a, static=False):
    at = a.workspace.numel() - (0 if static else P.LBM_REDUCTION_BYTES) - SYNC_BYTES
    w = a.workspace[at:at + SYNC_BYTES].view(torch.int32)
    assert int(w.abs().max()) == 0


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16", "f16r"])
def test_replays_equal_plain_launches(storage):
    banner(f"graphs, 898 chunks {storage}")
    a, b = pair(storage)
    done = 0
    for n in (1, 32, 65, 31, 96, 3, 64):
        a.step(n)
        b.step(n)
        done += n
        same(a, b, done)
    no_several(a)
    a.close()
    b.close()


def test_replays_follow_settings_changes():
    banner("graphs across settings, 898 chunks")
    a, b = pair("f32")
    field = (1e-5 * torch.randn(3, a.n_fluid, generator=torch.Generator().manual_seed(1))).cuda()
    done = 0
    for change in (lambda s: None, lambda s: s.set_collision("trt"), lambda s: s.set_force_field(field),
                   lambda s: s.set_wall("fullway"), lambda s: s.set_symmetry(True, False),
                   lambda s: (s.set_wall("halfway"), s.set_force_field(None), s.set_symmetry(False, False)),
                   lambda s: s.set_collision("mrt")):
        for s in (a, b):
            change(s)
            s.step(70)
        done += 70
        same(a, b, done)
    no_several(a)
    a.close()
    b.close()


def test_replays_follow_the_storage_exponent():
    banner("graphs across exponents, 898 chunks")
    a, b = pair("f16r")
    for e in (12, 17, 12):
        for s in (a, b):
            s.set_storage_exponent(e)
            s.step(70)
    same(a, b, 210)
    a.close()
    b.close()


def test_replays_with_the_static_scratch():
    banner("graphs, static scratch, 898 chunks")
    a, b = pair("f16", static=True)
    for n in (1, 70, 33):
        a.step(n)
        b.step(n)
    same(a, b, 104)
    no_several(a, static=True)
    a.close()
    b.close()
