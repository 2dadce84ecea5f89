"""The sums over the image do not depend on how the steps are launched: the
block sums are grouped alike, also at the chunk counts where the blocks of a
single step no longer all fit the GPU at once (F16R: three per compute unit,
768).  Every pore is a single voxel, which keeps its density: large ones of
either sign that cancel over the image and small ones of six decades less, so
that sums grouped differently leave other rounding errors."""
import numpy as np
import pytest

import paper_1902_11193_amd as P
from gpu_helpers import W_LIB, banner

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,collision", [("f16r", "mrt"), ("f16r", "trt"), ("f32", "mrt")])
@pytest.mark.parametrize("chunks", [768, 769, 896])
def test_sums_do_not_depend_on_the_launches(chunks, storage, collision):
    banner(f"sums {chunks} chunks {storage} {collision}")
    nf = chunks * 256 - 6
    mask = np.ones((124, 124, 124), np.uint8)
    pores = np.zeros((62, 62, 62), bool)
    pores.reshape(-1)[:nf] = True
    mask[::2, ::2, ::2][pores] = 0
    rng = np.random.default_rng(4)
    half = 10.0 ** rng.uniform(2, 4, nf // 2) * rng.choice([-1.0, 1.0], nf // 2)
    small = rng.random(nf // 2) < 0.1
    drho = np.concatenate([half, -half]).astype(np.float16).astype(np.float64)   # kept whole in the reference
    drho[np.concatenate([small, small])] = 1e-3 * rng.standard_normal(2 * small.sum())
    out = []
    for graphs, calls in ((True, (16,)), (True, (3, 3, 7, 3)), (False, (16,))):
        s = P.Solver(mask, 0.9, 3 / 16, "E", (1e-5, 2e-6, -1e-6), storage, "bitmap")
        s.set_graphs(graphs)
        s.set_collision(collision)
        s.set_state(W_LIB[:, None] * (1 + drho))
        for n in calls:
            s.step(n)
        out.append((s.history(16), s.mass_deviation(), s.get_state()))
        s.close()
    for o in out[1:]:
        assert np.array_equal(o[0], out[0][0]) and o[1] == out[0][1]
        assert np.array_equal(o[2], out[0][2])
