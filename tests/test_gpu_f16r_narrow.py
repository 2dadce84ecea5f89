"""FP16 storage with a per-node reference density on images of one and two
voxels along x, where both wrapped neighbours of a voxel are the voxel itself
or its only neighbour: the bitmap index decodes every population against the
same reference as the table index, bit for bit, in single-step launches and in
several steps a launch, and stays with the FP64 oracle."""
import numpy as np
import pytest

import oracle as O
import paper_1902_11193_amd as P
from gpu_helpers import W_LIB, banner, dense_from_lib, lib_from_dense
from lbm_inputs import random_mask

pytestmark = pytest.mark.gpu


def dense_state(nf, seed):
    """A density deviation 1e3 times the velocity part: a wrong reference shows at once."""
    rng = np.random.default_rng(seed)
    f = W_LIB[:, None] * (1.0 + 1e-3 * rng.standard_normal(nf)[None, :])
    return f + 1e-6 * rng.standard_normal((19, nf))


@pytest.mark.parametrize("nx", [1, 2, 3])
@pytest.mark.parametrize("ny,nz,solid", [(2, 2, 0.0), (7, 5, 0.3), (40, 30, 0.3)])
def test_narrow_images_table_and_bitmap_agree(nx, ny, nz, solid):
    mask = random_mask((nz, ny, nx), solid, 5) if solid else np.zeros((nz, ny, nx), np.uint8)
    banner(f"f16r table vs bitmap {mask.shape}")
    g = (1e-5, 2e-6, -1e-6)
    s = {i: P.Solver(mask, 0.9, 1 / 12, "E", g, "f16r", i) for i in ("table", "bitmap")}
    f0 = dense_state(s["table"].n_fluid, 2)
    p = O.Problem(mask, 0.9, 1 / 12, "E", g)
    done = 0
    for v in s.values():
        v.set_state(f0)
    fh = dense_from_lib(p, s["table"].get_state())
    for n in (1, 2, 20):                 # the last one takes several steps a launch
        out = []
        for v in s.values():
            v.step(n)
            out.append(v.get_state())
        done += n
        assert np.array_equal(out[0], out[1]), n
        for _ in range(n):
            fh, _ = p.step(fh)
        ref = lib_from_dense(p, fh)
        small = ref - W_LIB[:, None] * ref.sum(0)[None, :]
        # the bound of the wider images' comparison (FP16 rounding of the velocity part over 23 steps)
        assert np.abs(out[1] - ref).max() < 5e-3 * np.abs(small).max(), n
    assert np.array_equal(s["table"].history(done), s["bitmap"].history(done))
    for v in s.values():
        v.close()
