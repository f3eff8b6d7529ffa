"""The elements of the row layout that the header says are never read (columns
res+4 .. P-1 of a row and the rest of a layer behind its rows) may hold
anything: a stack whose padding is NaN renders to the same bits.  The cube is
opaque up to its corners, which lie within a thirtieth of the grid's edge under
a diagonal light, and the gathers reach up to five texels further, past the
border; images are of the size from which gathers read the stack through
windows staged in LDS."""
import numpy as np
import pytest
import torch

from paper_2008_06134_amd import vi
from paper_2008_06134_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"

GATHERS = [("cone", {"cone_grid": 5}), ("cone", {"cone_rings": 1, "cone_tan": 1.4}), ("cone", {}), ("shell", {}),
           ("shadow", {})]


@pytest.mark.parametrize("res", [40, 41, 42, 43])
@pytest.mark.parametrize("dtype", [vi.VI_F32, vi.VI_BF16, vi.VI_F16])
def test_padding_is_never_read(dtype, res):
    slabs = 12
    tf = vi.TF.from_numpy(W.tf_ramp(), DEV)
    vol = vi.Volume.from_numpy(np.full((24, 24, 24), 30, np.uint8), DEV).to_quads()
    cams = (W.camera_ortho_front(641, 487), W.camera_orbit(641, 487, -2.3, 0.6), W.camera_orbit(641, 487, 0.8, -0.6))
    for light in (W.DIAGONAL_LIGHT, [-a for a in W.DIAGONAL_LIGHT]):
        buf = vi.stack_buffer(slabs, res, dtype, DEV, 1)
        st = vi.build_attenuation(vol, tf, light, slabs, res, dtype, buf, layout=1)
        images = [vi.render(vol, tf, st, cam, mode, 0.5, opts) for cam in cams for mode, opts in GATHERS]
        buf.as_strided((slabs + 2, res + 4, vi.row_pitch(res, dtype) - res - 4), buf.stride(), res + 4).fill_(np.nan)
        flat = buf.as_strided((slabs + 2, vi.row_layer(res, dtype)), (vi.row_layer(res, dtype), 1))
        flat[:, (res + 4) * vi.row_pitch(res, dtype):] = np.nan
        again = [vi.render(vol, tf, st, cam, mode, 0.5, opts) for cam in cams for mode, opts in GATHERS]
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(images, again)):
            assert torch.equal(a, b), (i // len(GATHERS), GATHERS[i % len(GATHERS)], light)
