"""The gathers that can read the stack through a window staged in LDS, with the
window switched on and off for the same frame, whatever the rule that decides
it would say: grids and slab counts about the window's own size with small
images, and volumes fine enough that a step's samples lie 0.2 to 1.9 texels
apart, so that some of a wave's samples fit the window and the others read the
stack.  Both read the same texels with the same weights, so the images are the
same bits; and so is the tiled layout's, which has no windows.  Every
combination that is meant to fit asserts that it does."""
import pytest
import torch

import frame_harness as H
from paper_2008_06134_amd import vi
from paper_2008_06134_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"

GATHERS = [("cone", {"cone_grid": 1}), ("cone", {"cone_grid": 2}), ("cone", {"cone_grid": 5}),
           ("cone", {"cone_grid": 7, "cone_tan": 0.5}), ("cone", {}), ("cone", {"cone_rings": 3, "cone_angles": 5}),
           ("cone", {"cone_rings": 1, "cone_angles": 3, "cone_tan": 2.0}), ("shell", {}), ("shell", {"shell_count": 2}),
           ("shell", {"shell_h_vox": 0.5})]


def compare(vol, tf, slabs, res, cams, lights=(W.DIAGONAL_LIGHT, [0.0, 0.0, -1.0], [0.3, -0.8, 0.5])):
    """Renders every gather that fits with the window on and off; returns those."""
    fitted = set()
    for light in lights:
        for dt in (vi.VI_F32, vi.VI_BF16, vi.VI_F16):
            rows = vi.build_attenuation(vol, tf, light, slabs, res, dt, layout=1)
            tiled = None if dt == vi.VI_F16 else vi.build_attenuation(vol, tf, light, slabs, res, dt, layout=0)
            for cam in cams:
                for i, (mode, opts) in enumerate(GATHERS):
                    if not H.window(vol.s, tf.s, rows.s, cam, mode, 0.5, opts)[0]:
                        continue
                    fitted.add((dt, i))
                    on, off = (H.render(vol, tf, rows, cam, mode, 0.5, opts, s) for s in (1, 0))
                    torch.cuda.synchronize()
                    what = f"{slabs} slabs of {res}^2, dtype {dt}, {mode} {opts}, {cam['width']}x{cam['height']}"
                    assert float(off[..., 3].max()) > 0.5, what
                    assert torch.equal(on, off), what
                    if tiled is not None:
                        assert torch.equal(on, vi.render(vol, tf, tiled, cam, mode, 0.5, opts)), what
    return fitted


@pytest.mark.parametrize("slabs,res", [(1, 12), (2, 12), (3, 13), (4, 16), (5, 17), (9, 12), (33, 41)])
def test_small_grids(slabs, res):
    vol = vi.Volume.from_numpy(W.sphere_u8(24, radius=11.5, seed=7), DEV).to_quads()
    tf = vi.TF.from_numpy(W.tf_ramp(), DEV)
    vol = vol.with_minmax(8).with_occupancy(tf)
    fitted = compare(vol, tf, slabs, res, (W.camera_orbit(41, 37, 0.7, 0.4), W.camera_ortho_front(64, 48),
                                           W.camera_ortho_front(9, 7)))
    # a lattice of one tap fits wherever the window's 4 layers do
    assert ((vi.VI_F32, 0) in fitted) == (slabs >= 2)
    if slabs >= 9:
        assert {(vi.VI_BF16, 7), (vi.VI_F16, 4), (vi.VI_F32, 2)} <= fitted


@pytest.mark.parametrize("N,slabs,res,image", [(128, 200, 350, 200), (128, 256, 520, 300), (256, 256, 512, 560),
                                               (256, 300, 413, 240), (100, 90, 180, 640)])
def test_fine_grids(N, slabs, res, image):
    """apart = texels between neighbouring pixels' rays: 0.2 to 1.9 over these."""
    vol = vi.Volume.from_numpy(W.sphere_u8(N, radius=0.47 * N, seed=5), DEV).to_quads()
    tf = vi.TF.from_numpy(W.tf_ramp(), DEV)
    vol = vol.with_minmax(16).with_occupancy(tf)
    fitted = compare(vol, tf, slabs, res, (W.camera_orbit(image, image * 3 // 4, 0.7, 0.4), W.camera_ortho_front(image, image)))
    want = {0, 1, 2, 3, 4, 7, 9}
    assert want <= {i for dt, i in fitted if dt == vi.VI_BF16}, fitted
    assert want <= {i for dt, i in fitted if dt == vi.VI_F16}, fitted
    assert {0, 1, 2, 3} <= {i for dt, i in fitted if dt == vi.VI_F32}, fitted
