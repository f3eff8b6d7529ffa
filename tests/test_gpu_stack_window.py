"""Gathers that read the stack through windows staged in LDS (the cone lattice
of every row stack, all directional gathers of the 2-byte row stacks) against
gathers that read the stack itself, at the sizes where a window meets the
stored range: grids and slab counts about the window's own size, taps past
the grid, and reaches that leave the window little or no room.

The tiled layout never stages, so for the float and bfloat16 stacks its image
is the same bits.  The half stack exists in rows only: its texels are within
2^-12 of the float ones (rounding of a value at most 1), a gather averages
texels, and a pixel is a sum of emissions of total weight at most 1 times the
coefficient, so its image is within 2^-12 of the float stack's, plus 1e-5 for
the rounding of up to some hundred segments."""
import pytest
import torch

from paper_2008_06134_amd import vi
from paper_2008_06134_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"

# (slabs, res): about the windows' 16 x 8 or 16 rows x 4, 5 or 6 layers
SIZES = [(1, 8), (2, 12), (3, 13), (4, 16), (5, 17), (9, 12), (33, 40)]
GATHERS = [("cone", {"cone_grid": 2}), ("cone", {"cone_grid": 5}), ("cone", {"cone_grid": 7, "cone_tan": 3.0}),
           ("cone", {}), ("cone", {"cone_rings": 3, "cone_angles": 5}), ("cone", {"cone_rings": 1, "cone_tan": 0.0}),
           ("shell", {}), ("shell", {"shell_count": 3}), ("shell", {"shell_h_vox": 8.0})]


def compare(slabs, res, cams, gathers):
    raw = W.sphere_u8(24, radius=9.5, seed=7)
    tf = vi.TF.from_numpy(W.tf_ramp(), DEV)
    vol = vi.Volume.from_numpy(raw, DEV).to_quads().with_minmax(8).with_occupancy(tf)
    for light in (W.DIAGONAL_LIGHT, [0.0, 0.0, -1.0]):
        st = {}
        for dt, layout in ((vi.VI_F32, 0), (vi.VI_F32, 1), (vi.VI_BF16, 0), (vi.VI_BF16, 1), (vi.VI_F16, 1)):
            st[dt, layout] = vi.build_attenuation(vol, tf, light, slabs, res, dt, layout=layout)
        for cam in cams:
            for mode, opts in gathers:
                img = {k: vi.render(vol, tf, s, cam, mode, 0.5, opts) for k, s in st.items()}
                torch.cuda.synchronize()
                what = f"{slabs} slabs of {res}^2, {mode} {opts}, {cam['width']}x{cam['height']}"
                for dt in (vi.VI_F32, vi.VI_BF16):
                    assert torch.equal(img[dt, 0], img[dt, 1]), what
                off = float((img[vi.VI_F16, 1] - img[vi.VI_F32, 1]).abs().max())
                assert off <= 2.0 ** -12 + 1e-5, (what, off)


@pytest.mark.parametrize("slabs,res", SIZES)
def test_window_equals_stack(slabs, res):
    compare(slabs, res, (W.camera_orbit(41, 37, 0.7, 0.4), W.camera_ortho_front(64, 48), W.camera_ortho_front(9, 7)),
            GATHERS)


@pytest.mark.parametrize("slabs,res", SIZES + [(9, 350), (20, 520)])
def test_window_equals_stack_larger_images(slabs, res):
    """Images on both sides of the sizes from which a frame stages: cubes of 70 K and
    110 K pixels, rays 0.01 to 0.9 texels apart, and one of 40 K."""
    compare(slabs, res, (W.camera_orbit(569, 391, 0.7, 0.4), W.camera_orbit(641, 487, -0.4, 0.9),
                         W.camera_ortho_front(641, 487), W.camera_orbit(401, 299, 0.7, 0.4)), GATHERS)
