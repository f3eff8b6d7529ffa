"""Which frames read the stack through a window (host only): what decides it are
the taps a sample, the pixels that the cube covers, the texels between
neighbouring rays and the room that the frame's tables leave in LDS."""
import pytest

import frame_harness as H
from paper_2008_06134_amd import vi
from paper_2008_06134_amd import workloads as W

F32, BF16, F16 = vi.VI_F32, vi.VI_BF16, vi.VI_F16


def _decision(edge, slabs, res, dtype, size, mode, opts, entries=256, position=None):
    s = vi.light_frame(W.DIAGONAL_LIGHT, slabs, res, dtype, vi.VI_STACK_ROWS, position=position).s
    s.data, s.vol_n = 1 << 20, edge
    vol = vi.Volume_t(1 << 20, vi.VI_U16, edge, 1.0 / 4095.0, vi.VI_LAYOUT_QUAD4, None, 0)
    cam = W.camera_orbit(*size, 0.7, 0.4)
    return H.window(vol, vi.TF_t(1 << 20, entries, 1), s, cam, mode, 0.5, opts)


LARGE, MEDIUM = (512, 512, 1024), (256, 256, 512)
HD, MP = (1920, 1080), (1024, 1024)   # 550 K and 494 K pixels of the cube


@pytest.mark.parametrize("scene,dtype,size,mode,opts,entries,staged", [
    (MEDIUM, F32, MP, "cone", {"cone_grid": 5}, 256, True),
    (LARGE, F32, HD, "cone", {"cone_grid": 5}, 256, True),
    (MEDIUM, F32, MP, "cone", {"cone_grid": 3}, 256, True),
    (MEDIUM, BF16, MP, "shell", {}, 256, True),
    (MEDIUM, F16, MP, "shell", {"shell_count": 2}, 256, True),
    (MEDIUM, F16, MP, "cone", {}, 256, True),
    # 2-byte lattices far apart or on smaller images
    (LARGE, BF16, (640, 600), "cone", {"cone_grid": 5}, 256, True),
    (MEDIUM, BF16, (400, 420), "cone", {"cone_grid": 5}, 256, True),
    # few taps save less than the window costs
    (MEDIUM, BF16, MP, "cone", {"cone_grid": 1}, 256, False),
    (LARGE, BF16, HD, "cone", {"cone_grid": 2}, 256, False),
    (LARGE, F32, HD, "cone", {"cone_grid": 1}, 256, False),
    (MEDIUM, F16, MP, "cone", {"cone_rings": 1, "cone_angles": 2}, 256, False),
    (MEDIUM, BF16, MP, "cone", {"cone_rings": 2, "cone_angles": 2}, 256, False),
    # large tables leave room for four workgroups
    (MEDIUM, BF16, MP, "cone", {}, 1024, False),
    (MEDIUM, F32, MP, "cone", {"cone_grid": 3}, 1024, False),
    (MEDIUM, F32, MP, "cone", {"cone_grid": 5}, 1024, True),
    # one round of waves, or rays far apart
    (MEDIUM, F32, (256, 256), "cone", {"cone_grid": 5}, 256, False),
    (MEDIUM, BF16, (400, 300), "shell", {}, 256, False),
    (LARGE, F32, (640, 600), "cone", {"cone_grid": 5}, 256, False),
    # gathers and lookups without windows
    (MEDIUM, F32, MP, "shell", {}, 256, False),
    (MEDIUM, F32, MP, "cone", {}, 256, False),
    (MEDIUM, BF16, MP, "shadow", {}, 256, False),
    (MEDIUM, BF16, MP, "cone", {"cone_grid": 5, "nearest_layer": 1}, 256, False),
])
def test_rule(scene, dtype, size, mode, opts, entries, staged):
    assert _decision(*scene, dtype, size, mode, opts, entries)[1] == staged


def test_a_window_that_does_not_fit_is_never_staged():
    # reach of 2 sqrt(2) x 4 texels; fewer layers than a window; a point light
    assert _decision(256, 128, 512, F32, MP, "cone", {"cone_grid": 5, "cone_tan": 2.0}) == (False, False)
    assert _decision(256, 1, 512, F32, MP, "cone", {"cone_grid": 5}) == (False, False)
    assert _decision(*MEDIUM, F32, MP, "cone", {"cone_grid": 5}, position=[1.9, -0.4, 2.1]) == (False, False)
