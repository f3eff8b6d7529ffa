"""The tiled build where rows of more than 800 texels of a linear volume take
four slabs at a time, against the row layout's build (which shares a column's
arithmetic but neither its mapping, its batches nor its stores), bit for bit:
slab counts that leave a remainder of every size, and both kinds of light."""
import pytest
import torch

from paper_2008_06134_amd import vi
from paper_2008_06134_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("kind", ["u8", "f16", "f32"])
@pytest.mark.parametrize("slabs,res", [(1, 801), (6, 800), (7, 801), (8, 1025), (13, 900)])
def test_tiled_equals_rows(kind, slabs, res):
    tf = vi.TF.from_numpy(W.tf_ramp(), DEV)
    raw = W.sphere_u8(40, radius=17.0, seed=11)
    raw = raw if kind == "u8" else (raw / 255.0).astype("float16" if kind == "f16" else "float32")
    vol = vi.Volume.from_numpy(raw, DEV)
    for v in (vol, vol.with_minmax(8).with_occupancy(tf)):
        for pos in (None, [1.9, -0.4, 2.1]):
            for dt in (vi.VI_F32, vi.VI_BF16):
                rows, tiled = (vi.build_attenuation(v, tf, W.DIAGONAL_LIGHT, slabs, res, dt, layout=l, position=pos)
                               for l in (1, 0))
                torch.cuda.synchronize()
                assert torch.equal(rows.dense(), tiled.dense()), (kind, slabs, res, pos, dt)


@pytest.mark.parametrize("kind", ["u8 linear", "f32 linear", "f32 quads", "u8 bricks"])
@pytest.mark.parametrize("slabs,res", [(5, 651), (5, 653), (5, 709), (9, 711), (9, 743), (9, 745), (3, 770), (9, 772)])
def test_row_shapes(kind, slabs, res):
    """Row builds about the layer sizes where they change: 430,000 texels without
    bits (8 to 16 waves), 510,000 for bricks, 560,000 (two to four slabs in flight of
    linear volumes under a directional light), 600,000 with bits."""
    tf = vi.TF.from_numpy(W.tf_ramp(), DEV)
    raw = W.sphere_u8(40, radius=17.0, seed=11)
    vol = vi.Volume.from_numpy(raw if kind.startswith("u8") else (raw / 255.0).astype("float32"), DEV)
    vol = vol.to_quads() if kind.endswith("quads") else vol.to_bricks() if kind.endswith("bricks") else vol
    for v in (vol, vol.with_minmax(8).with_occupancy(tf)):
        for pos in (None, [1.9, -0.4, 2.1]):
            for dt in (vi.VI_F32, vi.VI_BF16):
                rows, tiled = (vi.build_attenuation(v, tf, W.DIAGONAL_LIGHT, slabs, res, dt, layout=l, position=pos)
                               for l in (1, 0))
                torch.cuda.synchronize()
                assert torch.equal(rows.dense(), tiled.dense()), (kind, slabs, res, pos, dt)
