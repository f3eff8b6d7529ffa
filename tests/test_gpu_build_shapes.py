"""The row-layout build in each of its launch shapes (4, 8 or 16 waves by the
size of a layer and the kind of volume, sets of eight slabs) and the tiled
build in both of its, at the sizes where they change and where the last set,
stretch or line is a part of one.  The two layouts' builds share a column's
arithmetic but neither their mapping nor their stores, so their stacks are the
same bits; the row layout's border, leading and trailing layers are exact by
definition.  The half stack (rows only) rounds the transmittance whose optical
depth the bfloat16 stack rounds: against the float stack it is within half a
unit in the last place of a half, 2^-12, plus 2e-5 for the two accumulations."""
import pytest
import torch

from paper_2008_06134_amd import vi
from paper_2008_06134_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _volume(kind):
    raw = W.sphere_u8(40, radius=17.0, seed=11)
    if kind == "u8 quads":
        return vi.Volume.from_numpy(raw, DEV).to_quads()
    if kind == "u16 bricks":
        return vi.Volume.from_numpy((raw.astype("uint16") * 16), DEV).to_bricks()
    if kind == "f32 quads":
        return vi.Volume.from_numpy((raw / 255.0).astype("float32"), DEV).to_quads()
    return vi.Volume.from_numpy((raw / 255.0).astype("float16"), DEV)  # linear


# (slabs, res): a layer holds (res + 4)^2 texels and a little more, against
# 160 000, 500 000 (linear) and 600 000; 512 and 513 change the tiled build's shape
SIZES = [(1, 1), (7, 5), (8, 61), (9, 130), (17, 395), (5, 397), (3, 512), (4, 513), (6, 703), (7, 704), (9, 769), (10, 772)]


@pytest.mark.parametrize("kind", ["u8 quads", "u16 bricks", "f32 quads", "f16 linear"])
@pytest.mark.parametrize("slabs,res", SIZES)
def test_row_and_tiled_builds_agree(kind, slabs, res):
    tf = vi.TF.from_numpy(W.tf_ramp(), DEV)
    vol = _volume(kind)
    for v in (vol, vol.with_minmax(8).with_occupancy(tf)):
        for pos in (None, [1.9, -0.4, 2.1]):
            for darken in (0.0, 1.5):
                stacks = {}
                for dt in (vi.VI_F32, vi.VI_BF16, vi.VI_F16):
                    # a buffer of other values: what the build leaves out shows
                    buf = vi.stack_buffer(slabs, res, dt, DEV, 1)
                    buf.fill_(7.0)
                    rows = vi.build_attenuation(v, tf, W.DIAGONAL_LIGHT, slabs, res, dt, buf, layout=1, darken=darken,
                                                position=pos)
                    torch.cuda.synchronize()
                    what = f"{kind}, {slabs} slabs of {res}^2, dtype {dt}, light at {pos}, darken {darken}"
                    p = rows.padded().float()
                    lit = 0.0 if dt == vi.VI_BF16 else 1.0
                    assert bool((p[0] == lit).all()), what
                    assert torch.equal(p[-1], p[-2]), what
                    for edge in (p[:, :2], p[:, -2:], p[:, :, :2], p[:, :, -2:]):
                        assert bool((edge == lit).all()), what
                    stacks[dt] = rows.dense().float()
                    if dt != vi.VI_F16:
                        tiled = vi.build_attenuation(v, tf, W.DIAGONAL_LIGHT, slabs, res, dt, layout=0, darken=darken,
                                                     position=pos)
                        torch.cuda.synchronize()
                        assert torch.equal(rows.dense(), tiled.dense()), what
                off = float((stacks[vi.VI_F16] - stacks[vi.VI_F32]).abs().max())
                assert off <= 2.0 ** -12 + 2e-5, (what, off)


@pytest.mark.parametrize("slabs,res", [(9, 651), (9, 653), (3, 395), (5, 300)])
def test_builds_without_bits_agree(slabs, res):
    """The row shapes of a quad volume without bits change at 430 000 texels a
    layer; the tiled build on rows that 256 does not divide."""
    tf = vi.TF.from_numpy(W.tf_ramp(), DEV)
    vol = _volume("u8 quads")
    for dt in (vi.VI_F32, vi.VI_BF16):
        rows = vi.build_attenuation(vol, tf, W.DIAGONAL_LIGHT, slabs, res, dt, layout=1)
        tiled = vi.build_attenuation(vol, tf, W.DIAGONAL_LIGHT, slabs, res, dt, layout=0)
        torch.cuda.synchronize()
        assert torch.equal(rows.dense(), tiled.dense()), (slabs, res, dt)
