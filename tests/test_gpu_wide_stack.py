"""Descriptors that a program makes itself, with layers beyond what the build
makes (up to 8192^2 texels): the row layout's layer offsets do not fit a 24-bit
product there.  The tiled layout, which addresses each layer by its own 32-bit
product, holds the same texels and gives the same image, bit for bit."""
import pytest
import torch

from paper_2008_06134_amd import vi
from paper_2008_06134_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _texels(n, res, dtype):
    """n x res x res values that differ between neighbours, rows and layers."""
    i = torch.arange(res, device=DEV, dtype=torch.int32)
    v = torch.empty(n, res, res, device=DEV, dtype=dtype)
    for k in range(n):
        v[k] = ((i[:, None] * 37 + i[None, :] * 11 + k * 101) % 127).float() / 127.0
    return v


def _stacks(n, res, dtype, position):
    t = _texels(n, res, torch.float32 if dtype == vi.VI_F32 else torch.bfloat16)
    out = []
    for layout in (0, 1):
        buf = vi.stack_buffer(n, res, dtype, DEV, layout)
        if layout:
            buf.fill_(1.0 if dtype == vi.VI_F32 else 0.0)
            buf[1:n + 1, 2:res + 2, 2:res + 2] = t
            buf[n + 1] = buf[n]
        else:
            r8, r4 = buf.shape[2] * 8, buf.shape[1] * 4
            p = torch.zeros(n, r4, r8, device=DEV, dtype=t.dtype)
            p[:, :res, :res] = t
            buf.copy_(p.reshape(n, r4 // 4, 4, r8 // 8, 8).permute(0, 1, 3, 2, 4))
            del p
        st = vi.light_frame(W.DIAGONAL_LIGHT, n, 8, dtype, layout, position=position)
        st.s.res, st.s.data, st.s.vol_n = res, buf.data_ptr(), 24
        st.data = buf
        out.append(st)
    return out


# 11,600^2: a layer of 2^23 x 16 elements and more; (2, 13,000): products past 2^24 x 16
@pytest.mark.parametrize("n,res,dtype", [(1, 11600, vi.VI_F32), (2, 11600, vi.VI_BF16), (2, 13000, vi.VI_F32),
                                         (3, 17000, vi.VI_BF16), (2, 8200, vi.VI_F32)])
@pytest.mark.parametrize("position", [None, [1.9, -0.4, 2.1]])
def test_wide_layers(n, res, dtype, position):
    tf = vi.TF.from_numpy(W.tf_ramp(), DEV)
    vol = vi.Volume.from_numpy(W.sphere_u8(24, radius=11.0, seed=3), DEV).to_quads()
    tiled, rows = _stacks(n, res, dtype, position)
    cam = W.camera_orbit(61, 47, 0.7, 0.4)
    for mode, opts in [("shadow", {}), ("shell", {}), ("cone", {}), ("cone", {"cone_grid": 2}),
                       ("cone", {"nearest_layer": 1}), ("cone", {"cone_grid": 3, "cone_tan": 1e-4})]:
        a, b = (vi.render(vol, tf, s, cam, mode, 0.5, opts) for s in (tiled, rows))
        torch.cuda.synchronize()
        assert float(a.max()) > 0.0
        assert torch.equal(a, b), (n, res, dtype, mode, opts)
