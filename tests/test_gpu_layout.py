"""Volume preparation against plain NumPy, bit for bit: bricks, quads, the
empty-space map and the occupancy and super-cell bits, for every voxel type and
layout, at edges about the kernels' own sizes (bricks of 4, runs of 16 bricks,
cells of 4 to 32, one to four waves a cell).  Every value is a copy, a minimum
or maximum, or one float32 product, so nothing may differ."""
import numpy as np
import pytest
import torch

from paper_2008_06134_amd import vi
from paper_2008_06134_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"
DTYPES = {"u8": np.uint8, "u16": np.uint16, "f16": np.float16, "f32": np.float32}


def _raw(name, N):
    rng = np.random.default_rng(N)
    if name in ("u8", "u16"):
        v = rng.integers(0, 256 if name == "u8" else 4200, (N, N, N)).astype(DTYPES[name])
    else:
        v = rng.uniform(-0.1, 1.1, (N, N, N)).astype(DTYPES[name])
        v[N // 2, N // 2, :2] = [np.nan, np.inf]
    v[: N // 3] = 0                     # a region that the table leaves empty
    return v


def _bricks(raw):
    N, P = raw.shape[0], -(-raw.shape[0] // 4) * 4
    p = np.zeros((P, P, P), raw.dtype)
    p[:N, :N, :N] = raw
    b = P // 4
    return p.reshape(b, 4, b, 4, b, 4).transpose(0, 2, 4, 1, 3, 5).reshape(-1)


def _quads(raw):
    N = raw.shape[0]
    i = np.minimum(np.arange(N) + 1, N - 1)
    corners = [raw, raw[:, :, i], raw[:, i], raw[:, i][:, :, i]]
    return np.stack([_bricks(c) for c in corners], -1).reshape(-1)


def _map(raw, scale, cell):
    N = raw.shape[0]
    with np.errstate(over="ignore"):
        v = raw.astype(np.float32) * np.float32(scale)
    v = np.clip(np.where(np.isnan(v), np.float32(0), v), 0, 1)
    nc = -(-N // cell)
    out = np.empty((nc, nc, nc, 2), np.float32)
    for z in range(nc):
        for y in range(nc):
            for x in range(nc):
                s = v[z * cell:(z + 1) * cell + 1, y * cell:(y + 1) * cell + 1, x * cell:(x + 1) * cell + 1]
                out[z, y, x] = s.min(), s.max()
    return out


def _words(bits):
    b = np.zeros(-(-bits.size // 32) * 32, np.uint8)
    b[:bits.size] = bits.reshape(-1)
    return np.packbits(b, bitorder="little").view(np.uint32)


def _occupancy(mm, tab):
    K, nc = tab.shape[0], mm.shape[0]
    nxt = np.full(K, K)
    for e in range(K - 1, -1, -1):
        nxt[e] = e if tab[e, 3] > 0 else (nxt[e + 1] if e + 1 < K else K)
    lo = np.maximum((mm[..., 0] * np.float32(K - 1)).astype(np.int32) - 1, 0)
    hi = np.minimum((mm[..., 1] * np.float32(K - 1)).astype(np.int32) + 2, K - 1)
    cells = nxt[lo] <= hi
    S = -(-nc // 4)
    p = np.zeros((4 * S,) * 3, bool)
    p[:nc, :nc, :nc] = cells
    return np.concatenate([_words(cells), _words(p.reshape(S, 4, S, 4, S, 4).any((1, 3, 5)))])


@pytest.mark.parametrize("name", list(DTYPES))
@pytest.mark.parametrize("N", [2, 5, 16, 33, 67])
def test_preparation_matches_numpy(name, N):
    raw = _raw(name, N)
    lin = vi.Volume.from_numpy(raw, DEV)
    vols = {"linear": lin, "bricks": lin.to_bricks(), "quads": lin.to_quads()}
    torch.cuda.synchronize()
    as_bytes = lambda a: np.ascontiguousarray(a).view(np.uint8)  # noqa: E731  (NaNs compare by their bits)
    assert np.array_equal(as_bytes(vols["bricks"].data.cpu().numpy()), as_bytes(_bricks(raw)))
    assert np.array_equal(as_bytes(vols["quads"].data.cpu().numpy()), as_bytes(_quads(raw)))
    for cell in (4, 8, 16, 32):
        want = _map(raw, lin.scale, cell)
        for K in (2, 64, 100, 1024):
            tab = W.tf_ct(K).astype(np.float32)
            if K == 64:
                tab[:, 3] = 0.0         # nothing opaque: walks to the end of the table
            tf = vi.TF.from_numpy(tab, DEV)
            for layout, vol in vols.items():
                got = vol.with_minmax(cell).with_occupancy(tf)
                torch.cuda.synchronize()
                what = f"{layout}, cells of {cell}, {K} entries"
                assert np.array_equal(got.minmax.cpu().numpy().reshape(want.shape), want), what
                assert np.array_equal(got.occ.cpu().numpy().view(np.uint32), _occupancy(want, tab)), what
