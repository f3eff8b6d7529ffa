// vi_layout.hip -- one-off preparation of a volume: layout conversion from
// linear raw[z][y][x] to 4x4x4 bricks (one 64-element brick = one 128-byte
// line at 16 bits) or the quad layout (brick order, every slot holding its
// voxel's 2x2 x/y neighbourhood), the empty-space map, and its occupancy and
// super-cell bits.  The conversions are bit-exact copies: results computed
// from the bricked volume equal those from the linear one.  All of them are
// bound by memory; what they had spent instead was index arithmetic (three
// divisions a slot) and one lane a cell.
#include "vi_device.h"
#include "vi_internal.h"

namespace vi {

// --------------------------------------------------------------------------
// bricks and quads: a workgroup converts 16 bricks along x, a thread one row
// (y, z) of a brick, so that a wave's stores are contiguous and the workgroup
// reads whole lines of its 16 source rows.
// --------------------------------------------------------------------------
// Elements x0 .. x0+CNT-1 of a source row, clamped to its last.
template <typename T, int CNT>
__device__ __forceinline__ void load_row(const T* __restrict__ row, int x0, int N, T (&out)[CNT])
{
    if (x0 + CNT <= N) {
        __builtin_memcpy(out, row + x0, sizeof out);
    } else {
#pragma unroll
        for (int i = 0; i < CNT; ++i) out[i] = row[min(x0 + i, N - 1)];
    }
}

template <typename T>
__global__ __launch_bounds__(256) void to_bricks_kernel(const T* __restrict__ src, T* __restrict__ dst, int N,
                                                        uint32_t nb)
{
    const uint32_t r = threadIdx.x & 15u, bx = blockIdx.x * 16u + (threadIdx.x >> 4);
    if (bx >= nb) return;
    const int x0 = (int)bx * 4, y = (int)(blockIdx.y * 4u + (r & 3u)), z = (int)(blockIdx.z * 4u + (r >> 2));
    T out[4] = {T(0), T(0), T(0), T(0)};
    if (y < N && z < N) {
        load_row<T, 4>(src + ((size_t)z * N + y) * N, x0, N, out);
#pragma unroll
        for (int i = 1; i < 4; ++i)
            if (x0 + i >= N) out[i] = T(0);  // padding
    }
    const uint64_t brick = ((uint64_t)blockIdx.z * nb + blockIdx.y) * nb + bx;
    // (a brick buffer is only aligned as its elements are)
    __builtin_memcpy(dst + brick * 64u + r * 4u, out, sizeof out);
}

template <typename T>
static hipError_t launch_t(const void* src, void* dst, int N, hipStream_t s)
{
    const uint32_t nb = ((uint32_t)N + 3u) / 4u;
    hipLaunchKernelGGL((to_bricks_kernel<T>), dim3((nb + 15u) / 16u, nb, nb), dim3(256), 0, s, (const T*)src, (T*)dst,
                       N, nb);
    return hipGetLastError();
}

hipError_t launch_to_bricks(const void* src, void* dst, int dtype, int N, hipStream_t s)
{
    switch (dtype) {
    case VI_U8: return launch_t<uint8_t>(src, dst, N, s);
    case VI_U16:
    case VI_F16: return launch_t<uint16_t>(src, dst, N, s);
    default: return launch_t<uint32_t>(src, dst, N, s);
    }
}

// Quad layout: a slot holds its voxel's 2x2 neighbourhood in x and y, indices
// clamped to N-1.  A workgroup makes 16 bricks along x from the 5 x 4 source
// rows they touch, read once as whole lines into LDS (slots made from global
// memory cost the L1 16 look-ups a load, and ran at half the write rate).  A
// thread stores 16 bytes of slots that lie side by side (4, 2 or 1 for 1-, 2-
// and 4-byte voxels), so a wave stores one contiguous kilobyte.  Padding slots
// hold zeros (never read).  512^3 u16: 541 us with a slot a thread from global
// memory, 253 now (1.34 GB, 5.3 TB/s).
template <typename T, typename T4>
__global__ __launch_bounds__(256) void to_quads_kernel(const T* __restrict__ src, T4* __restrict__ dst, int N,
                                                       uint32_t nb)
{
    constexpr int W = 68;  // 64 voxels of a row and the next one, in fours
    constexpr uint32_t SP = 16 / sizeof(T4);
    __shared__ T rows[20 * W];
    const int x0 = (int)blockIdx.x * 64, y0 = (int)blockIdx.y * 4, z0 = (int)blockIdx.z * 4;
    for (int i = threadIdx.x; i < 20 * (W / 4); i += 256) {
        // row = 5 * z + y, the fifth of each z the first of the next brick's
        const int row = i / (W / 4), x = 4 * (i % (W / 4)), y = min(y0 + row % 5, N - 1), z = min(z0 + row / 5, N - 1);
        T v[4];
        load_row<T, 4>(src + ((size_t)z * N + y) * N, x0 + x, N, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) rows[row * W + x + k] = v[k];
    }
    __syncthreads();
    const uint64_t brick0 = ((uint64_t)blockIdx.z * nb + blockIdx.y) * nb + blockIdx.x * 16u;
    const uint32_t bricks = min(nb - blockIdx.x * 16u, 16u);
#pragma unroll
    for (uint32_t i = 0; i < 4u / SP; ++i) {
        const uint32_t s = (i * 256u + threadIdx.x) * SP;  // first slot
        if (s >= bricks * 64u) break;
        const int x = (int)(s >> 6) * 4 + (int)(s & 3u), y = (int)((s >> 2) & 3u), z = (int)((s >> 4) & 3u);
        union Out {
            T4 q[SP];
            uint4 w;
            __device__ Out() {}
        } o;
        o.w = make_uint4(0u, 0u, 0u, 0u);
        const T* a = rows + (5 * z + y) * W + x;
        if (y0 + y < N && z0 + z < N)
#pragma unroll
            for (int k = 0; k < (int)SP; ++k)
                if (x0 + x + k < N) o.q[k].x = a[k], o.q[k].y = a[k + 1], o.q[k].z = a[W + k], o.q[k].w = a[W + k + 1];
        // (a quad buffer is only aligned as its slots are)
        __builtin_memcpy(dst + brick0 * 64u + s, &o, sizeof o);
    }
}

template <typename T, typename T4>
static hipError_t launch_q(const void* src, void* dst, int N, hipStream_t s)
{
    const uint32_t nb = ((uint32_t)N + 3u) / 4u;
    hipLaunchKernelGGL((to_quads_kernel<T, T4>), dim3((nb + 15u) / 16u, nb, nb), dim3(256), 0, s, (const T*)src,
                       (T4*)dst, N, nb);
    return hipGetLastError();
}

hipError_t launch_to_quads(const void* src, void* dst, int dtype, int N, hipStream_t s)
{
    switch (dtype) {
    case VI_U8: return launch_q<uint8_t, uchar4>(src, dst, N, s);
    case VI_U16:
    case VI_F16: return launch_q<uint16_t, ushort4>(src, dst, N, s);
    default: return launch_q<uint32_t, uint4>(src, dst, N, s);
    }
}

// --------------------------------------------------------------------------
// Empty-space map: the least and greatest normalised value over a cell's
// voxels and the next one along each axis (clamped).  A workgroup of four waves
// takes 4 / WAVES cells: WAVES = 4 share a cell of 16^3 voxels and more (few
// cells, long walks; see the launch for the quads), smaller cells have a wave
// each.  A launch dimension holds less than 2^32 work items, which the cells of
// 4^3 voxels of a volume near 4 GiB pass (1625^3: 407^3 waves), so the
// workgroups are spread over two.  A lane keeps the range
// of what it reads; the cells are taken last to first, since a volume that has
// just been laid out still has its end in the last-level cache.  512^3 u16
// quads, 16^3 cells: 868 us with a lane a cell, 259 now (1.07 GB, 4.1 TB/s).
// --------------------------------------------------------------------------
// Range of raw values.  Normalising, clamp(x * scale), does not decrease with
// x, so the 8- and 16-bit types keep the raw range and normalise its ends;
// floats normalise every value (a NaN counts as 0, as in the passes).
template <typename VT> struct Range {
    uint32_t lo = 0xffffffffu, hi = 0;
    __device__ __forceinline__ void add(VT v, float)
    {
        lo = min(lo, (uint32_t)v);
        hi = max(hi, (uint32_t)v);
    }
    __device__ __forceinline__ float2 ends(float scale) const
    {
        return make_float2(clampf01((float)lo * scale), clampf01((float)hi * scale));
    }
};
struct FloatRange {
    float lo = 1.0f, hi = 0.0f;
    __device__ __forceinline__ void add_value(float v)
    {
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
    }
    __device__ __forceinline__ float2 ends(float) const { return make_float2(lo, hi); }
};
template <> struct Range<__half> : FloatRange {
    __device__ __forceinline__ void add(__half v, float scale) { add_value(norm1(v, scale)); }
};
template <> struct Range<float> : FloatRange {
    __device__ __forceinline__ void add(float v, float scale) { add_value(norm1(v, scale)); }
};

// The voxels of a face of a cell, rows of `nu` by `nv`, from the `first` every
// `step`-th: voxel (u, v) -> element offset.
template <typename VT, typename AT>
__device__ __forceinline__ void add_face(Range<VT>& r, const VT* __restrict__ vol, float scale, int nu, int nv,
                                         int first, int step, AT at)
{
    const float inv = 1.0f / (float)nu;
    for (int i = first; i < nu * nv; i += step) {
        // i / nu exactly: i < 2^11, and the quotient is half a step from an integer
        const int v = (int)(((float)i + 0.5f) * inv), u = i - v * nu;
        r.add(ld32<VT>(vol, at(u, v)), scale);
    }
}

template <typename VT, int LAYOUT, int WAVES>
__global__ __launch_bounds__(256) void minmax_kernel(const VT* __restrict__ vol, VolIndex I, int N, float scale,
                                                     int shift, uint32_t nc, float2* __restrict__ out)
{
    const uint32_t cells = nc * nc * nc, block = blockIdx.y * gridDim.x + blockIdx.x;
    const uint32_t from_end = block * (4u / WAVES) + (threadIdx.x >> 6) / WAVES;
    if (from_end >= cells) return;  // whole waves (WAVES = 1), whole workgroups (WAVES = 4)
    const uint32_t c = cells - 1u - from_end;
    const int lane = threadIdx.x & 63, wave = (int)(threadIdx.x >> 6) % WAVES;
    const int first = wave * 64 + lane, step = WAVES * 64;
    const int cx = (int)(c % nc), cy = (int)((c / nc) % nc), cz = (int)(c / (nc * nc));
    const int B = 1 << shift;
    const int x0 = cx * B, y0 = cy * B, z0 = cz * B;
    // the cell's own voxels, and whether there is a next one along each axis
    // (beyond the last voxel the next is the last itself, already in)
    const int nx = min(B, N - x0), ny = min(B, N - y0), nz = min(B, N - z0);
    const bool mx = x0 + B < N, my = y0 + B < N, mz = z0 + B < N;
    Range<VT> r;
    // four elements loaded as one unit (a quad slot, or four voxels along x)
    using Q = typename QuadRaw<VT>::T;
    union Four {
        Q q;
        VT v[4];
        __device__ Four() {}
    };
    if constexpr (LAYOUT == VI_LAYOUT_QUAD4) {
        // a slot holds the next voxels along x and y as well: whole bricks,
        // one slot a lane, then the first plane of the bricks above
        const int lx = lane & 3, ly = (lane >> 2) & 3, lz = lane >> 4;
        const int bx1 = (nx + 3) / 4, by1 = (ny + 3) / 4, bz1 = (nz + 3) / 4 + (mz ? 1 : 0);
        const auto add_slot = [&](int bx, int by, int bz, bool in) {
            if (!in) return;
            const size_t at = (size_t)vol_oz<LAYOUT>(I, z0 + 4 * bz + lz) + vol_oy<LAYOUT>(I, y0 + 4 * by + ly) +
                              vol_ox<LAYOUT>(I, x0 + 4 * bx + lx);
            Four s;
            s.q = ((const Q*)vol)[at];
#pragma unroll
            for (int i = 0; i < 4; ++i) r.add(s.v[i], scale);
        };
        for (int bz = wave; bz < bz1; bz += WAVES) {
            const bool inz = 4 * bz + lz < nz + (mz ? 1 : 0);
            for (int by = 0; by < by1; ++by) {
                const bool iny = inz && 4 * by + ly < ny;
#pragma unroll 4
                for (int bx = 0; bx < bx1; ++bx) add_slot(bx, by, bz, iny && 4 * bx + lx < nx);
            }
        }
    } else {
        // own voxels, four along x a lane, then the three faces beyond them
        const int rows = ny * nz, quads = (nx + 3) / 4;
        const float inv_q = 1.0f / (float)quads, inv_y = 1.0f / (float)ny;
#pragma unroll 4
        for (int i = first; i < rows * quads; i += step) {
            // (i < 2^13; exact as in add_face)
            const int row = (int)(((float)i + 0.5f) * inv_q), qx = 4 * (i - row * quads);
            const int z = (int)(((float)row + 0.5f) * inv_y), y = row - z * ny;
            const uint32_t at = vol_oz<LAYOUT>(I, z0 + z) + vol_oy<LAYOUT>(I, y0 + y) + vol_ox<LAYOUT>(I, x0 + qx);
            Four f;
            if (qx + 4 <= nx) {
                Q q;
                __builtin_memcpy(&q, (const char*)vol + (size_t)at * sizeof(VT), sizeof q);
                f.q = q;
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) f.v[k] = ld32<VT>(vol, at + (uint32_t)min(k, nx - 1 - qx));
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) r.add(f.v[k], scale);
        }
        const int ex = nx + (mx ? 1 : 0), ey = ny + (my ? 1 : 0);
        if (mx)
            add_face<VT>(r, vol, scale, ny, nz, first, step, [&](int u, int v) {
                return vol_oz<LAYOUT>(I, z0 + v) + vol_oy<LAYOUT>(I, y0 + u) + vol_ox<LAYOUT>(I, x0 + B);
            });
        if (my)
            add_face<VT>(r, vol, scale, ex, nz, first, step, [&](int u, int v) {
                return vol_oz<LAYOUT>(I, z0 + v) + vol_oy<LAYOUT>(I, y0 + B) + vol_ox<LAYOUT>(I, x0 + u);
            });
        if (mz)
            add_face<VT>(r, vol, scale, ex, ey, first, step, [&](int u, int v) {
                return vol_oz<LAYOUT>(I, z0 + B) + vol_oy<LAYOUT>(I, y0 + v) + vol_ox<LAYOUT>(I, x0 + u);
            });
    }
    for (int off = 32; off > 0; off >>= 1) {
        const auto lo = __shfl_xor(r.lo, off), hi = __shfl_xor(r.hi, off);
        r.lo = lo < r.lo ? lo : r.lo;
        r.hi = hi > r.hi ? hi : r.hi;
    }
    if constexpr (WAVES > 1) {
        __shared__ decltype(r.lo) lo[WAVES], hi[WAVES];
        if (lane == 0) lo[wave] = r.lo, hi[wave] = r.hi;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            r.lo = lo[w] < r.lo ? lo[w] : r.lo;
            r.hi = hi[w] > r.hi ? hi[w] : r.hi;
        }
    }
    if (lane == 0 && wave == 0) out[c] = r.ends(scale);
}

constexpr uint32_t kMapBlocksX = 1u << 23;  // of 256 lanes: 2^31 work items
template <typename VT, int LAYOUT>
static hipError_t launch_mm_l(const void* vol, VolIndex I, int N, float scale, int shift, float* out, hipStream_t s)
{
    const uint32_t nc = ((uint32_t)N + (1u << shift) - 1) >> shift, cells = nc * nc * nc;
    // (a wave a cell, 4096 cells fill the chip's SIMDs four deep; beyond that
    // the quads' one wave a cell is the faster, 265 us against 312 at 512^3,
    // the other layouts' longer walks are not, 1081 against 633 at 1024^3)
    const bool shared = shift >= 4 && (LAYOUT != VI_LAYOUT_QUAD4 || cells <= 4096u);
    const uint32_t blocks = shared ? cells : (cells + 3u) / 4u, rows = (blocks + kMapBlocksX - 1) / kMapBlocksX;
    const dim3 grid((blocks + rows - 1) / rows, rows);
    if (shared)
        hipLaunchKernelGGL((minmax_kernel<VT, LAYOUT, 4>), grid, dim3(256), 0, s, (const VT*)vol, I, N, scale, shift,
                           nc, (float2*)out);
    else
        hipLaunchKernelGGL((minmax_kernel<VT, LAYOUT, 1>), grid, dim3(256), 0, s, (const VT*)vol, I, N, scale, shift,
                           nc, (float2*)out);
    return hipGetLastError();
}

template <typename VT>
static hipError_t launch_mm(const void* vol, int layout, VolIndex I, int N, float scale, int shift, float* out,
                            hipStream_t s)
{
    if (layout == VI_LAYOUT_QUAD4) return launch_mm_l<VT, VI_LAYOUT_QUAD4>(vol, I, N, scale, shift, out, s);
    return layout == VI_LAYOUT_BRICK4 ? launch_mm_l<VT, VI_LAYOUT_BRICK4>(vol, I, N, scale, shift, out, s)
                                      : launch_mm_l<VT, VI_LAYOUT_LINEAR>(vol, I, N, scale, shift, out, s);
}

hipError_t launch_minmax(const void* vol, int dtype, int layout, uint32_t vsy, uint32_t vsz, int N, float scale,
                         int shift, float* out, hipStream_t s)
{
    const VolIndex I = {1u, vsy, vsz};
    switch (dtype) {
    case VI_U8: return launch_mm<uint8_t>(vol, layout, I, N, scale, shift, out, s);
    case VI_U16: return launch_mm<uint16_t>(vol, layout, I, N, scale, shift, out, s);
    case VI_F16: return launch_mm<__half>(vol, layout, I, N, scale, shift, out, s);
    default: return launch_mm<float>(vol, layout, I, N, scale, shift, out, s);
    }
}

// --------------------------------------------------------------------------
// Occupancy bits for one transfer function: cell c may hold opacity (the
// negation of the map's emptiness test against the table's next-opaque
// indices, built in LDS per workgroup).  One lane a cell, each half of a
// wave's ballot one word.  Super-cell (X, Y, Z) covers cells 4X .. 4X+3 (and
// so on, clipped at nc) and is set when any of them is: one wave a super-cell
// with a cell a lane, 32 super-cells (one word) a workgroup.  Both in one
// launch: the first `cell_blocks` workgroups write cell words.
// --------------------------------------------------------------------------
constexpr uint32_t kOccThreads = 1024;
__global__ __launch_bounds__(1024) void occupancy_kernel(const float2* __restrict__ mm, uint32_t nc,
                                                         const float* __restrict__ tf, int K, uint32_t cell_blocks,
                                                         uint32_t* __restrict__ bits)
{
    extern __shared__ int s_next[];
    __shared__ uint32_t s_word;
    if (threadIdx.x == 0) s_word = 0u;
    build_next_opaque(s_next, tf, K);
    __syncthreads();
    const uint32_t cells = nc * nc * nc, words = (cells + 31u) / 32u;
    const float Km1 = (float)(K - 1);
    const uint32_t lane = threadIdx.x & 63u;
    if (blockIdx.x < cell_blocks) {
        const uint32_t c = blockIdx.x * kOccThreads + threadIdx.x;
        const uint64_t m = __ballot(c < cells && !cell_empty(mm[min(c, cells - 1u)], s_next, Km1, K));
        if ((lane & 31u) == 0u && c < cells) bits[c >> 5] = (uint32_t)(lane ? (m >> 32) : m);
        return;
    }
    const uint32_t snc = (nc + 3u) / 4u, scells = snc * snc * snc, w = blockIdx.x - cell_blocks;
    for (uint32_t k = threadIdx.x >> 6; k < 32u; k += kOccThreads / 64u) {
        const uint32_t sc = w * 32u + k;
        if (sc >= scells) break;
        const uint32_t x = sc % snc * 4u + (lane & 3u), y = sc / snc % snc * 4u + ((lane >> 2) & 3u),
                       z = sc / (snc * snc) * 4u + (lane >> 4);
        const bool in = x < nc && y < nc && z < nc;
        const bool any = __any(in && !cell_empty(mm[in ? (z * nc + y) * nc + x : 0u], s_next, Km1, K));
        if (lane == 0u && any) atomicOr(&s_word, 1u << k);
    }
    __syncthreads();
    if (threadIdx.x == 0) bits[words + w] = s_word;
}

hipError_t launch_occupancy(const float* minmax, uint32_t nc, const float* tf, int K, uint32_t* bits,
                            hipStream_t s)
{
    const uint32_t cells = nc * nc * nc, cell_blocks = (cells + kOccThreads - 1u) / kOccThreads;
    const uint32_t snc = (nc + 3u) / 4u, swords = (snc * snc * snc + 31u) / 32u;
    hipLaunchKernelGGL(occupancy_kernel, dim3(cell_blocks + swords), dim3(kOccThreads), sizeof(int) * (size_t)K, s,
                       (const float2*)minmax, nc, tf, K, cell_blocks, bits);
    return hipGetLastError();
}

}  // namespace vi
