// vi_render.hip -- eye-space ray march with the slice-based illumination
// coefficient (sections 3.2.2, 3.2.3 and 4).
//
// The four lanes of a quad march one ray together (each takes every fourth
// segment; the four segments of a step are composited by a scan over the quad).  Per ray, once
// (float): the camera ray, the slab test against the unit cube, the entry
// point in volume and light-grid coordinates and the increments of both per
// voxel of path; for the cone, the per-ray frame (B, L x B) in texel units.
// Per segment: position = entry + s * direction in offset coordinates (so
// the fraction of every interpolation is taken on small magnitudes),
// trilinear fetch, transfer function from LDS, extinction-corrected opacity,
// and -- only when the opacity is non-zero -- the coefficient gather from the
// stack, then the front-to-back update (Eq. 3) with the coefficient weighting
// the emission (Eq. 7).  A ray stops when it exits the cube or its remaining
// transmittance drops to term_eps.
//
// A wave covers 4 x 4 pixels (16 rays x 4 lanes), a workgroup 8 x 8 pixels,
// so the rays of a wave sample neighbouring voxels and texels.
#include <type_traits>

#include "vi_device.h"
#include "vi_internal.h"

namespace vi {

// --------------------------------------------------------------------------
// stack access
// --------------------------------------------------------------------------
// A float stack holds transmittance T; a bfloat16 stack holds optical depth
// in base-2 units, tau2 = -log2 T (Eq. 6's exponent summed over the slabs in
// front, over ln 2), so that each texel converts to T = 2^-tau2 with one
// exponential before the interpolation; a half-precision stack holds T
// (from the float optical depth), converted with no exponential, and has the row
// layout only.
template <int SDT>
__device__ __forceinline__ float stack_texel(const void* __restrict__ S, uint32_t idx);

template <>
__device__ __forceinline__ float stack_texel<VI_F32>(const void* __restrict__ S, uint32_t idx)
{
    return ((const float*)S)[idx];
}
template <>
__device__ __forceinline__ float stack_texel<VI_BF16>(const void* __restrict__ S, uint32_t idx)
{
    return fast_exp2(-bf16_to_f32(((const uint16_t*)S)[idx]));
}
// Row layout: the two texels (i, i+1) of one bilinear row, element e and
// e+1, with one load: 8 bytes (4-byte aligned) for float, 4 bytes (2-byte
// aligned, which global loads allow) for bfloat16.
typedef float f32x2_a4 __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32_a2 __attribute__((aligned(2)));

// The load and the conversion are separate steps (PairRaw holds the loaded
// bits), so that a gather can issue the loads of several taps before it
// converts any of them.
template <int SDT> struct PairRaw;
template <> struct PairRaw<VI_F32> { f32x2_a4 v; };
template <> struct PairRaw<VI_BF16> { uint32_t w; };
template <> struct PairRaw<VI_F16> { uint32_t w; };

template <int SDT>
__device__ __forceinline__ PairRaw<SDT> pair_load(const void* __restrict__ S, uint32_t e);
// (Byte offsets are formed in 32 bits -- a stack is below 4 GiB -- so that
// each load takes the stack's base from scalar registers and a 32-bit
// offset, with no 64-bit address arithmetic per load.)
template <>
__device__ __forceinline__ PairRaw<VI_F32> pair_load<VI_F32>(const void* __restrict__ S, uint32_t e)
{
    return PairRaw<VI_F32>{*(const f32x2_a4*)((const char*)S + (e << 2))};
}
template <>
__device__ __forceinline__ PairRaw<VI_BF16> pair_load<VI_BF16>(const void* __restrict__ S, uint32_t e)
{
    return PairRaw<VI_BF16>{*(const u32_a2*)((const char*)S + (e << 1))};
}
template <>
__device__ __forceinline__ PairRaw<VI_F16> pair_load<VI_F16>(const void* __restrict__ S, uint32_t e)
{
    return PairRaw<VI_F16>{*(const u32_a2*)((const char*)S + (e << 1))};
}
__device__ __forceinline__ float2 pair_value(const PairRaw<VI_F32>& r) { return make_float2(r.v.x, r.v.y); }
__device__ __forceinline__ float2 pair_value(const PairRaw<VI_F16>& r)
{
    return make_float2(__half2float(__ushort_as_half((unsigned short)(r.w & 0xffffu))),
                       __half2float(__ushort_as_half((unsigned short)(r.w >> 16))));
}
__device__ __forceinline__ float2 pair_value(const PairRaw<VI_BF16>& r)
{
    // element e in the low half, e + 1 in the high half (little-endian)
    return make_float2(fast_exp2(-__uint_as_float(r.w << 16)), fast_exp2(-__uint_as_float(r.w & 0xffff0000u)));
}

// A lookup in three parts, so that the taps of a gather that lie at one depth
// share the first and a gather can issue the loads of several taps before it
// needs any of them: the depth part (layers and weight), the loads of the
// bilinear footprint in both layers, and the two layers' values.
//
// Row layout: every footprint is a plain read.  Layer -1 (face 0) transmits
// fully, so a depth index in front of the first face needs no test; layer n
// repeats layer n-1, so the second layer needs no clamp; and the two-texel
// border lets a footprint that reaches past the grid clamp onto border texels
// only (a column a < -2 reads the pair (-2, -1), a > res the pair (res,
// res+1): both 1).  Clamping the coordinates (not the texel indices) keeps
// every footprint on stored texels: beyond the grid both texels of a row are
// border texels (1), so the value is the same 1 whatever the weight.  One
// offset serves all four loads, whose next row and next layer come from the
// shifted bases.
template <int SL> struct ZPart;
template <> struct ZPart<VI_STACK_ROWS> {
    uint32_t e;  // element of the layer's row 0, column 0 (light-grid offsets)
    float w;
};
template <> struct ZPart<VI_STACK_TILED> {
    uint32_t b0, b1;  // elements of the two layers
    float w;
    bool front;  // before the first layer: the nearer face is face 0
};
template <int SDT, int SL> struct Tap;
template <int SDT> struct Tap<SDT, VI_STACK_ROWS> {
    PairRaw<SDT> a0, a1, b0, b1;  // nearer layer rows j, j+1; farther layer rows j, j+1
    float wx, wy;
};
template <int SDT> struct Tap<SDT, VI_STACK_TILED> {
    float t0, t1;  // the layers' values
};

// A frame's kernel: kStaged where its waves read the stack through windows in
// LDS, kWide where a layer's offset does not fit a 24-bit product (see rl16).
// Kernels of their own: the staging march keeps a wave's lanes together and takes
// 12 to 20 KB of LDS a workgroup, which frames without it would pay for nothing,
// and a branch to a 32-bit product cost small frames of every mode 2 to 4 %.
enum class Form { kPlain, kStaged, kWide };

// nearest-face lookups: never, always (copies of a gather behind one branch
// that is uniform per frame), or, for wide layers, asked of the frame, with the
// layer's offset in 32 bits
enum class Near { kNo, kYes, kWide };
template <Near V> using NearC = std::integral_constant<Near, V>;
template <int SL, Near NEAR>
__device__ __forceinline__ ZPart<SL> z_part(const RenderFrame& F, float z)
{
    if (NEAR == Near::kYes) z = floorf(z + 0.5f);
    if (NEAR == Near::kWide) {
        const float face = floorf(z + 0.5f);
        z = F.nearest ? face : z;
    }
    z = __builtin_amdgcn_fmed3f(z, F.zlo, F.zhi);
    const int iz = floor_int(z);
    ZPart<SL> p;
    p.w = __builtin_amdgcn_fractf(z);
    if constexpr (SL == VI_STACK_ROWS) {
        if (NEAR == Near::kWide) p.e = ((uint32_t)iz * (uint32_t)F.rl16 + (uint32_t)F.rb16) << 4;
        else p.e = (uint32_t)(__mul24(iz, F.rl16) + F.rb16) << 4;
    } else {
        const int k0 = iz + F.Mz;
        p.front = k0 < 0;
        p.b0 = (uint32_t)max(k0, 0) * F.layer;
        p.b1 = (uint32_t)min(k0 + 1, F.n - 1) * F.layer;
    }
    return p;
}

template <int SDT>
__device__ __forceinline__ void tap_load(const RenderFrame& F, const ZPart<VI_STACK_ROWS>& p, float x, float y,
                                         Tap<SDT, VI_STACK_ROWS>& t)
{
    x = __builtin_amdgcn_fmed3f(x, F.xlo, F.xhi);
    y = __builtin_amdgcn_fmed3f(y, F.xlo, F.xhi);
    const int ix = floor_int(x), iy = floor_int(y);
    t.wx = __builtin_amdgcn_fractf(x);
    t.wy = __builtin_amdgcn_fractf(y);
    const uint32_t e = p.e + (uint32_t)(__mul24(iy, (int)F.rpitch) + ix);
    t.a0 = pair_load<SDT>(F.stack, e);
    t.a1 = pair_load<SDT>(F.stack_r1, e);
    t.b0 = pair_load<SDT>(F.stack_l1, e);
    t.b1 = pair_load<SDT>(F.stack_l1r1, e);
}
// the layers' bilinear values, nearer (x) and farther (y)
template <int SDT>
__device__ __forceinline__ float2 tap_layers(const Tap<SDT, VI_STACK_ROWS>& t)
{
    float2 r0 = pair_value(t.a0), r1 = pair_value(t.a1);
    float ab = fmaf(t.wx, r0.y - r0.x, r0.x), cd = fmaf(t.wx, r1.y - r1.x, r1.x);
    const float t0 = fmaf(t.wy, cd - ab, ab);
    r0 = pair_value(t.b0);
    r1 = pair_value(t.b1);
    ab = fmaf(t.wx, r0.y - r0.x, r0.x);
    cd = fmaf(t.wx, r1.y - r1.x, r1.x);
    return make_float2(t0, fmaf(t.wy, cd - ab, ab));
}

// Tiled layout: eight loads with bounds selects, converted at once.  The
// bounds are combined without short circuits and face 0 is selected behind its
// loads: with `&&` and a branch around the nearer layer the compiler moved the
// loads of a row or a layer into the branches of the lanes that need them, up to
// four waits a tap one after the other (256^3 quads, default options: ring cone
// at 320 x 240 368 us, 320 now; shell at 1024^2 1100, 965).
template <int SDT>
__device__ __forceinline__ void tap_load(const RenderFrame& F, const ZPart<VI_STACK_TILED>& p, float x, float y,
                                         Tap<SDT, VI_STACK_TILED>& t)
{
    x = __builtin_amdgcn_fmed3f(x, F.xlo, F.xhi);
    y = __builtin_amdgcn_fmed3f(y, F.xlo, F.xhi);
    const int i0 = floor_int(x) + F.Mr, j0 = floor_int(y) + F.Mr;
    const float wx = __builtin_amdgcn_fractf(x), wy = __builtin_amdgcn_fractf(y);
    const int res = F.res;
    const bool vi0 = (unsigned)i0 < (unsigned)res, vi1 = (unsigned)(i0 + 1) < (unsigned)res;
    const bool vj0 = (unsigned)j0 < (unsigned)res, vj1 = (unsigned)(j0 + 1) < (unsigned)res;
    const uint32_t oi0 = stack_oi(clampi(i0, 0, res - 1)), oi1 = stack_oi(clampi(i0 + 1, 0, res - 1));
    const uint32_t oj0 = stack_oj(clampi(j0, 0, res - 1), F.row_tiles32);
    const uint32_t oj1 = stack_oj(clampi(j0 + 1, 0, res - 1), F.row_tiles32);
    const auto layer = [&](uint32_t base) {
        const uint32_t r0 = base + oj0, r1 = base + oj1;
        float a = stack_texel<SDT>(F.stack, r0 + oi0), b = stack_texel<SDT>(F.stack, r0 + oi1);
        float c = stack_texel<SDT>(F.stack, r1 + oi0), d = stack_texel<SDT>(F.stack, r1 + oi1);
        a = (vi0 & vj0) ? a : 1.0f;
        b = (vi1 & vj0) ? b : 1.0f;
        c = (vi0 & vj1) ? c : 1.0f;
        d = (vi1 & vj1) ? d : 1.0f;
        const float ab = fmaf(wx, b - a, a), cd = fmaf(wx, d - c, c);
        return fmaf(wy, cd - ab, ab);
    };
    const float t0 = layer(p.b0);
    t.t1 = layer(p.b1);
    t.t0 = p.front ? 1.0f : t0;
}
template <int SDT>
__device__ __forceinline__ float2 tap_layers(const Tap<SDT, VI_STACK_TILED>& t)
{
    return make_float2(t.t0, t.t1);
}

// Where a gather reads the stack: device memory, or the window of it that its
// wave has staged in LDS (see stage_window).
template <int SDT, int SL, Near NEAR>
struct FromStack {
    using Z = ZPart<SL>;
    using T = Tap<SDT, SL>;
    static constexpr bool kTiled = SL == VI_STACK_TILED;
    const RenderFrame& F;
    __device__ __forceinline__ Z z_part(float z) const { return vi::z_part<SL, NEAR>(F, z); }
    __device__ __forceinline__ void load(const Z& p, float x, float y, T& t) const { tap_load<SDT>(F, p, x, y, t); }
    __device__ __forceinline__ float2 layers(const T& t) const { return tap_layers<SDT>(t); }
};

// The window holds kWinX x WY texels of WZ layers as floats, transmittance
// whatever the stack's type.  Taps lie inside it (the fit test), so nothing
// is clamped; the weights and values are those a read of the stack gives, bit
// for bit.
template <int WY>
struct FromWindow {
    struct Z {
        int e;
        float w;
    };
    struct T {
        float a0, a1, a2, a3, b0, b1, b2, b3, wx, wy;
    };
    static constexpr bool kTiled = false;
    const float* tile;
    int org;  // element of light-grid cell (0, 0, 0)
    __device__ __forceinline__ Z z_part(float z) const
    {
        return Z{floor_int(z) * (kWinX * WY) + org, __builtin_amdgcn_fractf(z)};
    }
    __device__ __forceinline__ void load(const Z& p, float x, float y, T& t) const
    {
        const int ix = floor_int(x), iy = floor_int(y);
        t.wx = __builtin_amdgcn_fractf(x);
        t.wy = __builtin_amdgcn_fractf(y);
        const float* q = tile + (iy * kWinX + ix + p.e);
        t.a0 = q[0], t.a1 = q[1], t.a2 = q[kWinX], t.a3 = q[kWinX + 1];
        q += kWinX * WY;
        t.b0 = q[0], t.b1 = q[1], t.b2 = q[kWinX], t.b3 = q[kWinX + 1];
    }
    __device__ __forceinline__ float2 layers(const T& t) const
    {
        float ab = fmaf(t.wx, t.a1 - t.a0, t.a0), cd = fmaf(t.wx, t.a3 - t.a2, t.a2);
        const float v0 = fmaf(t.wy, cd - ab, ab);
        ab = fmaf(t.wx, t.b1 - t.b0, t.b0);
        cd = fmaf(t.wx, t.b3 - t.b2, t.b2);
        return make_float2(v0, fmaf(t.wy, cd - ab, ab));
    }
};

// Transmittance at light-grid offset coordinates (z, x, y): depth between
// faces (layer z and z+1 in stack order, layer -1 = 1), bilinear in the
// layer, fully transmitting outside the texel grid.
template <int SDT, int SL, Near NEAR>
__device__ __forceinline__ float stack_lookup(const RenderFrame& F, float z, float x, float y)
{
    const ZPart<SL> p = z_part<SL, NEAR>(F, z);
    Tap<SDT, SL> t;
    tap_load<SDT>(F, p, x, y, t);
    const float2 v = tap_layers<SDT>(t);
    return fmaf(p.w, v.y - v.x, v.x);
}

// --------------------------------------------------------------------------
// one ray
// --------------------------------------------------------------------------
struct ConeFrame {
    float bx, by;  // B in texels per world unit (x, y)
    float px, py;  // L x B in texels per world unit
};

// NB stack lookups at once: all their loads are issued before any of them
// is converted, so a gather waits on one round trip per batch of taps.  Larger
// batches keep more loads in flight per wave but take registers, i.e. resident
// waves; measured on the 512^3 workload: the ring cone and the float-stack shell
// (held to six waves per SIMD) run fastest with two taps per batch, the 5 x 5
// lattice with one (four loads); the bfloat16 shell, whose decoding takes more
// registers, keeps one.
template <int MODE, int SDT>
constexpr int shell_batch()
{
    return MODE == VI_MODE_SHELL && SDT == VI_F32 ? 2 : 1;
}
// The six taps of a shell are unrolled over a row stack, so that one shell's
// offsets stay in scalar registers; over a tiled stack, whose taps are long,
// that costs registers (115 with the branches that tap_load
// names, a wave a SIMD or two; 256^3 at 1024^2 998 us unrolled, 965 in a loop).
template <bool TILED> constexpr int kShellUnroll = TILED ? 1 : 6;

// Nothing is scheduled across the end of a batch: the scheduler would issue
// the next batches' loads ahead of it and take the registers of one or two
// more waves a SIMD (point shell 122 VGPRs against 88).
__device__ __forceinline__ void end_batch() { __builtin_amdgcn_sched_barrier(0); }

template <int NB, typename SRC>
__device__ __forceinline__ void lookup_batch(const SRC& src, const float (&z)[NB], const float (&x)[NB],
                                             const float (&y)[NB], float (&out)[NB])
{
    typename SRC::T t[NB];
    float w[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const typename SRC::Z p = src.z_part(z[u]);
        w[u] = p.w;
        src.load(p, x[u], y[u], t[u]);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const float2 v = src.layers(t[u]);
        out[u] = fmaf(w[u], v.y - v.x, v.x);
    }
    end_batch();
}

// NB taps at one depth added to the two layers' sums.
template <int NB, typename SRC>
__device__ __forceinline__ void add_taps(const SRC& src, const typename SRC::Z& p, const float (&x)[NB],
                                         const float (&y)[NB], float2& s)
{
    typename SRC::T t[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) src.load(p, x[u], y[u], t[u]);
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const float2 v = src.layers(t[u]);
        s.x += v.x;
        s.y += v.y;
    }
    end_batch();
}

template <int MODE, int NB, typename SRC>
__device__ __forceinline__ float gather(const RenderFrame& F, const SRC& src, const ConeFrame& cf, float z, float x,
                                        float y)
{
    if (MODE == VI_MODE_SHADOW) {
        const float zz[1] = {z}, xx[1] = {x}, yy[1] = {y};
        float v[1];
        lookup_batch<1>(src, zz, xx, yy, v);
        return v[0];
    }
    if (MODE == VI_MODE_SHELL) {
        // weighted taps (shell r's six taps share w_r / (6 sum w))
        float zz[NB], xx[NB], yy[NB], v[NB], s = 0.0f;
        for (int t = 0; t < F.ntaps; t += 6) {
#pragma unroll kShellUnroll<SRC::kTiled>
            for (int q = 0; q < 6; q += NB) {
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    zz[u] = z + F.tz[t + q + u];
                    xx[u] = x + F.tx_[t + q + u];
                    yy[u] = y + F.ty_[t + q + u];
                }
                lookup_batch<NB>(src, zz, xx, yy, v);
#pragma unroll
                for (int u = 0; u < NB; ++u) s = fmaf(F.tw[t + q + u], v[u], s);
            }
        }
        return s;
    }
    // Cone: the taps of a ring, and of the whole lattice, lie at one depth, so
    // their bilinear values are summed per layer and the depth weight is
    // applied to the sums.
    if (MODE == VI_MODE_CONE) {
        // rings (Eq. 11)
        float s = 0.0f;
        for (int m = 1; m <= F.cone_rings; ++m) {
            const float r = (float)m * F.ds * F.cone_tan;
            const float bx = r * cf.bx, by = r * cf.by, px = r * cf.px, py = r * cf.py;
            const typename SRC::Z p = src.z_part(z - (float)m);
            float2 t = make_float2(0.0f, 0.0f);
            if (F.cone_angles == 4) {
                // a quarter turn apart: +-B and +-(L x B)
                const float xb[2] = {x + bx, x - bx}, yb[2] = {y + by, y - by};
                const float xp[2] = {x + px, x - px}, yp[2] = {y + py, y - py};
                add_taps<2>(src, p, xb, yb, t);
                add_taps<2>(src, p, xp, yp, t);
            } else {
                for (int q = 0; q < F.cone_angles; ++q) {
                    const float ca = F.cone_cos[q], sa = F.cone_sin[q];
                    const float xq[1] = {x + fmaf(ca, bx, sa * px)}, yq[1] = {y + fmaf(ca, by, sa * py)};
                    add_taps<1>(src, p, xq, yq, t);
                }
            }
            s += fmaf(p.w, t.y - t.x, t.x);
        }
        return s * F.tap_w;
    }
    // lattice form, one slab toward the light (a kernel of its own)
    const int G = F.cone_grid;
    const float rho = F.ds * F.cone_tan * 0.5f, half = 0.5f * (float)(G - 1);
    const float bx = rho * cf.bx, by = rho * cf.by, px = rho * cf.px, py = rho * cf.py;
    const typename SRC::Z p = src.z_part(z - 1.0f);
    float2 t = make_float2(0.0f, 0.0f);
    float a = -half;
    for (int ia = 0; ia < G; ++ia, a += 1.0f) {
        const float xa = fmaf(a, bx, x), ya = fmaf(a, by, y);
        float b = -half;
        for (int ib = 0; ib < G; ++ib, b += 1.0f) {
            const float xq[1] = {fmaf(b, px, xa)}, yq[1] = {fmaf(b, py, ya)};
            add_taps<1>(src, p, xq, yq, t);
        }
    }
    return fmaf(p.w, t.y - t.x, t.x) * F.tap_w;
}

// Point light: the light grid is a frustum with its apex at P.  A lookup at
// depth d = L.(p - P) and lateral offsets (u, v) = (U, V).(p - P) reads texel
// column (u / d) sc + xo; a point at or behind the apex's plane (d <= 0) lies
// outside every texel, where the stack reads 1.  The column is clamped to a
// band just outside the grid, which keeps huge quotients finite.
__device__ __forceinline__ float frustum_col(const RenderFrame& F, float u, float rd, bool ahead)
{
    const float x = ahead ? fmaf(u * rd, F.sc, F.xo) : -3.0e38f;
    return fminf(fmaxf(x, (float)(-3 - F.Mr)), (float)(F.res + 2 - F.Mr));
}

// Cone (Eq. 11) about the light's direction at the sample.  With r = (d, u,
// v) the sample's offset from the light in the light frame (voxels), the
// axis is L_s = r / |r|, and one slab of depth toward the light lies
// S = ds |r| / d along it.  Tap (c, a, b) sits at
//   r - c S L_s + S (a B + b L_s x B) = r (1 - c ds / d) + S (a B + b L_s x B),
// B the view vector w = (wd, wu, wv) with its L_s part removed (U's, when w
// runs along L_s), of unit length; ring m has c = m and (a, b) = m tan phi
// (cos, sin) theta, the lattice c = 1 and (a, b) on a grid of spacing
// tan phi / 2.  The tap's slab index moves with its depth: c slabs, plus
// the depth part of the lateral offset.  Taps are summed in the order rings
// (or lattice rows), then angles (or columns), in batches as in gather().
template <int SDT, int SL, Near NEAR>
__device__ __forceinline__ float gather_point_cone(const RenderFrame& F, float z, float d, float u, float v, float wd,
                                                   float wu, float wv)
{
    const float r2 = fmaf(d, d, fmaf(u, u, v * v)), ir = __builtin_amdgcn_rsqf(r2);
    const float ld = d * ir, lu = u * ir, lv = v * ir;
    const float wl = fmaf(wd, ld, fmaf(wu, lu, wv * lv));
    float bd = fmaf(-wl, ld, wd), bu = fmaf(-wl, lu, wu), bv = fmaf(-wl, lv, wv);
    float nb = fmaf(bd, bd, fmaf(bu, bu, bv * bv));
    if (nb < 1e-12f) {
        // U is (0, 1, 0) in the light frame
        bd = -lu * ld;
        bu = fmaf(-lu, lu, 1.0f);
        bv = -lu * lv;
        nb = fmaf(bd, bd, fmaf(bu, bu, bv * bv));
    }
    const float q = F.ds * __builtin_amdgcn_rcpf(d);                  // ds / d
    const float sb = (q * r2 * ir) * __builtin_amdgcn_rsqf(nb);       // S / |B|
    bd *= sb;
    bu *= sb;
    bv *= sb;
    const float cd = fmaf(lu, bv, -lv * bu), cu = fmaf(lv, bd, -ld * bv), cv = fmaf(ld, bu, -lu * bd);
    const auto tap = [&](float c, float a, float b, float& zz, float& xx, float& yy) {
        const float k = fmaf(-c, q, 1.0f);
        const float od = fmaf(a, bd, b * cd);
        const float dd = fmaf(d, k, od);
        const float rd = __builtin_amdgcn_rcpf(dd);
        zz = fmaf(od, F.ids, z - c);
        xx = frustum_col(F, fmaf(u, k, fmaf(a, bu, b * cu)), rd, dd > 0.0f);
        yy = frustum_col(F, fmaf(v, k, fmaf(a, bv, b * cv)), rd, dd > 0.0f);
    };
    constexpr int NB = 2;
    float zz[NB], xx[NB], yy[NB], val[NB];
    float s = 0.0f;
    if (F.cone_grid == 0) {
        for (int m = 1; m <= F.cone_rings; ++m) {
            const float c = (float)m, r = c * F.cone_tan;
            for (int t = 0; t < F.cone_angles; t += NB) {
#pragma unroll
                for (int w = 0; w < NB; ++w) {
                    const int i = min(t + w, F.cone_angles - 1);
                    tap(c, F.cone_cos[i] * r, F.cone_sin[i] * r, zz[w], xx[w], yy[w]);
                }
                lookup_batch<NB>(FromStack<SDT, SL, NEAR>{F}, zz, xx, yy, val);
#pragma unroll
                for (int w = 0; w < NB; ++w)
                    if (t + w < F.cone_angles) s += val[w];
            }
        }
    } else {
        const int G = F.cone_grid;
        const float rho = 0.5f * F.cone_tan, half = 0.5f * (float)(G - 1);
        for (int ia = 0; ia < G; ++ia) {
            const float a = ((float)ia - half) * rho;
            for (int ib = 0; ib < G; ib += NB) {
#pragma unroll
                for (int w = 0; w < NB; ++w)
                    tap(1.0f, a, ((float)min(ib + w, G - 1) - half) * rho, zz[w], xx[w], yy[w]);
                lookup_batch<NB>(FromStack<SDT, SL, NEAR>{F}, zz, xx, yy, val);
#pragma unroll
                for (int w = 0; w < NB; ++w)
                    if (ib + w < G) s += val[w];
            }
        }
    }
    return s * F.tap_w;
}

template <int MODE, int SDT, int SL, Near NEAR>
__device__ __forceinline__ float gather_point(const RenderFrame& F, float z, float d, float u, float v, float wd,
                                              float wu, float wv)
{
    if (MODE == kModePointShadow) {
        const float rd = __builtin_amdgcn_rcpf(d);
        return stack_lookup<SDT, SL, NEAR>(F, z, frustum_col(F, u, rd, d > 0.0f), frustum_col(F, v, rd, d > 0.0f));
    }
    if constexpr (MODE == kModePointCone) return gather_point_cone<SDT, SL, NEAR>(F, z, d, u, v, wd, wu, wv);
    // shell taps: world-frame offsets, each projected through its own depth
    // (batched as in gather())
    float s = 0.0f;
    constexpr int NB = shell_batch<MODE, SDT>();
    float zz[NB], xx[NB], yy[NB], val[NB];
    for (int t = 0; t < F.ntaps; t += 6) {
#pragma unroll kShellUnroll<SL == VI_STACK_TILED>
        for (int h = 0; h < 6; h += NB) {
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const int i = t + h + q;
                const float dt = d + F.td_[i], rd = __builtin_amdgcn_rcpf(dt);
                zz[q] = z + F.tz[i];
                xx[q] = frustum_col(F, u + F.tx_[i], rd, dt > 0.0f);
                yy[q] = frustum_col(F, v + F.ty_[i], rd, dt > 0.0f);
            }
            lookup_batch<NB>(FromStack<SDT, SL, NEAR>{F}, zz, xx, yy, val);
#pragma unroll
            for (int q = 0; q < NB; ++q) s = fmaf(F.tw[t + h + q], val[q], s);
        }
    }
    return s;
}

// The four lanes of a quad march one ray together: lane g takes segment k + g
// of every step.  The opacities of the four segments are composited front to
// back with a scan over the quad (inclusive product of (1 - alpha)), each
// segment's emission is weighted by the transmittance in front of it, and the
// ray stops exactly at the first segment after which 1 - alpha_dst <=
// term_eps.  All lanes of a quad carry the same ray state but for the colour,
// of which each lane sums its own segments until the ray ends.  Quads shorten
// the longest waves (rays of ~1000 non-empty segments) and pack the samples
// of a step within a couple of voxels.
//
// The quad's lanes exchange values by DPP quad permutes, which are operand
// modifiers of the VALU instruction that uses them; lane shuffles (thirteen
// LDS permutes a step, each with its index arithmetic and a wait) took a
// fifth of a frame's VALU instructions and all of its LDS waits.
template <int A, int B, int C, int D>
__device__ __forceinline__ float quad_perm(float x)
{
    return __int_as_float(
        __builtin_amdgcn_mov_dpp(__float_as_int(x), A | (B << 2) | (C << 4) | (D << 6), 0xf, 0xf, true));
}
// products of lanes 0..g
__device__ __forceinline__ float quad_scan_mul(float x, int g)
{
    float t = quad_perm<0, 0, 1, 2>(x);
    x = g >= 1 ? x * t : x;
    t = quad_perm<0, 1, 0, 1>(x);
    return g >= 2 ? x * t : x;
}
__device__ __forceinline__ float quad_min(float x)
{
    x = fminf(x, quad_perm<1, 0, 3, 2>(x));
    return fminf(x, quad_perm<2, 3, 0, 1>(x));
}
__device__ __forceinline__ float quad_sum(float x)
{
    x += quad_perm<1, 0, 3, 2>(x);
    return x + quad_perm<2, 3, 0, 1>(x);
}
// whether p holds in all four lanes of the quad (scalar arithmetic on the
// wave's ballot; lanes of finished rays do not matter)
__device__ __forceinline__ bool quad_all(bool p)
{
    unsigned long long m = __ballot(p);
    m &= m >> 1;
    m &= m >> 2;
    m &= 0x1111111111111111ull;
    m |= m << 1;
    m |= m << 2;
    return __builtin_amdgcn_inverse_ballot_w64(m);
}

// Per-ray march state (identical in the four lanes of a ray's quad but for
// the colour): the ray in offset-voxel coordinates, its light-grid maps, the
// cone basis or Phong vectors, the empty-space cache and the compositing
// state.
struct RayState {
    float hx0, hy0, hz0, hdx, hdy, hdz;  // entry point and direction
    float Df;                            // chord length, voxels
    float K;                             // segments (an integer below 2^24, as k and count)
    float qz0, qx0, qy0, qdz, qdx, qdy, pd0, pdd;
    ConeFrame cf;
    float lx, ly, lz, vx, vy, vz, lv;
    // distance to the face at voxel coordinate f (from the volume's corner)
    // along an axis: f ih + jb, with the faces moved inward (see ray_step)
    float ihx, ihy, ihz, jbx, jby, jbz;
    float Cr, Cg, Cb, T;
    uint32_t last_cell;                  // map without bits: the last cell looked up
    bool cell_is_empty;
    float k, count;
};

// how far the faces of an empty box are moved inward, in voxels: two orders
// above the float position error
constexpr float kJumpEps = 0.02f;

constexpr bool is_point_gather(int mode)
{
    return mode == kModePointShadow || mode == kModePointShell || mode == kModePointCone;
}

// Ray set-up for pixel (px, py): false if the ray misses the cube (the pixel
// is then the background).
template <typename VT, int LAYOUT, int MODE, int SDT, int SL>
__device__ __forceinline__ bool ray_setup(const RenderFrame& F, int px, int py, RayState& S)
{
    // ---- camera ray, in offset-voxel coordinates, in float pairs (the
    // host folded the camera and the light grid into float-pair
    // coefficients of h; see F2): pixel (px, py) -> b = base + px sx + py sy
    F2 o[3], d[3];
    {
        const F2 fx = f2((float)px), fy = f2((float)py);
        for (int a = 0; a < 3; ++a) {
            const F2 b = f2_add(F2{F.cam_b[a], F.cam_bl[a]},
                                f2_add(f2_mul(fx, F2{F.cam_sx[a], F.cam_sxl[a]}), f2_mul(fy, F2{F.cam_sy[a], F.cam_syl[a]})));
            if (F.cam_kind == VI_CAM_PERSP) {
                o[a] = F2{F.cam_o[a], F.cam_ol[a]};
                d[a] = b;
            } else {
                o[a] = b;
                d[a] = F2{F.cam_f[a], F.cam_fl[a]};
            }
        }
        if (F.cam_kind == VI_CAM_PERSP) {
            const F2 inv = f2_rsqrt(f2_dot3(d, d));
            for (int a = 0; a < 3; ++a) d[a] = f2_mul(d[a], inv);
        }
    }
    // ---- slab test against the cube [lo, hi]^3 (distances in voxels): the
    // entry and exit faces are picked in float, their distances then taken on
    // the pairs
    float tn = -3.0e38f, tf_ = 3.0e38f, bn = 0.0f, bf = 0.0f;
    int an = -1, af = -1;
    bool hit = true;
    for (int a = 0; a < 3; ++a) {
        if (d[a].hi == 0.0f) {
            if (o[a].hi < F.lo || o[a].hi > F.hi) hit = false;
            continue;
        }
        const float r = __builtin_amdgcn_rcpf(d[a].hi);
        const float near = d[a].hi > 0.0f ? F.lo : F.hi, far = d[a].hi > 0.0f ? F.hi : F.lo;
        const float t1 = (near - o[a].hi) * r, t2 = (far - o[a].hi) * r;
        if (t1 > tn) tn = t1, an = a, bn = near;
        if (t2 < tf_) tf_ = t2, af = a, bf = far;
    }
    if (!hit || af < 0 || !(tf_ > fmaxf(tn, 0.0f))) return false;
    // the chosen faces' numerators and denominators, gathered with constant
    // indices (a variable index would put o and d in scratch memory)
    F2 on = f2(0.0f), dn = f2(1.0f), of = f2(0.0f), df = f2(1.0f);
    for (int a = 0; a < 3; ++a) {
        on = a == an ? o[a] : on;
        dn = a == an ? d[a] : dn;
        of = a == af ? o[a] : of;
        df = a == af ? d[a] : df;
    }
    const F2 ti = (an >= 0 && tn > 0.0f) ? f2_div(f2_sub(f2(bn), on), dn) : f2(0.0f);
    const F2 tf = f2_div(f2_sub(f2(bf), of), df);
    if (!f2_lt(ti, tf)) return false;

    const F2 Dc = f2_sub(tf, ti);  // chord length, voxels
    S.Df = Dc.hi;
    {
        // K = ceil(D / dt), decided on the pair
        const F2 q = f2_mul(Dc, F2{F.idt, F.idtl});
        float c = ceilf(q.hi);
        if (c == q.hi && q.lo > 0.0f) c += 1.0f;
        else if (c - 1.0f - q.hi >= q.lo) c -= 1.0f;
        S.K = c;
    }
    // volume: entry point (value, remainder) and direction (value, remainder)
    F2 pin[3];
    for (int a = 0; a < 3; ++a) pin[a] = f2_add(o[a], f2_mul(ti, d[a]));
    S.hx0 = pin[0].hi, S.hy0 = pin[1].hi, S.hz0 = pin[2].hi;
    const float hdx = d[0].hi, hdy = d[1].hi, hdz = d[2].hi;
    S.hdx = hdx, S.hdy = hdy, S.hdz = hdz;
    // light grid: depth index (Eq. 9, minus one) and texel coordinates (Eq. 10)
    // (point light: qx / qy hold the lateral offsets U.(h - Ph), V.(h - Ph)
    // and pd the depth L.(h - Ph), all affine along the ray)
    constexpr bool PT = is_point_gather(MODE);
    constexpr bool PTP = MODE == kModePointPhong, PHONG = MODE == VI_MODE_PHONG || PTP;
    float& qz0 = S.qz0; float& qx0 = S.qx0; float& qy0 = S.qy0; float& qdz = S.qdz; float& qdx = S.qdx;
    float& qdy = S.qdy; float& pd0 = S.pd0; float& pdd = S.pdd;
    ConeFrame& cf = S.cf;
    qz0 = qx0 = qy0 = qdz = qdx = qdy = pd0 = pdd = 0.f;
    cf = ConeFrame{0.f, 0.f, 0.f, 0.f};
    // Phong: light vector l = -L and, folded in, l.v with v = -d
    // (point light: l is taken per sample toward P, and lx, ly, lz hold h_in - Ph)
    float& lx = S.lx; float& ly = S.ly; float& lz = S.lz; float& vx = S.vx; float& vy = S.vy; float& vz = S.vz;
    float& lv = S.lv;
    lx = ly = lz = vx = vy = vz = lv = 0.f;
    if (PHONG) {
        lx = -F.L[0];
        ly = -F.L[1];
        lz = -F.L[2];
        vx = -hdx;
        vy = -hdy;
        vz = -hdz;
        lv = fmaf(F.L[0], hdx, fmaf(F.L[1], hdy, F.L[2] * hdz));
        if (PTP) {
            lx = f2_sub(pin[0], F2{F.Ph[0], F.Phl[0]}).hi;
            ly = f2_sub(pin[1], F2{F.Ph[1], F.Phl[1]}).hi;
            lz = f2_sub(pin[2], F2{F.Ph[2], F.Phl[2]}).hi;
        }
    }
    if (MODE != VI_MODE_NONE && !PHONG) {
        const F2 Lq[3] = {F2{F.Lq[0], F.Lql[0]}, F2{F.Lq[1], F.Lql[1]}, F2{F.Lq[2], F.Lql[2]}};
        qz0 = f2_add(f2_dot3(Lq, pin), F2{F.Lq0, F.Lq0l}).hi;
        qdz = fmaf(F.Lq[0], hdx, fmaf(F.Lq[1], hdy, F.Lq[2] * hdz));
        if (PT) {
            const F2 r[3] = {f2_sub(pin[0], F2{F.Ph[0], F.Phl[0]}), f2_sub(pin[1], F2{F.Ph[1], F.Phl[1]}),
                             f2_sub(pin[2], F2{F.Ph[2], F.Phl[2]})};
            const F2 L[3] = {F2{F.L[0], F.Ll[0]}, F2{F.L[1], F.Ll[1]}, F2{F.L[2], F.Ll[2]}};
            const F2 U[3] = {F2{F.U[0], F.Ul[0]}, F2{F.U[1], F.Ul[1]}, F2{F.U[2], F.Ul[2]}};
            const F2 V[3] = {F2{F.V[0], F.Vl[0]}, F2{F.V[1], F.Vl[1]}, F2{F.V[2], F.Vl[2]}};
            pd0 = f2_dot3(L, r).hi;
            pdd = fmaf(F.L[0], hdx, fmaf(F.L[1], hdy, F.L[2] * hdz));
            qx0 = f2_dot3(U, r).hi;
            qdx = fmaf(F.U[0], hdx, fmaf(F.U[1], hdy, F.U[2] * hdz));
            qy0 = f2_dot3(V, r).hi;
            qdy = fmaf(F.V[0], hdx, fmaf(F.V[1], hdy, F.V[2] * hdz));
        } else {
            const F2 Ux[3] = {F2{F.Ux[0], F.Uxl[0]}, F2{F.Ux[1], F.Uxl[1]}, F2{F.Ux[2], F.Uxl[2]}};
            const F2 Vy[3] = {F2{F.Vy[0], F.Vyl[0]}, F2{F.Vy[1], F.Vyl[1]}, F2{F.Vy[2], F.Vyl[2]}};
            qx0 = f2_add(f2_dot3(Ux, pin), F2{F.Ux0, F.Ux0l}).hi;
            qy0 = f2_add(f2_dot3(Vy, pin), F2{F.Vy0, F.Vy0l}).hi;
            qdx = fmaf(F.Ux[0], hdx, fmaf(F.Ux[1], hdy, F.Ux[2] * hdz));
            qdy = fmaf(F.Vy[0], hdx, fmaf(F.Vy[1], hdy, F.Vy[2] * hdz));
        }
        if (MODE == VI_MODE_CONE || MODE == kModeConeGrid) {
            // B: direction toward the viewer with its L component removed
            // (U when the view runs along L)
            const float wl = -fmaf(hdx, F.L[0], fmaf(hdy, F.L[1], hdz * F.L[2]));
            float B[3] = {fmaf(-wl, F.L[0], -hdx), fmaf(-wl, F.L[1], -hdy), fmaf(-wl, F.L[2], -hdz)};
            const float nb = sqrtf(fmaf(B[0], B[0], fmaf(B[1], B[1], B[2] * B[2])));
            if (nb < 1e-6f) {
                for (int a = 0; a < 3; ++a) B[a] = F.U[a];
            } else {
                const float inb = 1.0f / nb;
                for (int a = 0; a < 3; ++a) B[a] *= inb;
            }
            const float P[3] = {F.L[1] * B[2] - F.L[2] * B[1], F.L[2] * B[0] - F.L[0] * B[2],
                                F.L[0] * B[1] - F.L[1] * B[0]};
            // B and L x B in texels per voxel
            cf.bx = fmaf(F.Ux[0], B[0], fmaf(F.Ux[1], B[1], F.Ux[2] * B[2]));
            cf.by = fmaf(F.Vy[0], B[0], fmaf(F.Vy[1], B[1], F.Vy[2] * B[2]));
            cf.px = fmaf(F.Ux[0], P[0], fmaf(F.Ux[1], P[1], F.Ux[2] * P[2]));
            cf.py = fmaf(F.Vy[0], P[0], fmaf(F.Vy[1], P[1], F.Vy[2] * P[2]));
        }
    }

    // (an axis the ray does not move along never limits a jump)
    const auto jump_axis = [&](float h0, float hd, float& ih, float& jb) {
        ih = hd != 0.f ? __builtin_amdgcn_rcpf(hd) : 0.f;
        jb = hd != 0.f ? ((hd > 0.f ? -kJumpEps : kJumpEps) - (float)F.M - h0) * ih : 3.0e38f;
    };
    jump_axis(S.hx0, hdx, S.ihx, S.jbx);
    jump_axis(S.hy0, hdy, S.ihy, S.jby);
    jump_axis(S.hz0, hdz, S.ihz, S.jbz);
    return true;
}

// Stage the window of the stack that the taps of the wave's `lit` samples (at
// light-grid position z, x, y) can reach in the wave's LDS tile; returns
// whether this lane's taps lie in it, and the tile element of light-grid cell
// (0, 0, 0).  Called with every lane of the wave.
//
// What bounds a gather of device memory is the L1: the 64 lanes of a load
// touch about 22 lines, one tag look-up each, and a cone's 32 loads took 79 %
// of the L1's cycles of a frame.  The samples of a step, 4 x 4 pixels by four
// segments, lie within a few texels, so the window that holds all their taps
// is read with a few 16-byte loads straight into LDS (one for every 16 rows
// of 16 texels), and the taps are LDS reads with immediate offsets and no
// clamps.  The window is centred between the first and the last lit sample;
// samples whose taps do not fit it (rays that see different depths) read the
// stack, and so does a wave with few samples.
constexpr int kStageMin = 12;  // samples
template <int MODE, int SDT, int SL>
constexpr bool kWindowed = SL == VI_STACK_ROWS && win_z(MODE, SDT) > 0;
template <int MODE, int SDT>
__device__ __forceinline__ bool stage_window(const RenderFrame& F, float* __restrict__ tile, bool lit, float z, float x,
                                             float y, int& org)
{
    constexpr int WY = win_y(MODE), WZ = win_z(MODE, SDT);
    constexpr int kLoads = WY * WZ / 16, kStep = 16 / WY;  // loads of 16 rows; layers per load
    static_assert(WY * WZ % 16 == 0 && 16 % WY == 0, "a load covers whole layers");
    const unsigned long long m = __ballot(lit);
    if (__popcll(m) < kStageMin) return false;
    // the window's first column, row and layer as stored (border and leading
    // layer included); columns on 16 bytes
    const int first = __ffsll(m) - 1, last = 63 - __clzll(m);
    const int ix = floor_int(x), iy = floor_int(y), iz = floor_int(z);
    const int mx = (__builtin_amdgcn_readlane(ix, first) + __builtin_amdgcn_readlane(ix, last)) >> 1;
    const int my = (__builtin_amdgcn_readlane(iy, first) + __builtin_amdgcn_readlane(iy, last)) >> 1;
    const int mz = (__builtin_amdgcn_readlane(iz, first) + __builtin_amdgcn_readlane(iz, last)) >> 1;
    // (its last column at most the last border texel's: a row's elements past
    // that one are the caller's, whatever they hold)
    const int wx = min(max((mx + F.Mr - 3) & ~3, 0), (F.res + 4 - kWinX) & ~3);
    const int wy = min(max(my + F.Mr + 2 - (WY / 2 - 1), 0), F.res + 4 - WY);
    const int wz = min(max(mz + F.Mz + 1 + F.st_oz, 0), F.n + 2 - WZ);
    // the same in light-grid coordinates, and the samples that fit
    const int ox = wx - 2 - F.Mr, oy = wy - 2 - F.Mr, oz = wz - 1 - F.Mz;
    const float hx = 0.5f * (float)(kWinX - 1), hy = 0.5f * (float)(WY - 1);
    const bool fit = lit & (fabsf(x - ((float)ox + hx)) < hx - F.st_reach) &
                     (fabsf(y - ((float)oy + hy)) < hy - F.st_reach) & (z + F.st_zmin >= (float)oz) &
                     (z + F.st_zmax < (float)(oz + WZ - 1));
    if (__popcll(__ballot(fit)) < kStageMin) return false;
    org = -((oz * WY + oy) * kWinX + ox);
    // row r of a load is row r % WY of layer r / WY; four lanes a row
    const uint32_t lane = threadIdx.x & 63u, r = lane >> 2;
    const uint32_t e0 = (uint32_t)wz * F.rlayer + (uint32_t)wy * F.rpitch + (uint32_t)wx;
    const uint32_t el = (r / WY) * F.rlayer + (r % WY) * F.rpitch + (lane & 3u) * 4u;
    // (this wave's reads of the last window have returned)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if constexpr (SDT == VI_F32) {
        const char* base = (const char*)F.stack_base + ((size_t)e0 << 2);
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(base + (el << 2)),
                                             (__attribute__((address_space(3))) void*)(tile + i * 256), 16, 0, 0);
            base += (size_t)(kStep * F.rlayer) << 2;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else {
        const char* base = (const char*)F.stack_base + ((size_t)e0 << 1);
        uint2 raw[kLoads];
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            raw[i] = *(const uint2*)(base + (el << 1));
            base += (size_t)(kStep * F.rlayer) << 1;
        }
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const float2 u = pair_value(PairRaw<SDT>{raw[i].x}), v = pair_value(PairRaw<SDT>{raw[i].y});
            ((float4*)tile)[i * 64 + lane] = make_float4(u.x, u.y, v.x, v.y);
        }
        // one wave writes and reads its tile: the LDS keeps its accesses in
        // order, only the compiler must
        asm volatile("" ::: "memory");
    }
    return fit;
}

// Composite the four segments of a step of every live ray (opacity 1 - om,
// colour er, eg, eb at distance sm), lit by the coefficient.
template <typename VT, int LAYOUT, int MODE, int SDT, int SL, Form FORM>
__device__ __forceinline__ void ray_shade(const RenderFrame& F, float* __restrict__ tile, RayState& S, bool live,
                                          bool in, float om, float er, float eg, float eb, float sm, float hx, float hy,
                                          float hz, uint32_t& nop)
{
    const int g = threadIdx.x & 3;
    constexpr bool PT = is_point_gather(MODE);
    constexpr bool PTP = MODE == kModePointPhong, PHONG = MODE == VI_MODE_PHONG || PTP;
    [[maybe_unused]] const VT* __restrict__ vol = (const VT*)F.vol;
    [[maybe_unused]] const VolIndex VI_ = {1u, F.vsy, F.vsz};
    // front to back over the four segments of this step (Eq. 3 in product
    // form): a segment is composited while the transmittance in front of it
    // is above term_eps, and the ray's transmittance becomes the last
    // composited segment's
    const float incl = quad_scan_mul(om, g);  // prod_{h<=g} (1 - alpha_h)
    const float up = quad_perm<0, 0, 1, 2>(incl);
    const float before = g == 0 ? S.T : S.T * up, after = S.T * incl;
    const bool seen = before > F.term_eps;
    const float Tnew = quad_min(seen ? after : 2.0f);
    const bool lit = seen && om < 1.0f;
    if (live) S.T = Tnew;
    // the taps of the wave's samples, staged in LDS where they lie close
    bool staged = false;
    [[maybe_unused]] FromWindow<win_y(MODE)> win{tile, 0};
    [[maybe_unused]] float qz, qx, qy;
    if constexpr (MODE != VI_MODE_NONE && !PHONG) {
        qz = fmaf(sm, S.qdz, S.qz0), qx = fmaf(sm, S.qdx, S.qx0), qy = fmaf(sm, S.qdy, S.qy0);
        if constexpr (FORM == Form::kStaged) staged = stage_window<MODE, SDT>(F, tile, lit, qz, qx, qy, win.org);
    }
    if (lit) {
        // emission alpha (sd rgb + ss) light: Eq. 7 with the coefficient A,
        // or the local Phong terms
        ++nop;
        const float wgt = before * (1.0f - om);
        float sd, ss = 0.0f;
        if (PHONG) {
            // central differences one voxel either side (exact
            // offsets in voxel units)
            const float gx = 0.5f * (sample_volume<VT, LAYOUT>(vol, VI_, F.N, F.M, F.vlo, F.vhi, F.scale, hx + 1.f, hy, hz) -
                                     sample_volume<VT, LAYOUT>(vol, VI_, F.N, F.M, F.vlo, F.vhi, F.scale, hx - 1.f, hy, hz));
            const float gy = 0.5f * (sample_volume<VT, LAYOUT>(vol, VI_, F.N, F.M, F.vlo, F.vhi, F.scale, hx, hy + 1.f, hz) -
                                     sample_volume<VT, LAYOUT>(vol, VI_, F.N, F.M, F.vlo, F.vhi, F.scale, hx, hy - 1.f, hz));
            const float gz = 0.5f * (sample_volume<VT, LAYOUT>(vol, VI_, F.N, F.M, F.vlo, F.vhi, F.scale, hx, hy, hz + 1.f) -
                                     sample_volume<VT, LAYOUT>(vol, VI_, F.N, F.M, F.vlo, F.vhi, F.scale, hx, hy, hz - 1.f));
            const float gn = sqrtf(fmaf(gx, gx, fmaf(gy, gy, gz * gz)));
            const float inv = -1.0f / fmaxf(gn, F.grad_eps);  // n = -g / max(|g|, eps)
            const float nx = gx * inv, ny = gy * inv, nz = gz * inv;
            const float vx = S.vx, vy = S.vy, vz = S.vz;
            float llx = S.lx, lly = S.ly, llz = S.lz, llv = S.lv;
            if (PTP) {
                // l = (P - p) / |P - p|
                const float rx = fmaf(sm, -vx, llx), ry = fmaf(sm, -vy, lly), rz = fmaf(sm, -vz, llz);
                const float ir = -__builtin_amdgcn_rsqf(fmaf(rx, rx, fmaf(ry, ry, rz * rz)));
                llx = rx * ir;
                lly = ry * ir;
                llz = rz * ir;
                llv = fmaf(llx, vx, fmaf(lly, vy, llz * vz));
            }
            const float nl = fmaf(nx, llx, fmaf(ny, lly, nz * llz));
            const float nv = fmaf(nx, vx, fmaf(ny, vy, nz * vz));
            const float nn = fmaf(nx, nx, fmaf(ny, ny, nz * nz));
            const float rv = fmaf(2.0f * nl, nv, -nn * llv);  // r.v, r = 2(n.l)n - (n.n)l
            sd = fmaf(F.phong_kd, fmaxf(nl, 0.0f), F.phong_ka);
            if (rv > 0.0f) ss = F.phong_ks * fast_exp2(F.phong_shin * fast_log2(rv));
        } else {
            // (the nearest-face form is a second copy of the
            // gather behind a branch that is uniform per frame)
            float A = 1.0f;
            const auto near_or_not = [&](auto from) {
                if constexpr (FORM == Form::kWide) return from(NearC<Near::kWide>());
                else return F.nearest ? from(NearC<Near::kYes>()) : from(NearC<Near::kNo>());
            };
            if constexpr (PT) {
                const float pd = fmaf(sm, S.pdd, S.pd0);
                A = near_or_not([&](auto near) {
                    return gather_point<MODE, SDT, SL, near()>(F, qz, pd, qx, qy, -S.pdd, -S.qdx, -S.qdy);
                });
            } else if constexpr (MODE != VI_MODE_NONE) {
                constexpr int NB = shell_batch<MODE, SDT>();
                const auto from = [&](auto near) {
                    return gather<MODE, NB>(F, FromStack<SDT, SL, near()>{F}, S.cf, qz, qx, qy);
                };
                if constexpr (FORM == Form::kStaged) A = staged ? gather<MODE, NB>(F, win, S.cf, qz, qx, qy)
                                                                : from(NearC<Near::kNo>());
                else A = near_or_not(from);
            }
            sd = fmaf(1.0f - F.ambient, A, F.ambient);
        }
        S.Cr = fmaf(wgt, fmaf(sd, er, ss), S.Cr);
        S.Cg = fmaf(wgt, fmaf(sd, eg, ss), S.Cg);
        S.Cb = fmaf(wgt, fmaf(sd, eb, ss), S.Cb);
    }
    if (live && S.T <= F.term_eps) {
        // composited segments of the step: the quad's lanes that were seen
        const unsigned long long m = __ballot(seen && in) >> (threadIdx.x & 60);
        S.count = S.k + (float)__popc((uint32_t)m & 15u);
    }
}

// One step of four segments of the march of every live ray of the wave (the
// lanes of a ray's quad take one segment each); clears `live` once a ray is
// done.  Where the gather stages windows the wave's lanes stay together
// (finished rays' lanes take part in the staging); elsewhere a quad leaves
// the loop with its ray.
template <typename VT, int LAYOUT, int MODE, int SDT, int SL, Form FORM>
__device__ __forceinline__ void ray_step(const RenderFrame& F, const float4* __restrict__ s_tf,
                                         const int* __restrict__ s_next, const uint32_t* __restrict__ s_bits,
                                         float* __restrict__ tile, RayState& S, bool& live, uint32_t& nop)
{
    const int g = threadIdx.x & 3;
    const VT* __restrict__ vol = (const VT*)F.vol;
    const VolIndex VI_ = {1u, F.vsy, F.vsz};
    const float Km1 = (float)(F.K - 1);
    const float kk = S.k + (float)g;
    const bool in = live && kk < S.K;
    float om = 1.f, sm = 0.f, hx = 0.f, hy = 0.f, hz = 0.f;  // om = 1 - alpha of the segment
    float er = 0.f, eg = 0.f, eb = 0.f;                      // its colour
    bool empty = true;
    float cx = 0.f, cy = 0.f, cz = 0.f;  // the segment's cell
    if (in) {
        const float s0 = kk * F.dt;
        const float s1 = fminf((kk + 1.0f) * F.dt, S.Df);
        const float len = s1 - s0;
        sm = 0.5f * (s0 + s1);
        hx = fmaf(sm, S.hdx, S.hx0), hy = fmaf(sm, S.hdy, S.hy0), hz = fmaf(sm, S.hdz, S.hz0);
        empty = false;
        if (F.occ.mm) {
            // The cell, by one multiply-add, clamp and truncation an axis.
            // Rounding may put a position within 1e-4 voxel of a cell's face
            // into the neighbour (h ic is exact, the sum rounds at 2^-24 of
            // at most 2^9 cells): its value is then within 1e-4 of the range
            // the map has for that cell, a tenth of a table entry for the
            // 1024 entries a table may have, and the emptiness test leaves
            // one whole entry on each side.
            cx = __builtin_amdgcn_fmed3f(fmaf(hx, F.occ.ic, F.occ.oc), 0.f, F.occ.cmax);
            cy = __builtin_amdgcn_fmed3f(fmaf(hy, F.occ.ic, F.occ.oc), 0.f, F.occ.cmax);
            cz = __builtin_amdgcn_fmed3f(fmaf(hz, F.occ.ic, F.occ.oc), 0.f, F.occ.cmax);
            const uint32_t c =
                __umul24(__umul24((uint32_t)cz, F.occ.nc) + (uint32_t)cy, F.occ.nc) + (uint32_t)cx;
            if (F.occ.bits) {
                empty = !occupancy_bit(s_bits, c);
            } else {
                if (c != S.last_cell) {
                    S.last_cell = c;
                    S.cell_is_empty = cell_empty(F.occ.mm[c], s_next, Km1, F.K);
                }
                empty = S.cell_is_empty;
            }
        }
        if (!empty) {
            const float v = sample_volume<VT, LAYOUT>(vol, VI_, F.N, F.M, F.vlo, F.vhi, F.scale, hx, hy, hz);
            const float x = v * Km1;
            const int e0 = min((int)x, F.K - 2);
            const float w = x - (float)e0;
            const float4 ta = s_tf[e0], tb = s_tf[e0 + 1];
            const float a = clampf01(fmaf(w, tb.w - ta.w, ta.w));
            // (1 - alpha) of a segment of length len: (1 - a)^(len / dref)
            if (len > 0.0f && a > 0.0f) om = fast_exp2(len * fast_log2(1.0f - a));
            er = fmaf(w, tb.x - ta.x, ta.x);
            eg = fmaf(w, tb.y - ta.y, ta.y);
            eb = fmaf(w, tb.z - ta.z, ta.z);
        }
    }
    const bool jump = live && quad_all(empty);
    float knext = S.k + 4.0f;
    if (jump) {
        // Every segment of this step is empty (or past the exit): jump to
        // the last segment midpoint inside the empty box around the step's
        // last segment -- the segment's cell, or the cell's super-cell (4 x 4
        // x 4 cells) when that is empty too -- with the box's faces moved
        // inward by kJumpEps voxels (far above the float position error), so
        // no segment with non-zero opacity is ever skipped.  The jump stays
        // on multiples of four so that the steps group segments as a march
        // without the map would (the products then round alike and the map
        // changes no bit of the result).  Each lane finds the last segment
        // inside the box around its own segment; the quad takes its last
        // lane's.  Per axis the exit face is the box's upper or lower one by
        // the ray's sign; no branches.  (A ray leaving through a lower face
        // of the volume takes the last half voxel, where positions clamp to
        // cell 0, in a step of its own.)
        float jl = S.K;
        if (in && F.occ.mm) {
            float size = (float)(1 << F.occ.shift), inv = 1.0f;
            if (F.occ.bits) {
                const uint32_t sx = (uint32_t)cx >> 2, sy = (uint32_t)cy >> 2, sz = (uint32_t)cz >> 2;
                const uint32_t sc = __umul24(__umul24(sz, F.occ.snc) + sy, F.occ.snc) + sx;
                if (!occupancy_bit(s_bits + F.occ.words, sc)) size *= 4.0f, inv = 0.25f;
            }
            const float fx = floorf(cx * inv) + (S.ihx > 0.f ? 1.0f : 0.0f);
            const float fy = floorf(cy * inv) + (S.ihy > 0.f ? 1.0f : 0.0f);
            const float fz = floorf(cz * inv) + (S.ihz > 0.f ? 1.0f : 0.0f);
            // distance along the ray to the box's exit faces
            const float se = fminf(fminf(fmaf(fx * size, S.ihx, S.jbx), fmaf(fy * size, S.ihy, S.jby)),
                                   fmaf(fz * size, S.ihz, S.jbz));
            // last full segment whose midpoint (j + 1/2) dt is <= se
            jl = fminf(floorf(fmaf(se, F.idt, -0.5f)), S.K - 1.0f);
        }
        const float jlast = quad_perm<3, 3, 3, 3>(jl);
        knext = fmaxf(knext, 4.0f * floorf(0.25f * (jlast + 1.0f)));
    }
    if (FORM == Form::kStaged ? __any(live && !jump) : !jump)
        ray_shade<VT, LAYOUT, MODE, SDT, SL, FORM>(F, tile, S, live, in, om, er, eg, eb, sm, hx, hy, hz, nop);
    S.k = knext;
    if (S.T <= F.term_eps || S.k >= S.K) live = false;
}

// The finished ray's colour over the background, and its segment count.
__device__ __forceinline__ float4 ray_result(const RenderFrame& F, const RayState& S)
{
    const float r = quad_sum(S.Cr) * F.light[0], g = quad_sum(S.Cg) * F.light[1], b = quad_sum(S.Cb) * F.light[2];
    return make_float4(fmaf(S.T, F.bg[0], r), fmaf(S.T, F.bg[1], g), fmaf(S.T, F.bg[2], b),
                       fmaf(S.T, F.bg[3], 1.0f - S.T));
}

// The per-ray values that the set-up hands to the march, in one order for
// writing and reading.
template <int MODE, typename FN>
__device__ __forceinline__ void ray_fields(RayState& S, FN f)
{
    constexpr bool PHONG = MODE == VI_MODE_PHONG || MODE == kModePointPhong;
    f(S.K), f(S.Df);
    f(S.hx0), f(S.hy0), f(S.hz0), f(S.hdx), f(S.hdy), f(S.hdz);
    f(S.ihx), f(S.ihy), f(S.ihz), f(S.jbx), f(S.jby), f(S.jbz);
    if constexpr (PHONG) {
        f(S.lx), f(S.ly), f(S.lz), f(S.lv);
    } else if constexpr (MODE != VI_MODE_NONE) {
        f(S.qz0), f(S.qx0), f(S.qy0), f(S.qdz), f(S.qdx), f(S.qdy);
        if constexpr (is_point_gather(MODE)) f(S.pd0), f(S.pdd);
        if constexpr (MODE == VI_MODE_CONE || MODE == kModeConeGrid) f(S.cf.bx), f(S.cf.by), f(S.cf.px), f(S.cf.py);
    }
}
constexpr int kRayFields = 24;  // the most of any mode

// --------------------------------------------------------------------------
// lane -> pixel mapping: kG lanes per ray; a wave covers WX x WY pixels, a
// workgroup 2 x 2 waves = BX x BY pixels.
// --------------------------------------------------------------------------
constexpr int kG = 4;  // lanes per ray: a DPP quad
constexpr int kWX = 4, kWY = 4;
constexpr int kBX = 2 * kWX, kBY = 2 * kWY;

// ray 0..63 of a workgroup, 16 a wave
__device__ __forceinline__ void ray_pixel(int ray, int* px, int* py)
{
    *px += ((ray >> 4) & 1) * kWX + ray % kWX;
    *py += (ray >> 5) * kWY + (ray & 15) / kWX;
}

// Segment counters: a wave sums its lanes' counts, the workgroup's waves add
// theirs in LDS, and the last wave to finish adds the workgroup's totals to
// the frame's counters -- one global atomic per workgroup and counter (one
// per wave measured up to twice the unlit frame's time: every wave of the
// frame hits the same two words).  No barrier: finished waves still leave.
struct GroupCount {
    unsigned long long ns, nop;
    uint32_t waves_done;
};
__device__ __forceinline__ void group_count_init(GroupCount* g)
{
    if (threadIdx.x == 0) {
        g->ns = 0;
        g->nop = 0;
        g->waves_done = 0;
    }
}
__device__ __forceinline__ void group_count_add(const RenderFrame& F, GroupCount* g, uint32_t ns, uint32_t nop)
{
    if (!F.samples) return;
    for (int off = 32; off > 0; off >>= 1) {
        ns += __shfl_xor(ns, off);
        nop += __shfl_xor(nop, off);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&g->ns, (unsigned long long)ns);
        atomicAdd(&g->nop, (unsigned long long)nop);
        __threadfence_block();
        if (atomicAdd(&g->waves_done, 1u) == blockDim.x / 64u - 1u) {
            const unsigned long long tn = atomicAdd(&g->ns, 0ull), to = atomicAdd(&g->nop, 0ull);
            if (tn) atomicAdd(F.samples, tn);
            if (to && F.count_opaque) atomicAdd(F.samples + 1, to);
        }
    }
}

// LDS of a workgroup: the frame's tables, then its four waves'
// areas, each for its stack window, if the frame stages, and, before the march,
// its rays.
constexpr size_t wave_words(int kmode, int stack_dtype, bool staged)
{
    const size_t w = staged ? window_bytes(kmode, stack_dtype) / 4 : 0;
    return w > 16 * kRayFields ? w : 16 * kRayFields;
}
constexpr size_t wave_bytes(int kmode, int stack_dtype, bool staged)
{
    return 4 * sizeof(float) * wave_words(kmode, stack_dtype, staged);
}

// `n` words from device memory to LDS, by the whole workgroup, without waiting
// for them (loads straight into LDS, 64 consecutive words each).
__device__ __forceinline__ void stage_words(const void* src, void* dst, uint32_t n)
{
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t at = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 64u; at < n; at += 256u)
        if (at + lane < n)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)((const uint32_t*)src + at + lane),
                (__attribute__((address_space(3))) void*)((uint32_t*)dst + at), 4, 0, 0);
}

// A workgroup's 8 x 8 pixels from (x0, y0).  While the tables are on their way
// to LDS one of its waves sets up all 64 rays, one a lane, and leaves them in
// the waves' areas; after the barrier the four lanes of a quad read their
// ray.  (Every wave setting up its 16 rays with four lanes each did the same
// work four times, a tenth of a frame's VALU instructions, after having waited
// for the tables.)  The waves take turns at it by workgroup, so that no SIMD
// gets all of it.
template <typename VT, int LAYOUT, int MODE, int SDT, int SL, Form FORM>
__device__ __forceinline__ void shade_block(const RenderFrame& F, float4* s_tf, int x0, int y0, uint32_t turn)
{
    __shared__ GroupCount gc;
    group_count_init(&gc);
    int* s_next = (int*)(s_tf + F.K);        // of a map without bits
    uint32_t* s_bits = (uint32_t*)s_next;
    stage_words(F.tf, s_tf, 4u * (uint32_t)F.K);
    if (F.occ.bits) stage_words(F.occ.bits, s_bits, F.occ.words + F.occ.swords);
    else if (F.occ.mm) build_next_opaque(s_next, F.tf, F.K);

    constexpr uint32_t kWords = (uint32_t)wave_words(MODE, SDT, FORM == Form::kStaged);
    float* areas = (float*)((char*)s_tf + F.tables);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
    RayState S = {};
    if (wave == (turn & 3u)) {
        int px = x0, py = y0;
        ray_pixel((int)lane, &px, &py);
        bool hit = px < F.width && py < F.height;
        if (hit) hit = ray_setup<VT, LAYOUT, MODE, SDT, SL>(F, px, py, S);
        if (!hit) S.K = 0.0f;
        float* at = areas + (lane >> 4) * kWords + (lane & 15u);
        int i = 0;
        ray_fields<MODE>(S, [&](float& v) { at[16 * i++] = v; });
    }
    // (the words that this wave has on their way to LDS)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    float* tile = areas + wave * kWords;  // this wave's rays, then its stack window
    S = {};
    {
        const float* at = tile + (lane >> 2);
        int i = 0;
        ray_fields<MODE>(S, [&](float& v) { v = at[16 * i++]; });
    }
    S.vx = -S.hdx, S.vy = -S.hdy, S.vz = -S.hdz;
    S.last_cell = 0xffffffffu;
    // C: premultiplied colour so far (0); T = 1 - alpha_dst, the transmittance in
    // front of the next segment (kept as a product of exact per-segment
    // factors, which keeps its relative precision down to term_eps).
    S.T = 1.0f;
    S.count = S.K;
    const bool hit = S.K > 0.0f;
    bool live = hit;
    uint32_t ns = 0, nop = 0;
    while (FORM == Form::kStaged ? __any(live) : live)
        ray_step<VT, LAYOUT, MODE, SDT, SL, FORM>(F, s_tf, s_next, s_bits, tile, S, live, nop);
    int px = x0, py = y0;
    ray_pixel((int)(threadIdx.x >> 2), &px, &py);
    if (hit) {
        const float4 c = ray_result(F, S);
        if ((lane & 3u) == 0u) {
            ns = (uint32_t)fminf(S.count, S.K);
            F.out[(size_t)py * F.width + px] = c;
        }
    } else if (px < F.width && py < F.height && (lane & 3u) == 0u) {
        F.out[(size_t)py * F.width + px] = make_float4(F.bg[0], F.bg[1], F.bg[2], F.bg[3]);
    }
    group_count_add(F, &gc, ns, nop);
}

// --------------------------------------------------------------------------
// single-frame kernel
// --------------------------------------------------------------------------
template <typename VT, int LAYOUT, int MODE, int SDT, int SL, Form FORM>
__device__ __forceinline__ void render_frame(const RenderFrame& F)
{
    extern __shared__ float4 s_tf[];
    const uint32_t tiles_x = (F.width + kBX - 1) / kBX, tiles_y = (F.height + kBY - 1) / kBY;
    uint32_t tx, ty;
    if (!supertile_of(blockIdx.x, tiles_x, tiles_y, &tx, &ty)) return;
    shade_block<VT, LAYOUT, MODE, SDT, SL, FORM>(F, s_tf, (int)tx * kBX, (int)ty * kBY, blockIdx.x / kXcds);
}

// --------------------------------------------------------------------------
// batched kernel (serving): the launch lists 16 x 16-pixel tiles of any frames
// of one mode; each tile is covered by (16/BX) x (16/BY) workgroups, each
// reading its frame's parameters from device memory.  Per pixel it runs the
// same shade_block as render_kernel, so a frame is bit-identical alone and in a
// mix.  (One kernel per mode keeps each mode's register budget: a kernel
// holding every mode runs all of them at the occupancy of the largest.)
// --------------------------------------------------------------------------
constexpr uint32_t kSubX = 16 / kBX, kSubY = 16 / kBY, kSub = kSubX * kSubY;

template <typename VT, int LAYOUT, int MODE, int SDT, int SL, Form FORM>
__device__ __forceinline__ void render_tiles(const RenderFrame* __restrict__ frames, const uint32_t* __restrict__ tiles,
                                             uint32_t ntiles)
{
    extern __shared__ float4 s_tf[];
    uint32_t q;
    if (!list_of(blockIdx.x, ntiles * kSub, &q)) return;
    const uint32_t t = tiles[q / kSub], sub = q % kSub;
    const RenderFrame& F = frames[t >> 22];
    shade_block<VT, LAYOUT, MODE, SDT, SL, FORM>(F, s_tf, (int)((t & 2047u) * kSubX + sub % kSubX) * kBX,
                                           (int)(((t >> 11) & 2047u) * kSubY + sub / kSubX) * kBY, blockIdx.x / kXcds);
}

// The kernels, one per mode.  Over a float row stack the shell, the ring cone
// and the lattice are held to six waves per SIMD (80 VGPRs, no spills): the
// lattice 1155 -> 1094 us, the cone 1208 -> 1195.  Five holds the point cones (105
// to 96 VGPRs: 256^3 float 771 -> 728 us, half 835 -> 800; six spill, 863 and 900)
// and the staged half ring cone (100 to 91: 768 -> 686); the unlit, shadow, Phong,
// point shell and 2-byte shell kernels take 55 to 79 registers whatever is asked
// for and run in the same time.  The tiled layout's lookups keep the compiler's
// four (with the branches that tap_load names five and six were slower; without
// them five lets the bfloat16 decoding spill its time, ring cone 1310 -> 1565 us).
template <int MODE, int SDT, int SL>
constexpr int kMinWaves = SL != VI_STACK_ROWS ? 1
                          : SDT == VI_F32 && (MODE == VI_MODE_SHELL || MODE == VI_MODE_CONE || MODE == kModeConeGrid)
                              ? 6
                              : 5;
template <typename VT, int LAYOUT, int MODE, int SDT, int SL, Form FORM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kMinWaves<MODE, SDT, SL>))) void render_kernel(
    RenderFrame F)
{
    render_frame<VT, LAYOUT, MODE, SDT, SL, FORM>(F);
}
template <typename VT, int LAYOUT, int MODE, int SDT, int SL, Form FORM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kMinWaves<MODE, SDT, SL>))) void
render_batch_kernel(const RenderFrame* __restrict__ frames, const uint32_t* __restrict__ tiles, uint32_t ntiles)
{
    render_tiles<VT, LAYOUT, MODE, SDT, SL, FORM>(frames, tiles, ntiles);
}

template <int MODE, int SL>
constexpr bool kReadsRows = SL == VI_STACK_ROWS && MODE != VI_MODE_NONE && MODE != VI_MODE_PHONG && MODE != kModePointPhong;

template <typename FN>
static hipError_t with_mode(int mode, FN fn)
{
    switch (mode) {
    case VI_MODE_NONE: fn(std::integral_constant<int, VI_MODE_NONE>()); break;
    case VI_MODE_SHADOW: fn(std::integral_constant<int, VI_MODE_SHADOW>()); break;
    case VI_MODE_SHELL: fn(std::integral_constant<int, VI_MODE_SHELL>()); break;
    case VI_MODE_CONE: fn(std::integral_constant<int, VI_MODE_CONE>()); break;
    case kModePointShadow: fn(std::integral_constant<int, kModePointShadow>()); break;
    case kModePointShell: fn(std::integral_constant<int, kModePointShell>()); break;
    case kModePointPhong: fn(std::integral_constant<int, kModePointPhong>()); break;
    case kModeConeGrid: fn(std::integral_constant<int, kModeConeGrid>()); break;
    case kModePointCone: fn(std::integral_constant<int, kModePointCone>()); break;
    default: fn(std::integral_constant<int, VI_MODE_PHONG>()); break;
    }
    return hipGetLastError();
}

template <typename VT, int LAYOUT, int SDT, int SL>
static hipError_t launch_batch_t(int mode, bool staged, const RenderFrame* d_frames, const uint32_t* d_tiles,
                                 uint32_t ntiles, size_t tables, hipStream_t s)
{
    const dim3 grid(list_grid(ntiles * kSub)), block(256);
    return with_mode(mode, [&](auto m) {
        constexpr int MODE = m();
        const size_t lds = tables + wave_bytes(MODE, SDT, staged);
        if constexpr (kWindowed<MODE, SDT, SL>)
            if (staged) {
                hipLaunchKernelGGL((render_batch_kernel<VT, LAYOUT, MODE, SDT, SL, Form::kStaged>), grid, block, lds, s, d_frames,
                                   d_tiles, ntiles);
                return;
            }
        hipLaunchKernelGGL((render_batch_kernel<VT, LAYOUT, MODE, SDT, SL, Form::kPlain>), grid, block, lds, s, d_frames,
                           d_tiles, ntiles);
    });
}

template <typename VT, int LAYOUT>
static hipError_t launch_batch_l(int sdt, int sl, int mode, bool staged, const RenderFrame* f, const uint32_t* t,
                                 uint32_t n, size_t tables, hipStream_t s)
{
    if (sdt == VI_BF16)
        return sl == VI_STACK_ROWS ? launch_batch_t<VT, LAYOUT, VI_BF16, VI_STACK_ROWS>(mode, staged, f, t, n, tables, s)
                                   : launch_batch_t<VT, LAYOUT, VI_BF16, VI_STACK_TILED>(mode, staged, f, t, n, tables, s);
    if (sdt == VI_F16)  // row layout only
        return launch_batch_t<VT, LAYOUT, VI_F16, VI_STACK_ROWS>(mode, staged, f, t, n, tables, s);
    return sl == VI_STACK_ROWS ? launch_batch_t<VT, LAYOUT, VI_F32, VI_STACK_ROWS>(mode, staged, f, t, n, tables, s)
                               : launch_batch_t<VT, LAYOUT, VI_F32, VI_STACK_TILED>(mode, staged, f, t, n, tables, s);
}

template <typename VT, int LAYOUT, int SDT, int SL>
static hipError_t launch_mode(const RenderFrame& f, hipStream_t s)
{
    const dim3 grid(supertile_grid((f.width + kBX - 1) / kBX, (f.height + kBY - 1) / kBY)), block(256);
    return with_mode(kernel_mode(f), [&](auto m) {
        constexpr int MODE = m();
        const size_t lds = f.tables + wave_bytes(MODE, SDT, f.stage != 0);
        if constexpr (kWindowed<MODE, SDT, SL>)
            if (f.stage) {
                hipLaunchKernelGGL((render_kernel<VT, LAYOUT, MODE, SDT, SL, Form::kStaged>), grid, block, lds, s, f);
                return;
            }
        // (no batch has wide layers: the server builds its stacks itself)
        if constexpr (kReadsRows<MODE, SL>)
            if (f.wide) {
                hipLaunchKernelGGL((render_kernel<VT, LAYOUT, MODE, SDT, SL, Form::kWide>), grid, block, lds, s, f);
                return;
            }
        hipLaunchKernelGGL((render_kernel<VT, LAYOUT, MODE, SDT, SL, Form::kPlain>), grid, block, lds, s, f);
    });
}

template <typename VT, int LAYOUT>
static hipError_t launch_sdt(const RenderFrame& f, hipStream_t s)
{
    const bool q = f.stack_layout == VI_STACK_ROWS;
    if (f.stack_dtype == VI_BF16)
        return q ? launch_mode<VT, LAYOUT, VI_BF16, VI_STACK_ROWS>(f, s) : launch_mode<VT, LAYOUT, VI_BF16, VI_STACK_TILED>(f, s);
    if (f.stack_dtype == VI_F16)  // row layout only
        return launch_mode<VT, LAYOUT, VI_F16, VI_STACK_ROWS>(f, s);
    return q ? launch_mode<VT, LAYOUT, VI_F32, VI_STACK_ROWS>(f, s) : launch_mode<VT, LAYOUT, VI_F32, VI_STACK_TILED>(f, s);
}

// One compilation of this file holds the kernels of one voxel type and volume
// layout (VI_RENDER_PART = dtype * 3 + layout; the builder compiles all
// twelve side by side: one compilation of every kernel took six minutes).
#ifndef VI_RENDER_PART
#error "compile with -DVI_RENDER_PART=dtype*3+layout (0..11)"
#endif
constexpr int kPartDtype = VI_RENDER_PART / 3, kPartLayout = VI_RENDER_PART % 3;
template <int DT> struct VoxelType { using T = float; };
template <> struct VoxelType<VI_U8> { using T = uint8_t; };
template <> struct VoxelType<VI_U16> { using T = uint16_t; };
template <> struct VoxelType<VI_F16> { using T = __half; };

template <>
hipError_t launch_render_part<VI_RENDER_PART>(const RenderFrame& f, hipStream_t s)
{
    return launch_sdt<VoxelType<kPartDtype>::T, kPartLayout>(f, s);
}

template <>
hipError_t launch_render_batch_part<VI_RENDER_PART>(int stack_dtype, int stack_layout, int mode, bool staged,
                                                    const RenderFrame* d_frames, const uint32_t* d_tiles,
                                                    uint32_t ntiles, size_t tables, hipStream_t s)
{
    return launch_batch_l<VoxelType<kPartDtype>::T, kPartLayout>(stack_dtype, stack_layout, mode, staged, d_frames,
                                                                 d_tiles, ntiles, tables, s);
}

}  // namespace vi
