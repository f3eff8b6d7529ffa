// vi_build.hip -- light-space attenuation build (section 3.2.1, Alg. 1).
//
// Every texel column of the light square is scanned over the n slabs from
// the light (Eq. 8 ordering): per slab the volume is sampled at the slab
// midpoint, the transfer-function opacity is looked up and corrected to the
// slab thickness (extinction form, Eq. 6), and the running transmittance is
// multiplied by (1 - alpha) -- Eq. 4 applied to opacity.  Every layer is
// written within a few slabs of being known (the row layout holds eight
// layers in LDS before storing them), so the pass is one
// streaming sweep: the volume is read through the caches and the stack is
// written once.
//
// Mapping: one workgroup per run of consecutive elements of a layer, one
// column per lane.  In the row layout a run is a stretch of the layer's element
// range, border included (build_rows); in the tiled layout a run of one stack
// row (build_tiled).
// At every slab a workgroup stores its run as one contiguous stretch of the
// layer (up to 4 KiB); many short runs spread over the layer
// (64 x 4 texel tiles per workgroup) measured at half that write rate.  The
// 64 lanes of a wave hold 64 neighbouring columns (of at most two rows), so
// each volume gather of a wave stays compact.
//
// Per column the slabs whose midpoints lie in the cube form one interval
// [k_in, k_out], found once, exactly; a wave runs the full
// per-slab work (fetch, transfer function, Eq. 6 correction, product) only
// for slabs in its columns' union of intervals, and otherwise only stores
// (the unattenuated value in front, the final transmittance behind).
// Empty-space verdicts come from the occupancy bits in LDS (without bits
// every slab in the cube is fetched).
//
// Slab-midpoint positions are fixed-point numbers (h * 2^40 in an int64, h
// the offset-voxel coordinate), so stepping from slab to slab is an exact
// integer add and the voxel index and trilinear weight are exact bit fields
// of the position: no rounding accumulates over the 512 slabs, and a float
// would resolve |h| ~ N/2 only to 2^-16 voxel.
#include <algorithm>

#include "vi_device.h"
#include "vi_internal.h"

namespace vi {

// Workgroup b -> (row, run): rows (in the row layout, runs of about a row
// of the layer's element range) are dealt to the 8 XCDs in groups of 4
// consecutive ones (neighbouring rows sample the same voxels and share an
// L2), the groups of an XCD spread over the whole light square.
constexpr uint32_t kRowGroup = 4;
__device__ __forceinline__ bool row_run_of(uint32_t b, uint32_t rows, uint32_t runs, uint32_t* row, uint32_t* run)
{
    const uint32_t x = b % kXcds, q = b / kXcds;  // XCD, index within it
    const uint32_t unit = q / runs, r = q % runs;
    const uint32_t grp = unit / kRowGroup, within = unit % kRowGroup;
    *row = (grp * kXcds + x) * kRowGroup + within;
    *run = r;
    return *row < rows;
}
inline uint32_t row_run_grid(uint32_t rows, uint32_t runs)
{
    const uint32_t groups = (rows + kRowGroup - 1) / kRowGroup;
    return (groups + kXcds - 1) / kXcds * kRowGroup * runs * kXcds;
}

// Q40 positions: floor(h) and the trilinear weight h - floor(h) (its top 24
// bits, exact in a float).
__device__ __forceinline__ int q_floor(int64_t H) { return (int)(H >> kQBits); }
__device__ __forceinline__ float q_frac(int64_t H)
{
    return (float)((uint32_t)((uint64_t)H >> (kQBits - 24)) & 0xFFFFFFu) * (1.0f / 16777216.0f);
}
__device__ __forceinline__ float q_to_float(int64_t H) { return (float)H * (1.0f / 1099511627776.0f); }

// floor(a / b) for b > 0, as far as it lies in [-1, n] (otherwise some value
// beyond that end): an estimate in float, within 2^-21 (n + 1) of the quotient
// clamped to [-1, n], corrected by the exact remainder.  (A 64-bit division is
// some hundred instructions, and a column takes six.)
__device__ __forceinline__ int floor_div(int64_t a, int64_t b, int n)
{
    const float q = __builtin_amdgcn_fmed3f((float)a * __builtin_amdgcn_rcpf((float)b), -1.0f, (float)n);
    int k = (int)floorf(q);
    const int64_t r = a - k * b;
    if (r < 0) --k;
    else if (r >= b) ++k;
    return k;
}
// The slabs of a column whose midpoints lie in the cube: k in [k_in, k_out]
// (empty when k_in > k_out), exactly as the per-slab test lo <= h_k <= hi
// on all three axes decides it: per axis a half-line or interval of k from
// exact quotients of Q40 values.
__device__ __forceinline__ void slab_range(const int64_t H[3], const int64_t A[3], int n, int64_t lo, int64_t hi,
                                           int* k_in, int* k_out)
{
    int kl = 0, kh = n - 1;
    for (int a = 0; a < 3; ++a) {
        if (A[a] == 0) {
            if (H[a] < lo || H[a] > hi) kl = n;  // never inside along this axis
        } else {
            // k A in [lo - H, hi - H]; for a step against the axis mirrored
            const int64_t st = A[a] > 0 ? A[a] : -A[a];
            const int64_t from = A[a] > 0 ? lo - H[a] : H[a] - hi, to = A[a] > 0 ? hi - H[a] : H[a] - lo;
            kl = max(kl, floor_div(from + (st - 1), st, n));  // the ceiling
            kh = min(kh, floor_div(to, st, n));
        }
    }
    if (kl > kh) {
        *k_in = n;
        *k_out = -1;
    } else {
        *k_in = kl;
        *k_out = kh;
    }
}

__device__ __forceinline__ int wave_min(int v)
{
    for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off));
    return v;
}
__device__ __forceinline__ int wave_max(int v)
{
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off));
    return v;
}

// One texel of a tiled stack: transmittance (F32) or optical depth in base-2
// units, -log2 T (BF16).
// (The stack is below 4 GiB: byte offsets in 32 bits, so a store takes the
// stack's base from scalar registers.)
template <int OUT_DTYPE>
__device__ __forceinline__ void put_texel(void* out, uint32_t at, float T, float tau)
{
    static_assert(OUT_DTYPE == VI_F32 || OUT_DTYPE == VI_BF16, "half stacks have the row layout");
    if (OUT_DTYPE == VI_F32) *(float*)((char*)out + (at << 2)) = T;
    else *(uint16_t*)((char*)out + (at << 1)) = f32_to_bf16(tau);
}

// An empty statement that reads a fetched footprint's registers.  Placed
// after all loads of a pair of slabs, it is the one point where they must
// have arrived, so the compiler waits there once for all of them; without it
// the loads of a slab fetched only by some lanes left their registers pending
// across the loop's back edge, and the compiler waited for the first slab's
// loads before issuing the second slab's (8 % slower).
template <typename T>
__device__ __forceinline__ void keep_value(const T& x)
{
    if constexpr (sizeof(T) == 8) asm volatile("" ::"v"(__builtin_bit_cast(uint64_t, x)));
    else if constexpr (sizeof(T) == 4) asm volatile("" ::"v"(__builtin_bit_cast(uint32_t, x)));
    else if constexpr (sizeof(T) == 2) asm volatile("" ::"v"((uint32_t)__builtin_bit_cast(uint16_t, x)));
    else if constexpr (sizeof(T) == 1) asm volatile("" ::"v"((uint32_t)__builtin_bit_cast(uint8_t, x)));
    else {
        struct W { uint64_t lo, hi; };
        const W w = __builtin_bit_cast(W, x);
        asm volatile("" ::"v"(w.lo), "v"(w.hi));
    }
}
template <typename VT, int LAYOUT>
__device__ __forceinline__ void keep_foot(const RawFoot<VT, LAYOUT>& r)
{
    if constexpr (LAYOUT == VI_LAYOUT_QUAD4) {
        keep_value(r.a);
        keep_value(r.b);
    } else if constexpr (LAYOUT == VI_LAYOUT_LINEAR) {
#pragma unroll
        for (int i = 0; i < 4; ++i) keep_value(r.p[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) keep_value(r.v[i]);
    }
}

// LDS of the tables (K alphas and `words` words of bits), up to 16 bytes.
__host__ __device__ inline size_t build_table_bytes(int K, uint32_t words)
{
    return (sizeof(float) * (size_t)K + sizeof(uint32_t) * (size_t)words + 15) / 16 * 16;
}

// Shared set-up of both layouts: the TF's opacities and the occupancy bits
// in LDS.  Empty-space verdicts come from the bits; without them one set bit
// stands for "every cell may hold opacity" (cell index 0).  Returns the
// number of 32-bit words the bits take.
__device__ __forceinline__ uint32_t stage_build_tables(const BuildParams& P, float* s_alpha, uint32_t* s_bits)
{
    for (int t = threadIdx.x; t < P.K; t += blockDim.x) s_alpha[t] = P.tf[4 * t + 3];
    if (P.occ.bits != nullptr) {
        stage_occupancy(P.occ, s_bits);
        return P.occ.words + P.occ.swords;
    }
    if (threadIdx.x == 0) s_bits[0] = 1u;
    return 1u;
}

// The slab-0 midpoint of column (i, j) and (point light) its step, in Q40,
// the step's length in voxels, and the column's slabs inside the cube.
template <bool PT>
__device__ __forceinline__ void column_setup(const BuildParams& P, int i, int j, bool grid, int64_t H[3], int64_t A[3],
                                             float* e, int* kin, int* kout)
{
    for (int a = 0; a < 3; ++a) H[a] = P.B0q[a] + (int64_t)i * P.BUq[a] + (int64_t)j * P.BVq[a];
    if constexpr (PT) {
        for (int a = 0; a < 3; ++a) A[a] = P.ALq[a] + (int64_t)i * P.ALUq[a] + (int64_t)j * P.ALVq[a];
        const float ax = q_to_float(A[0]), ay = q_to_float(A[1]), az = q_to_float(A[2]);
        *e = sqrtf(fmaf(ax, ax, fmaf(ay, ay, az * az)));
    } else {
        for (int a = 0; a < 3; ++a) A[a] = P.ALq[a];
        *e = P.e;
    }
    if (grid) {
        slab_range(H, A, P.n, P.loq, P.hiq, kin, kout);
    } else {
        *kin = P.n;  // border, padding or past the grid: no slab
        *kout = -1;
    }
}

// A slab midpoint in Q40: its footprint's lower voxel, trilinear weights and
// whether it must be fetched (slab k inside the column's cube interval and
// its cell possibly opaque; a zero-opacity cell leaves T unchanged exactly).
struct SlabProbe {
    int gx, gy, gz;
    float wx, wy, wz;
    bool fetch;
};
__device__ __forceinline__ SlabProbe probe_slab(const BuildParams& P, int64_t hx, int64_t hy, int64_t hz, int k, int kin,
                                                int kout, const uint32_t* s_bits, int cshift, uint32_t cnc)
{
    SlabProbe s;
    s.gx = q_floor(hx) + P.M;
    s.gy = q_floor(hy) + P.M;
    s.gz = q_floor(hz) + P.M;
    s.wx = q_frac(hx);
    s.wy = q_frac(hy);
    s.wz = q_frac(hz);
    const uint32_t cell = cell_of(s.gx, s.gy, s.gz, P.N, cshift, cnc);
    s.fetch = k >= kin && k <= kout && occupancy_bit(s_bits, cell);
    return s;
}

// One slab of a column (Alg. 1): the volume value at the slab midpoint, the
// TF opacity clamped to [0, 1] as the render clamps it, corrected to the
// slab thickness (Eq. 6, extinction form: e = ds / dref), applied to the
// transmittance T (F32) or added to the optical depth tau in base-2 units
// (2-byte stacks).  `darken` applies the section 4 compensation
// (1 + alpha)^m; m = 0 leaves every factor unchanged exactly.
template <typename VT, int LAYOUT, int OUT_DTYPE>
__device__ __forceinline__ void slab_step(const BuildParams& P, const float* s_alpha, const RawFoot<VT, LAYOUT>& raw,
                                          const SlabProbe& s, float e, bool darken, float& T, float& tau)
{
    const float v = foot_value<VT, LAYOUT>(raw, s.wx, s.wy, s.wz, P.scale);
    const float x = v * (float)(P.K - 1);
    const int e0 = min((int)x, P.K - 2);
    const float w = x - (float)e0;
    const float a = clampf01(fmaf(w, s_alpha[e0 + 1] - s_alpha[e0], s_alpha[e0]));
    const float l2 = fast_log2(1.0f - a);  // -inf for a = 1
    if (OUT_DTYPE == VI_F32) {
        // (1 - alpha(ds)) = (1 - a)^(ds / dref) = 2^(e log2(1 - a))
        float f = fast_exp2(e * l2);
        // section 4 compensation: times (1 + alpha)^m, at most 1
        if (darken) f = fminf(f * fast_exp2(P.darken * fast_log2(2.0f - f)), 1.0f);
        T *= f;
    } else {
        // optical depth in base-2 units: sigma ds / ln 2 = -e log2(1 - a),
        // capped at 64 / ln 2 per slab (a factor e^-64); the compensation
        // subtracts m log2(1 + alpha), floored at 0
        float dtau = -e * l2;
        if (darken) dtau = fmaxf(dtau - P.darken * fast_log2(2.0f - fast_exp2(e * l2)), 0.0f);
        tau += fminf(dtau, 92.332482616893656f);
    }
}

// Tiled layout: one workgroup per run of NT texels of one stack row, a column a
// lane.  Slabs in front of a wave's columns' union of cube intervals and behind it
// are stored without touching the volume; inside, batches of B slabs: positions
// and empty-space verdicts, then every volume load of the batch, and only then
// the arithmetic and the stores -- one wait per batch.
template <typename VT, int LAYOUT, int OUT_DTYPE, bool PT, int NT, int B>
__device__ __forceinline__ void build_tiled(const BuildParams& P)
{
    extern __shared__ float s_alpha[];  // K alphas, then the occupancy bits
    uint32_t* s_bits = (uint32_t*)(s_alpha + P.K);
    stage_build_tables(P, s_alpha, s_bits);
    const bool use_bits = P.occ.bits != nullptr;
    const int cshift = use_bits ? P.occ.shift : 30;
    const uint32_t cnc = use_bits ? P.occ.nc : 1u;
    __syncthreads();

    const uint32_t runs = ((uint32_t)P.res + NT - 1) / NT;
    uint32_t row, run;
    if (!row_run_of(blockIdx.x, (uint32_t)P.res, runs, &row, &run)) return;
    const int i = (int)(run * NT + threadIdx.x), j = (int)row;
    const bool col = i < P.res;

    int64_t H[3], A[3];
    float ex;
    int kin, kout;
    column_setup<PT>(P, i, j, col, H, A, &ex, &kin, &kout);
    uint32_t at = stack_oj(j, P.row_tiles32) + stack_oi(i);
    // the wave's slabs with any midpoint in the cube: [kmin, kmax]
    const int kmin = __builtin_amdgcn_readfirstlane(wave_min(kin));
    const int kmax = __builtin_amdgcn_readfirstlane(wave_max(kout));
    const uint32_t layer = P.layer;

    // slabs in front of the cube: the light arrives unattenuated
    for (int k = 0; k < min(kmin, P.n); ++k) {
        if (col) put_texel<OUT_DTYPE>(P.out, at, 1.0f, 0.0f);
        at += layer;
    }

    const VT* __restrict__ vol = (const VT*)P.vol;
    const VolIndex VI_ = {1u, P.vsy, P.vsz};
    float T = 1.0f, tau = 0.0f;
    const int kstart = kmin < P.n ? kmin : 0;
    for (int a = 0; a < 3; ++a) H[a] += (int64_t)kstart * A[a];  // positions at slab kmin
    const bool darken = P.darken > 0.0f;

    for (int k0 = kmin; k0 <= kmax; k0 += B) {
        SlabProbe sp[B];
        RawFoot<VT, LAYOUT> raw[B];
#pragma unroll
        for (int u = 0; u < B; ++u)
            sp[u] = probe_slab(P, H[0] + (int64_t)u * A[0], H[1] + (int64_t)u * A[1], H[2] + (int64_t)u * A[2], k0 + u,
                               kin, kout, s_bits, cshift, cnc);
        for (int a = 0; a < 3; ++a) H[a] += (int64_t)B * A[a];
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (sp[u].fetch)
                foot_load_g<VT, LAYOUT>(raw[u], sp[u].wx, sp[u].wy, vol, VI_, P.N, sp[u].gx, sp[u].gy, sp[u].gz);
#pragma unroll
        for (int u = 0; u < B; ++u) {
            if (k0 + u > kmax) break;
            if (sp[u].fetch) slab_step<VT, LAYOUT, OUT_DTYPE>(P, s_alpha, raw[u], sp[u], ex, darken, T, tau);
            if (col) put_texel<OUT_DTYPE>(P.out, at, T, tau);
            at += layer;
        }
    }

    // slabs behind the cube: the transmittance stays as it left the cube
    for (int k = max(kmax + 1, kmin < P.n ? kmin : P.n); k < P.n; ++k) {
        if (col) put_texel<OUT_DTYPE>(P.out, at, T, tau);
        at += layer;
    }
}

// Row layout.  A layer, border and padding included, is one run of LS
// elements, LS times the element size an odd multiple of 64 bytes: the same
// texel of two neighbouring layers lies half a 128-byte line apart, as the
// render's lookups need (the lanes of a ray group read neighbouring layers
// at one texel position in the same load instruction; a whole-line layer
// stride made those reads collide in the L1 tags, 6-8 % slower frames).  In
// a buffer aligned to 128 bytes layers -1, 1, 3, ... then start on a line
// and layers 0, 2, 4, ... half a line past one.
//
// The workgroup owns NT consecutive elements of a layer's run in every layer
// from the leading layer -1 to the trailing layer n (a copy of layer n - 1),
// one column a lane.  It scans kSlabs slabs at a time into LDS (border and
// padding lanes the fully transmitting texel, without touching the volume), in
// the stack's own type, and after one barrier its waves share out the rows of
// that set and store them, 16 bytes a lane; in the layers half a line off the
// rows are rotated by half a line, so that every store starts on a line there
// too (stores straddling lines measured at half the write rate; only the two
// half-lines at the ends of the stretch are written in part).  Two sets of LDS
// rows in turn, so that one barrier a set keeps writes and reads apart; every
// wave reaches it the same number of times.  A wave with no slab of the set
// inside the cube only stores.
//
// CDNA counts loads and stores on one counter, so a wave that waits for its
// volume loads also waits for the stores it issued before them: with no store
// between a set's loads only its first wait pays for the previous set's
// stores, of which a lane now has two.  (One element a lane and slab, each
// with its address and LDS read, were half of the kernel's VALU instructions:
// 512^3 u16 quads, 512 x 1024^2 float 712 us, now 681; bfloat16 520, now 478.
// Waves that only store, two to four of sixteen, measured no faster, 732 us.)
constexpr int kSlabs = 8;
template <int OUT_DTYPE> struct OutElem { using T = uint16_t; };
template <> struct OutElem<VI_F32> { using T = float; };
template <int OUT_DTYPE>
__device__ __forceinline__ typename OutElem<OUT_DTYPE>::T texel_of(float T, float tau)
{
    if constexpr (OUT_DTYPE == VI_F32) return T;
    else if constexpr (OUT_DTYPE == VI_BF16) return f32_to_bf16(tau);
    else return __half_as_ushort(__float2half_rn(fast_exp2(-tau)));
}

// One layer's stretch (or the part of it that lanes first, first + lanes, ...
// hold), 16 bytes a lane: `row` is its LDS row, L = k + 1 its index as stored.
// FILL: the fully transmitting texel instead of the row.
template <int OUT_DTYPE, uint32_t NT, uint32_t LANES, bool FILL = false>
__device__ __forceinline__ void store_layer(const BuildParams& P, uint32_t unit, uint32_t L, uint32_t lane,
                                            const typename OutElem<OUT_DTYPE>::T* __restrict__ row)
{
    using OT = typename OutElem<OUT_DTYPE>::T;
    constexpr uint32_t ES = sizeof(OT), CH = 16 / ES, HALF = 64 / ES;  // elements of a chunk, of half a line
    constexpr uint32_t NC = NT / CH, NI = (NC + LANES - 1) / LANES;    // chunks of a stretch, stores of a lane
    const uint32_t f0 = unit * NT, rot = (L & 1u) ? HALF : 0u;         // odd L: half a line off
    char* base = (char*)P.out + ((size_t)L * P.rlayer + f0) * ES;
    uint4 v[NI];
    uint32_t el[NI];
#pragma unroll
    for (uint32_t i = 0; i < NI; ++i) {
        // (lanes past the last chunk read the first and store nothing)
        const uint32_t c = lane + LANES * i, e = (NC % LANES == 0 || c < NC ? c * CH : 0u) + rot;
        el[i] = e < NT ? e : e - NT;
        if (!FILL) v[i] = *(const uint4*)(row + el[i]);
        else v[i].x = v[i].y = v[i].z = v[i].w = OUT_DTYPE == VI_F32 ? 0x3f800000u : OUT_DTYPE == VI_BF16 ? 0u : 0x3c003c00u;
    }
#pragma unroll
    for (uint32_t i = 0; i < NI; ++i)
        if ((NC % LANES == 0 || lane + LANES * i < NC) && f0 + el[i] < P.rlayer) *(uint4*)(base + el[i] * ES) = v[i];
}

// NW waves a workgroup, D slabs' footprints in flight a lane.
template <typename VT, int LAYOUT, int OUT_DTYPE, bool PT, int NW, int D>
__device__ __forceinline__ void build_rows(const BuildParams& P)
{
    using OT = typename OutElem<OUT_DTYPE>::T;
    constexpr uint32_t NT = NW * 64u;
    extern __shared__ __attribute__((aligned(16))) float s_alpha[];  // K alphas, the occupancy bits, two sets of rows
    uint32_t* s_bits = (uint32_t*)(s_alpha + P.K);
    const uint32_t words = stage_build_tables(P, s_alpha, s_bits);
    OT* s_x = (OT*)((char*)s_alpha + build_table_bytes(P.K, words));
    const bool use_bits = P.occ.bits != nullptr;
    const int cshift = use_bits ? P.occ.shift : 30;
    const uint32_t cnc = use_bits ? P.occ.nc : 1u;
    __syncthreads();

    uint32_t unit, one;
    if (!row_run_of(blockIdx.x, (P.rlayer + NT - 1) / NT, 1u, &unit, &one)) return;  // uniform per workgroup
    const int wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the leading layer -1 (face 0) transmits fully
    if (wave == 0) store_layer<OUT_DTYPE, NT, 64, true>(P, unit, 0u, threadIdx.x, s_x);
    const uint32_t t = threadIdx.x, f = unit * NT + t;
    const int i = (int)(f % P.rpitch) - 2, j = (int)(f / P.rpitch) - 2;
    const bool grid = f < P.rlayer && i >= 0 && i < P.res && j >= 0 && j < P.res;

    int64_t H[3], A[3];
    float ex;
    int kin, kout;
    column_setup<PT>(P, i, j, grid, H, A, &ex, &kin, &kout);
    // the wave's slabs with any midpoint in the cube: [kmin, kmax]
    const int kmin = __builtin_amdgcn_readfirstlane(wave_min(kin));
    const int kmax = __builtin_amdgcn_readfirstlane(wave_max(kout));

    const VT* __restrict__ vol = (const VT*)P.vol;
    const VolIndex VI_ = {1u, P.vsy, P.vsz};
    const bool darken = P.darken > 0.0f;
    float T = 1.0f, tau = 0.0f;  // transmittance (float stack), optical depth (2-byte stacks)
    OT* x = s_x + t;
    for (int k0 = 0; k0 < P.n; k0 += kSlabs) {
        if (k0 + kSlabs > kmin && k0 <= kmax) {  // uniform per wave
#pragma unroll 1
            for (int q = 0; q < kSlabs; q += D) {
                SlabProbe sp[D];
                bool any = false;
#pragma unroll
                for (int u = 0; u < D; ++u) {
                    sp[u] = probe_slab(P, H[0], H[1], H[2], k0 + q + u, kin, kout, s_bits, cshift, cnc);
                    any = any || sp[u].fetch;
                    for (int a = 0; a < 3; ++a) H[a] += A[a];
                }
                OT* xq = x + q * NT;
                if (__any(any)) {
                    // Bricks and quads: every lane loads, the ones with nothing
                    // to fetch the first voxel.  With loads that only some
                    // lanes issue the compiler cannot count what is
                    // outstanding, and keeps the registers of those that were
                    // not across the loop (76 VGPRs against 45: one workgroup
                    // of 1024 lanes a CU instead of two).  In a linear volume
                    // the extra lines cost more than that saves (320^3 without
                    // a map 570 us against 529 with 8 waves).
                    RawFoot<VT, LAYOUT> raw[D];
                    constexpr bool kAll = LAYOUT != VI_LAYOUT_LINEAR;
#pragma unroll
                    for (int u = 0; u < D; ++u) {
                        const bool own = sp[u].fetch;
                        if (kAll || own)
                            foot_load_g<VT, LAYOUT>(raw[u], sp[u].wx, sp[u].wy, vol, VI_, P.N, own ? sp[u].gx : 0,
                                                    own ? sp[u].gy : 0, own ? sp[u].gz : 0);
                    }
                    if (!kAll)
#pragma unroll
                        for (int u = 0; u < D; ++u) keep_foot<VT, LAYOUT>(raw[u]);
#pragma unroll
                    for (int u = 0; u < D; ++u) {
                        if (sp[u].fetch)
                            slab_step<VT, LAYOUT, OUT_DTYPE>(P, s_alpha, raw[u], sp[u], ex, darken, T, tau);
                        xq[u * NT] = texel_of<OUT_DTYPE>(T, tau);
                    }
                } else {
                    const OT v = texel_of<OUT_DTYPE>(T, tau);
#pragma unroll
                    for (int u = 0; u < D; ++u) xq[u * NT] = v;
                }
            }
        } else {
            const OT v = texel_of<OUT_DTYPE>(T, tau);
#pragma unroll
            for (int q = 0; q < kSlabs; ++q) x[q * NT] = v;
            for (int a = 0; a < 3; ++a) H[a] += kSlabs * A[a];
        }
        __syncthreads();
        // every wave stores its share of the set: whole rows, or a part of one
        const OT* rows = x == s_x + t ? s_x : s_x + kSlabs * NT;
        constexpr int W = NW > kSlabs ? NW / kSlabs : 1, RW = NW > kSlabs ? 1 : kSlabs / NW;  // waves a row, rows a wave
        static_assert(NW % kSlabs == 0 || kSlabs % NW == 0, "a wave's share of a set");
        uint32_t lane = threadIdx.x % (W * 64u);
        // (opaque: what the stores derive from it would otherwise be kept in
        // registers across the whole batch, a quarter of the budget)
        asm volatile("" : "+v"(lane));
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const int q = wave / W * RW + r, k = k0 + q;
            if (k < P.n) store_layer<OUT_DTYPE, NT, W * 64>(P, unit, (uint32_t)k + 1u, lane, rows + q * NT);
            // the trailing layer n repeats layer n - 1
            if (k == P.n - 1) store_layer<OUT_DTYPE, NT, W * 64>(P, unit, (uint32_t)k + 2u, lane, rows + q * NT);
        }
        x = x == s_x + t ? x + kSlabs * NT : s_x + t;
    }
}

template <typename VT, int LAYOUT, int OUT_DTYPE, bool PT, int NW, int D>
__global__ __launch_bounds__(NW * 64) void build_rows_kernel(BuildParams P)
{
    build_rows<VT, LAYOUT, OUT_DTYPE, PT, NW, D>(P);
}
template <typename VT, int LAYOUT, int OUT_DTYPE, bool PT, int NT, int B>
__global__ __launch_bounds__(NT) void build_tiled_kernel(BuildParams P)
{
    build_tiled<VT, LAYOUT, OUT_DTYPE, PT, NT, B>(P);
}

template <typename VT, int LAYOUT, int OUT_DTYPE, bool PT, int NW, int D>
static hipError_t launch_rows(const BuildParams& p, hipStream_t s)
{
    constexpr uint32_t NT = NW * 64u;
    // (at least one word of bits: without them word 0 says "occupied")
    const size_t lds = build_table_bytes(p.K, std::max(p.occ.words + p.occ.swords, 1u)) +
                       2 * kSlabs * NT * sizeof(typename OutElem<OUT_DTYPE>::T);
    const dim3 grid(row_run_grid((p.rlayer + NT - 1) / NT, 1u));
    hipLaunchKernelGGL((build_rows_kernel<VT, LAYOUT, OUT_DTYPE, PT, NW, D>), grid, dim3(NW * 64), lds, s, p);
    return hipGetLastError();
}

template <typename VT, int LAYOUT, int OUT_DTYPE, bool PT, int NT, int B>
static hipError_t launch_tiled(const BuildParams& p, hipStream_t s)
{
    const size_t lds = build_table_bytes(p.K, std::max(p.occ.words + p.occ.swords, 1u));
    const uint32_t runs = ((uint32_t)p.res + NT - 1) / NT;
    hipLaunchKernelGGL((build_tiled_kernel<VT, LAYOUT, OUT_DTYPE, PT, NT, B>), dim3(row_run_grid((uint32_t)p.res, runs)),
                       dim3(NT), lds, s, p);
    return hipGetLastError();
}

template <typename VT, int LAYOUT, int OUT_DTYPE, bool PT>
static hipError_t launch_build_k(const BuildParams& p, hipStream_t s)
{
    if (p.out_layout == VI_STACK_ROWS) {
        // Two workgroups of 1024 lanes fit a CU, 512 of them the chip: up to
        // about that many columns (600 K) every column is resident whatever
        // the workgroup, the time is a column's chain of waits, and smaller
        // workgroups, which spread evenly and leave registers for more loads
        // in flight, are the faster; beyond it what counts is the write
        // stream, which wants long stretches and every lane.  Measured (16
        // waves with 2 slabs in flight | 8 with 4 | 4 with 4), u16 quads, us:
        // 128^3 and 256^2 97 | 62 | 53, 192^3 and 384^2 115 | 86 | 75, 256^3
        // and 512^2 167 | 130 | 132, 320^3 and 640^2 231 | 199 | 228, 384^3
        // and 768^2 344 | 346 | 450, 512^3 and 1024^2 681 | 788 | 892.
        // Footprints of eight loads (or of two of 16 bytes) keep two slabs in
        // flight: 256^3 bricks 210 with 16 waves, 147 with 8; 512^3 754 and
        // 884.
        constexpr bool kLinear = LAYOUT == VI_LAYOUT_LINEAR, kLight = LAYOUT == VI_LAYOUT_QUAD4 && sizeof(VT) <= 2;
        // Without bits, where every slab of every column is fetched, the change comes
        // earlier (16 waves | 8: 380^3 u8 quads and 600^2 354 | 317, 445^3 half and
        // 520^2 339 | 260, 697^2 321 | 363; float quads 337^3 and 665^2 394 | 405, 384^3
        // and 768^2 574 | 716; linear u16 320^3 and 640^2 707 | 526, 337^3 and 665^2 606 |
        // 706; bricks 350^3 and 690^2 481 | 402, 360^3 and 720^2 587 | 592, 384^3 and
        // 768^2 636 | 662; with bits linear 337^3 304 | 263, 360^3 399 | 377, u16 quads
        // 384^3 344 | 346).
        if (p.rlayer > (p.occ.bits ? 600000u : LAYOUT == VI_LAYOUT_BRICK4 ? 510000u : 430000u)) {
            // The largest linear volumes of 2-byte voxels and less take four slabs
            // in flight (two | four: u16 337^3 and 665^2 606 | 632, 384^3 and 768^2 1061 |
            // 1023, 420^3 and 840^2 1257 | 1149, 512^3 and 1024^2 2163 | 1875), except
            // under a point light, whose columns spread (512^3 1984 | 1988, 420^3 1153 |
            // 1199).
            if constexpr (kLinear && sizeof(VT) <= 2 && !PT)
                if (p.rlayer > 560000u) return launch_rows<VT, LAYOUT, OUT_DTYPE, PT, 16, 4>(p, s);
            return launch_rows<VT, LAYOUT, OUT_DTYPE, PT, 16, 2>(p, s);
        }
        if constexpr (kLight) {
            if (p.rlayer <= 160000u) return launch_rows<VT, LAYOUT, OUT_DTYPE, PT, 4, 4>(p, s);
            return launch_rows<VT, LAYOUT, OUT_DTYPE, PT, 8, 4>(p, s);
        }
        return launch_rows<VT, LAYOUT, OUT_DTYPE, PT, 8, 2>(p, s);
    }
    if constexpr (OUT_DTYPE != VI_F16) {
        // A workgroup covers a stretch of one row of texels.  1024 lanes on a
        // row of 256 leave three in four idle; but beyond 256 a row in one
        // workgroup is the faster (u16 quads, 1024 | 256 lanes: 366^2 110.7 |
        // 114.8 us, 480^2 224 | 234; linear 340^2 207 | 221) unless stretches
        // of 256 fill it (512^2 363 | 347).  Large linear volumes, whose columns
        // wait for lines of their own, take four slabs in flight (without a map, before
        // their rows came as pairs | two slabs | four: 512^3 u8 and 1024^2 bfloat16 2577 |
        // 2765 | 1836, float 3053 | 3090 | 2505; 450^3 and 900^2 1395 | 1427 | 1256; 384^3
        // and 768^2 980 | 838 | 931).
        if constexpr (LAYOUT == VI_LAYOUT_LINEAR)
            if (p.res > 800) return launch_tiled<VT, LAYOUT, OUT_DTYPE, PT, 1024, 4>(p, s);
        if (p.res > 512 || (p.res > 256 && p.res % 256 != 0))
            return launch_tiled<VT, LAYOUT, OUT_DTYPE, PT, 1024, 2>(p, s);
        return launch_tiled<VT, LAYOUT, OUT_DTYPE, PT, 256, 2>(p, s);
    }
    return hipErrorInvalidValue;
}

template <typename VT, int LAYOUT>
static hipError_t launch_build_t(const BuildParams& p, hipStream_t s)
{
    if (p.out_dtype == VI_F32)
        return p.point ? launch_build_k<VT, LAYOUT, VI_F32, true>(p, s) : launch_build_k<VT, LAYOUT, VI_F32, false>(p, s);
    if (p.out_dtype == VI_BF16)
        return p.point ? launch_build_k<VT, LAYOUT, VI_BF16, true>(p, s)
                       : launch_build_k<VT, LAYOUT, VI_BF16, false>(p, s);
    return p.point ? launch_build_k<VT, LAYOUT, VI_F16, true>(p, s) : launch_build_k<VT, LAYOUT, VI_F16, false>(p, s);
}

template <typename VT>
static hipError_t launch_build_l(const BuildParams& p, hipStream_t s)
{
    if (p.vol_layout == VI_LAYOUT_QUAD4) return launch_build_t<VT, VI_LAYOUT_QUAD4>(p, s);
    return p.vol_layout == VI_LAYOUT_BRICK4 ? launch_build_t<VT, VI_LAYOUT_BRICK4>(p, s)
                                            : launch_build_t<VT, VI_LAYOUT_LINEAR>(p, s);
}

hipError_t launch_build(const BuildParams& p, hipStream_t s)
{
    switch (p.vol_dtype) {
    case VI_U8: return launch_build_l<uint8_t>(p, s);
    case VI_U16: return launch_build_l<uint16_t>(p, s);
    case VI_F16: return launch_build_l<__half>(p, s);
    default: return launch_build_l<float>(p, s);
    }
}

}  // namespace vi
