// Linear layers of a decode step of 3 to 8 rows on the gfx950 matrix cores: wide models, and rows that are selected on the device (other steps of narrow models are
// one launch, flow_kernels.hip).
//
// The skinny kernels of mfma_kernels.hip fill a 32-column operand with rows (8 rows use a quarter of it, hi and lo twice), split the work of a layer
// over K and leave partial sums, and need packed, normalised activations: a launch per layer for the residual and the norm, and for wide models two
// more that finish the sums. Up to 8 rows the 16 columns of v_mfma_f32_16x16x32_bf16 hold everything: column m is the bf16 hi part of row m, column
// m + 8 its lo part (value = hi + lo, see split_hi_lo), so ONE instruction multiplies both against a weight operand, and the wavefronts' activation
// operands for the whole reduction dimension fit registers:
//   * 8 wavefronts of a workgroup split K (at most 16 steps of 32 each); each builds its operands from the fp32 rows at the start (times the norm's
//     gain; the sum of squares falls out on the way, and 1/rms is applied to the sums: W.(g*x/rms) = W.(g*x)/rms) and keeps them.
//   * A unit of work is 8 pairs of consecutive weight rows (of gate and of up rows). The weights of a unit sit in one register ring; entry s is refilled
//     with the next unit's step s right after the instruction that read it, so a whole unit is in flight ahead of the arithmetic.
//   * The partial sums of the 8 wavefronts meet in LDS (one barrier per unit, two buffers); one wavefront adds them in wavefront order, hi and lo
//     columns last, and runs the epilogue: rotation and cache append, SwiGLU, or the residual update.
// Launches a layer: qkv, attention, output projection, gate/up, down: no packing, no partials, no finishing. Weights are the tiles of repack_kernel; a
// 16 x 32 operand is half of two consecutive 32 x 16 ones.
// What bounds it: wide models the weight stream (7B-class gate/up 271 MB in 50 us = 5.4 TB/s), small ones launches and latency (0.5B-class layer at 7
// rows: q|k|v 5.7, output projection 4.2, gate/up 7.9, down 7.2 us, where the profiler shows 4.2 us for an empty kernel). Steps against the skinny
// kernels: 0.5B-class at 3 / 7 (paged) / 8 rows 950 / 1050 / 1040 -> 820 / 943 / 930 us, 7B-class 8 rows 3.97 -> 3.77 ms, selected on the device 4.11 -> 3.65 ms.
#include "mfma_common.h"
#include <algorithm>
#include <type_traits>

namespace tr {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int FEW_WAVES = 8;
constexpr int FEW_ROWS = FEW_MAX_ROWS;

struct FewArgs {
    const uint4 *Wt;    // tiled weights [tile][KS][64]
    int KS, per;        // K / 16; steps of 32 per wavefront
    int pairs;          // pairs of consecutive weight rows (of gate and of up rows) in all
    int gran, share, extra;   // pairs that stay together; such groups per workgroup, and workgroups with one more
    int R;              // rows
    const int *live;    // device-side row count or NULL
};

// Addresses are a uniform base plus a 32-bit offset per lane: one vector register per load whatever the step.
// (The empty assembly keeps the compiler from folding the base into 64-bit vector addresses.)
template <typename T> __device__ __forceinline__ T few_load(const void *base, uint32_t uniform, uint32_t off)
{
    const char *p = static_cast<const char *>(base) + uniform;
    asm("" : "+s"(p));
    return *reinterpret_cast<const T *>(p + off);
}

// The rows of a workgroup: an even share of all pairs, neighbouring shares on one XCD, walked in units of 8 pairs (the 16 rows of a matrix operand).
struct FewShare {
    int lo, hi;   // pairs lo .. hi - 1
    __device__ __forceinline__ explicit FewShare(const FewArgs &a)
    {
        const int per = gridDim.x >> 3, rem = gridDim.x & 7, xcd = blockIdx.x & 7, w = xcd * per + min(xcd, rem) + (blockIdx.x >> 3);
        lo = (w * a.share + min(w, a.extra)) * a.gran;
        hi = min(a.pairs, lo + (a.share + (w < a.extra)) * a.gran);
    }
    __device__ __forceinline__ int end(int p0) const { return min(p0 + 8, hi); }
};

// Byte offset of this lane's 16 bytes in the tiles: lane L takes row L % 16 of the unit p0 .. p1 - 1 (rows past it repeat the last one), columns
// 8 (L / 16) .. + 7 of a step of 32 columns (two k-steps of a tile, 2048 bytes). tile_step: tiles from one 32-row block to the next (2: gate, up alternate).
// A matrix is under 4 GiB.
__device__ __forceinline__ uint32_t few_weight_offset(int lane, int p0, int p1, int KS, int tile_step)
{
    const int row = min(2 * p0 + (lane & 15), 2 * p1 - 1);
    return (uint32_t)((row >> 5) * tile_step) * KS * 1024 + ((lane >> 5) * 64 + 32 * ((lane >> 4) & 1) + (row & 31)) * 16;
}

// Activations to an operand: a lane brings 4 values of its row, the lanes of columns 0-7 the first four of the 8 columns a lane multiplies and those of
// columns 8-15 the last four; each splits its own and hands its partner (8 lanes on) the half that is needed there: hi parts end up in columns 0-7.
__device__ __forceinline__ uint4 few_operand(const float (&v)[4], bool lo_col)
{
    const f32x2 x0 = {v[0], v[1]}, x1 = {v[2], v[3]};
    const uint32_t h0 = __builtin_bit_cast(uint32_t, __builtin_convertvector(x0, bf16x2)), h1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(x1, bf16x2));
    const f32x2 r0 = {v[0] - __uint_as_float(h0 << 16), v[1] - __uint_as_float(h0 & 0xffff0000u)};
    const f32x2 r1 = {v[2] - __uint_as_float(h1 << 16), v[3] - __uint_as_float(h1 & 0xffff0000u)};
    const uint32_t l0 = __builtin_bit_cast(uint32_t, __builtin_convertvector(r0, bf16x2)), l1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(r1, bf16x2));
    auto partner = [](uint32_t u) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)u, 0x128, 0xf, 0xf, true); };   // row_ror:8
    const uint32_t p0 = partner(lo_col ? h0 : l0), p1 = partner(lo_col ? h1 : l1);
    return lo_col ? make_uint4(p0, p1, l0, l1) : make_uint4(h0, h1, p0, p1);
}

// ---- activations: fp32 rows, times the gain of an RMSNorm (NORM: 1/rms is left to the epilogue), or as they are
template <bool NORM>
struct FewRows {
    const float *x;
    const bf16_t *gain;
    float eps;
};

// ---- epilogues: features f, f + 1 of row m. rs: 1/rms of the row (1 without a norm). Row: what the row's place needs, loaded first of all;
// Pre: what the features need, loaded ahead of the unit's arithmetic.

template <typename KT>
struct FewQkv {
    static constexpr bool pairs = false;
    QkvOut<KT> out;
    const int *slot, *pos, *ptab;
    int page, maxp;
    struct Row { int p, unit, up; };
    struct Pre { float a, b; float2 cs; };
    __device__ __forceinline__ Row row(int m) const
    {
        Row r{pos[m], slot[m], 0};
        r.up = r.p;
        if (page) { r.unit = ptab[(size_t)r.unit * maxp + r.p / page]; r.up = r.p % page; }
        return r;
    }
    // features f, f + 1 are the rotary pair (j, j + dh/2) of head hh (see repack_kernel)
    __device__ __forceinline__ void place(int f, int &hh, int &j) const
    {
        const int tph = out.dh >> 5, t = f >> 5;
        hh = t / tph; j = (t % tph) * 16 + ((f & 31) >> 1);
    }
    __device__ __forceinline__ Pre pre(const Row &r, int, int f) const
    {
        const int half = out.dh >> 1;
        int hh, j;
        place(f, hh, j);
        return Pre{out.bias[hh * out.dh + j], out.bias[hh * out.dh + half + j], out.rope[(size_t)r.p * half + j]};
    }
    __device__ __forceinline__ void store(const Row &r, const Pre &pr, int m, int f, float c0, float c1, float rs) const
    {
        const int half = out.dh >> 1;
        int hh, j;
        place(f, hh, j);
        const float a = fmaf(c0, rs, pr.a), b = fmaf(c1, rs, pr.b);
        float lo = a, hi = b;
        if (hh < out.Hq + out.Hkv) { lo = a * pr.cs.x - b * pr.cs.y; hi = b * pr.cs.x + a * pr.cs.y; }
        if (hh < out.Hq) {
            float *dst = out.q + (size_t)m * out.qw + hh * out.dh + j;
            dst[0] = lo; dst[half] = hi;
            return;
        }
        const bool key = hh < out.Hq + out.Hkv;
        const int head = key ? hh - out.Hq : hh - out.Hq - out.Hkv;
        if (key || out.vts == 0) {
            KT *dst = (key ? out.kc : out.vc) + (((size_t)r.unit * out.Hkv + head) * out.unit_len + r.up) * out.dh + j;
            kv_store1(dst, lo);
            kv_store1(dst + half, hi);
        } else {
            KT *dst = out.vc + ((((size_t)r.unit * out.Hkv + head) * (out.vts >> 5) + (r.up >> 5)) * out.dh + j) * 32 + (r.up & 31);
            kv_store1(dst, lo);
            kv_store1(dst + half * 32, hi);
        }
    }
};

// h = silu(gate) * up as the down projection's operand [F/32 steps][64 lanes][8 bf16] (rows past the batch give zeros)
struct FewSwiglu {
    static constexpr bool pairs = true;
    uint32_t *hpack;
    struct Row {};
    struct Pre {};
    __device__ __forceinline__ Row row(int) const { return {}; }
    __device__ __forceinline__ Pre pre(const Row &, int, int) const { return {}; }
    __device__ __forceinline__ void store2(int m, int f, float g0, float g1, float u0, float u1, float rs) const
    {
        const float t0 = g0 * rs, t1 = g1 * rs;
        const float h0 = t0 * __frcp_rn(1.0f + __expf(-t0)) * (u0 * rs), h1 = t1 * __frcp_rn(1.0f + __expf(-t1)) * (u1 * rs);
        const f32x2 v = {h0, h1};
        const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
        const f32x2 r = {h0 - __uint_as_float(hi << 16), h1 - __uint_as_float(hi & 0xffff0000u)};
        uint32_t *dst = hpack + ((size_t)(f >> 5) * 64 + 16 * ((f >> 3) & 3) + m) * 4 + ((f >> 1) & 3);
        dst[0] = hi;
        dst[4 * FEW_ROWS] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
    }
};

struct FewResidual {
    static constexpr bool pairs = false;
    float *x;
    int d;
    struct Row {};
    struct Pre { float2 old; };
    __device__ __forceinline__ Row row(int) const { return {}; }
    __device__ __forceinline__ Pre pre(const Row &, int m, int f) const { return Pre{*reinterpret_cast<const float2 *>(x + (size_t)m * d + f)}; }
    __device__ __forceinline__ void store(const Row &, const Pre &pr, int m, int f, float c0, float c1, float) const
    {
        *reinterpret_cast<float2 *>(x + (size_t)m * d + f) = make_float2(pr.old.x + c0, pr.old.y + c1);
    }
};

// The sums of a unit: LDS [wavefront][block][lane], added in wavefront order, then hi + lo. Lanes with bit 3 clear hold activation row lane % 8, the unit's
// pairs 2 (lane / 16) and + 1.
template <int NB>
__device__ __forceinline__ void few_sum(const f32x4 (*red)[NB][64], int lane, f32x4 (&v)[NB])
{
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        v[nb] = red[0][nb][lane];
#pragma unroll
        for (int w = 1; w < FEW_WAVES; ++w) {
            v[nb] += red[w][nb][lane];
            if (w % 3 == 0) __builtin_amdgcn_sched_barrier(0);   // a few at a time: the registers hold the next unit's weights
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) v[nb][e] += __shfl_xor(v[nb][e], 8, 64);
    }
}
// a pair's first feature: rows of a tile lie in the order of tile_feature, which keeps pairs together
__device__ __forceinline__ int few_feature(int pair) { return (pair >> 4) * 32 + tile_feature(2 * (pair & 15)); }

// NS: steps of 32 a wavefront keeps (K <= 256 NS); gate/up: the unit's rows of both matrices
template <int NS, int OCC, bool NORM, class Epi>
__global__ __launch_bounds__(64 * FEW_WAVES, OCC) void few_kernel(FewArgs a, FewRows<NORM> in, Epi epi)
{
    constexpr int NB = Epi::pairs ? 2 : 1;
    __shared__ f32x4 red[2][FEW_WAVES][NB][64];
    __shared__ float s_ss[FEW_WAVES][FEW_ROWS];
    const int R = a.live ? min(a.R, *a.live) : a.R;
    const FewShare share(a);
    if (R == 0 || share.lo == share.hi) return;   // uniform over the workgroup
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int K = a.KS * 16, n32 = a.KS / 2, s0 = min(wave * a.per, n32), ns = min(n32, s0 + a.per) - s0;
    uint4 w[NB][NS];
    auto load = [&](uint32_t off, int s) {   // steps past the wavefront's share repeat its last one (their activations are zero)
        const uint32_t at = min(s0 + min(s, max(ns - 1, 0)), n32 - 1) * 2048;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) w[nb][s] = few_load<uint4>(a.Wt, nb * a.KS * 1024 + at, off);
    };
    const int m = lane & 7, o = lane >> 4, mr = min(m, R - 1);
    const typename Epi::Row row = epi.row(mr);
    int p0 = share.lo;
    uint32_t off = few_weight_offset(lane, p0, share.end(p0), a.KS, NB);
    // activations: lane L takes row L % 8, columns 8 (L / 16) + 4 (L / 8 % 2) .. + 3 of each step, all requested before the weights (loads return in
    // order, and the rows come from the L2)
    const bool lo_col = lane & 8;
    const uint32_t col = o * 8 + (lo_col ? 4 : 0), x_off = (mr * K + col) * 4, g_off = col * 2;
    bf16x8 b[NS];
    float4 xv[NS];
    uint2 g[NS];
    float ss = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int k = min(s0 + s, n32 - 1) * 32;
        xv[s] = few_load<float4>(in.x, k * 4, x_off);
        if (NORM) g[s] = few_load<uint2>(in.gain, k * 2, g_off);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) load(off, s);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const bool use = m < R && s < ns;
        float v[4] = {xv[s].x, xv[s].y, xv[s].z, xv[s].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = use ? v[e] : 0.f;
        if (NORM) {
            const float gv[4] = {__uint_as_float(g[s].x << 16), __uint_as_float(g[s].x & 0xffff0000u), __uint_as_float(g[s].y << 16), __uint_as_float(g[s].y & 0xffff0000u)};
#pragma unroll
            for (int e = 0; e < 4; ++e) { ss = fmaf(v[e], v[e], ss); v[e] *= gv[e]; }
        }
        uint4 bs = few_operand(v, lo_col);
        asm("" : "+v"(bs.x), "+v"(bs.y), "+v"(bs.z), "+v"(bs.w));   // converted here, not where it is first used
        b[s] = __builtin_bit_cast(bf16x8, bs);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (NORM) {
        ss += __shfl_xor(ss, 8, 64);
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (lane < FEW_ROWS) s_ss[wave][lane] = ss;   // read after the first unit's barrier
    }
    float rs = 1.0f;
    bool have_rs = !NORM;
    // one unit; `more`: another follows, whose weights are requested as the ring empties
    auto unit = [&](int i, int p1, auto more) {
        if (more) off = few_weight_offset(lane, p1, share.end(p1), a.KS, NB);
        int f[2];
        typename Epi::Pre pre[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            f[e] = few_feature(min(p0 + 2 * o + e, p1 - 1));
            pre[e] = epi.pre(row, mr, f[e]);
        }
        f32x4 acc[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[nb][s]), b[s], acc[nb], 0, 0, 0);
            if (more) {
                load(off, s);
                __builtin_amdgcn_sched_barrier(0);   // the refill right behind the instructions that read the entry
            }
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) red[i & 1][wave][nb][lane] = acc[nb];
        __syncthreads();
        if (wave != (i & (FEW_WAVES - 1))) return;
        if (!have_rs) {
            float t = 0.f;
#pragma unroll
            for (int q = 0; q < FEW_WAVES; ++q) t += s_ss[q][m];
            rs = 1.0f / sqrtf(t / (float)K + in.eps);
            have_rs = true;
        }
        f32x4 v[NB];
        few_sum<NB>(red[i & 1], lane, v);
        if (lo_col || m >= (Epi::pairs ? FEW_ROWS : R)) return;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (p0 + 2 * o + e >= p1) continue;
            if constexpr (Epi::pairs) epi.store2(m, f[e], v[0][2 * e], v[0][2 * e + 1], v[1][2 * e], v[1][2 * e + 1], rs);
            else epi.store(row, pre[e], m, f[e], v[0][2 * e], v[0][2 * e + 1], rs);
        }
    };
    int i = 0;
#pragma unroll 1
    for (int p1 = share.end(p0); p1 < share.hi; p1 = share.end(p0)) {
        unit(i++, p1, std::true_type{});
        p0 = p1;
    }
    unit(i, share.hi, std::false_type{});
}

// The same for a long reduction dimension (the FFN output): the activations are already operands in memory ([step][64 lanes][16 bytes], FewSwiglu) and
// stream along with the weights; one block of 16 weight rows per workgroup, D steps in flight per wavefront.
template <int D, class Epi>
__global__ __launch_bounds__(64 * FEW_WAVES, 2) void few_long_kernel(FewArgs a, const uint4 *act, Epi epi)
{
    __shared__ f32x4 red[FEW_WAVES][1][64];
    const int R = a.live ? min(a.R, *a.live) : a.R;
    const FewShare share(a);   // one unit: the launcher sees to it
    if (R == 0 || share.lo == share.hi) return;   // uniform over the workgroup
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int m = lane & 7, o = lane >> 4;
    int f[2];
    typename Epi::Pre pre[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        f[e] = few_feature(min(share.lo + 2 * o + e, share.hi - 1));
        pre[e] = epi.pre({}, min(m, R - 1), f[e]);
    }
    // wavefront w takes the steps w, w + 8, ...: neighbouring wavefronts read neighbouring memory
    const int n32 = a.KS / 2, ns = n32 > wave ? (n32 - wave + FEW_WAVES - 1) / FEW_WAVES : 0;
    uint4 w[D], x[D];
    const uint32_t w_off = few_weight_offset(lane, share.lo, share.hi, a.KS, 1), x_off = lane * 16;
    const auto W = buffer_of(a.Wt, (uint32_t)((2 * a.pairs + 31) / 32) * a.KS * 1024), X = buffer_of(act, n32 * 1024);
    auto load = [&](int i, int s) {   // past the wavefront's last step: beyond the buffers, which costs no memory access (and counts like any load)
        const bool past = s >= ns;
        const int step = past ? 0 : wave + FEW_WAVES * s;
        w[i] = buffer_load16(W, past ? BUFFER_NOWHERE : w_off, step * 2048);
        x[i] = buffer_load16(X, past ? BUFFER_NOWHERE : x_off, step * 1024);
    };
#pragma unroll
    for (int i = 0; i < D; ++i) load(i, i);
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
    auto product = [&](int i) {
        f32x4 &acc = i & 1 ? acc1 : acc0;
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[i]), __builtin_bit_cast(bf16x8, x[i]), acc, 0, 0, 0);
    };
    int s = 0;
#pragma unroll 1
    for (; s + D < ns; s += D) {
#pragma unroll
        for (int i = 0; i < D; ++i) {
            product(i);
            load(i, s + D + i);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int i = 0; i < D; ++i) product(i);   // what lies past the last step is zero
    red[wave][0][lane] = acc0 + acc1;
    __syncthreads();
    if (wave != 0) return;
    f32x4 v[1];
    few_sum<1>(red, lane, v);
    if ((lane & 8) || m >= R) return;
#pragma unroll
    for (int e = 0; e < 2; ++e)
        if (share.lo + 2 * o + e < share.hi) epi.store({}, pre[e], m, f[e], v[0][2 * e], v[0][2 * e + 1], 1.0f);
}

// ------------------------------------------------------------------ launches

bool few_supported(const Dims &D)
{
    return D.d % 32 == 0 && D.F % 32 == 0 && D.d <= 4096 && D.qw <= 4096 && D.qw % 32 == 0 && (size_t)D.F * D.d < (size_t)1 << 30;
}

// workgroups, and their shares in groups of `gran` pairs: one workgroup per compute unit at most (with 512 the 0.5B-class gate/up takes 10.0 us, 8.6 with 256).
// Groups of 4 pairs are the 128 bytes of a cache line in every half tile: smaller ones spread the rows more evenly but fetch lines twice (7B-class
// gate/up by single pairs 58 us, by 4 pairs 50 us, by 8 pairs 50 us).
static int few_grid(FewArgs &a, int gran)
{
    const int groups = (a.pairs + gran - 1) / gran, grid = std::min(groups, 256);
    a.gran = gran; a.share = groups / grid; a.extra = groups % grid;
    return grid;
}

template <bool NORM, class Epi>
static void launch_few(hipStream_t s, FewArgs a, const FewRows<NORM> &in, const Epi &epi)
{
    a.per = (a.KS / 2 + FEW_WAVES - 1) / FEW_WAVES;
    const int grid = few_grid(a, 4);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * FEW_WAVES), 0, s, a, in, epi); };
    if (a.per <= 4) go(few_kernel<4, 4, NORM, Epi>);
    else if (a.per <= 8) go(few_kernel<8, 2, NORM, Epi>);
    else if (a.per <= 14) go(few_kernel<14, 2, NORM, Epi>);
    else go(few_kernel<16, 2, NORM, Epi>);
}

static FewArgs few_args(const void *Wt, int K, int pairs, int R, const int *live)
{
    FewArgs a{};
    a.Wt = (const uint4 *)Wt; a.KS = K / 16; a.pairs = pairs; a.R = R; a.live = live;
    return a;
}

void launch_few_qkv(hipStream_t s, int kdt, const Dims &D, const void *Wt, const float *x, const void *gain, const float *bias, Rows rows, const float2 *rope,
                    float *q, void *kc, void *vc)
{
    auto go = [&](auto kt) {
        using KT = decltype(kt);
        const FewQkv<KT> e{{bias, rope, q, (KT *)kc, (KT *)vc, D.Hq, D.Hkv, D.dh, kv_unit_len(D), D.qw, kv_unit_vts(D)}, rows.slot, rows.pos, D.ptab, D.page, D.maxp};
        launch_few(s, few_args(Wt, D.d, D.qw / 2 + D.kvw, rows.n, rows.live), FewRows<true>{x, (const bf16_t *)gain, D.eps}, e);
    };
    if (kdt == DT_F32) go(float{}); else go(bf16_t{});
}

void launch_few_oproj(hipStream_t s, const Dims &D, const void *Wt, const float *att, int R, float *x, const int *live)
{
    launch_few(s, few_args(Wt, D.qw, D.d / 2, R, live), FewRows<false>{att, nullptr, 0.f}, FewResidual{x, D.d});
}

void launch_few_swiglu(hipStream_t s, const Dims &D, const void *Wt, const float *x, const void *gain, int R, void *hpack, const int *live)
{
    launch_few(s, few_args(Wt, D.d, D.F / 2, R, live), FewRows<true>{x, (const bf16_t *)gain, D.eps}, FewSwiglu{(uint32_t *)hpack});
}

void launch_few_down(hipStream_t s, const Dims &D, const void *Wt, const void *hpack, int R, float *x, const int *live)
{
    // groups of 2 pairs (0.5B-class, 448 pairs: 224 workgroups 7.2 us, 112 of 4 pairs 7.9 us, 56 of 8 pairs 9.5 us); at most 8 pairs each, d <= 4096.
    // 20 steps in flight: the 0.5B-class wavefront's whole share, 7.9 us (7.1 with the smaller groups) against 8.2 with 8; 7B-class 32.9 against 34.0 us
    FewArgs a = few_args(Wt, D.F, D.d / 2, R, live);
    const int grid = few_grid(a, 2);
    hipLaunchKernelGGL((few_long_kernel<20, FewResidual>), dim3(grid), dim3(64 * FEW_WAVES), 0, s, a, (const uint4 *)hpack, FewResidual{x, D.d});
}

}  // namespace tr
