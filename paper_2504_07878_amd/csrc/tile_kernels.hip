// Linear layers over many rows (prompts, catch-up segments, large tails) on the gfx950 matrix cores.
//
// Y[M][N] = A[M][K] . W[N][K]^T with M in the hundreds to thousands: unlike the skinny products of mfma_kernels.hip, which are
// bound by streaming W once, these are bound by the matrix pipes, so both operands are staged through LDS and reused:
//   * A workgroup of 4 wavefronts (2 along the rows x 2 along the features) computes a block of 2*WM*32 rows x 2*WN*32 features; a
//     wavefront holds WM x WN accumulators of 32 x 32. Per k-step of 16 it reads WN weight operands and 2*WM activation operands (hi
//     and lo, see split_hi_lo) from LDS for 2*WM*WN matrix instructions: with 2 x 4 accumulators the four wavefronts read 32 KiB in 256
//     clocks of LDS time against 512 clocks of matrix time.
//   * Both operands already lie in memory in operand order (1 KiB per 32 x 16 operand, see repack_kernel and store_packed), so a stage
//     is copied to LDS by direct loads (no registers, no conversion, lane i's 16 bytes at byte 16 i) and read back without bank conflicts.
//   * ST stages (k-steps) form a ring filled ahead; one barrier per step; a step's operands are read from LDS into registers one step ahead. Two or
//     three workgroups share a compute unit: while one waits at its barrier or is in its epilogue, the matrix instructions of another run.
//   * A wavefront accumulates its whole K range itself, so there is no cross-wavefront sum: the accumulator registers of a lane are runs of
//     8 consecutive features of one row (tile_feature), which is what the epilogues consume.
//   * Blocks are dealt to the XCDs in contiguous pieces of an order that walks groups of gm row blocks x features, so that the workgroups
//     of an XCD share operands in its L2.
// What bounds it: the chip's power at this mix of matrix instructions and operand traffic. 1151 x 37888 x 3584 (hi and lo products, 0.63 TFLOP of bf16
// work) takes 515 to 525 us = 1.2 PFLOP/s at 1.6 GHz with the matrix pipes 72 % busy; a bf16 library product of the same work 569 us. Launches of few
// rounds of blocks leave the pipes idle at their ends: 8192 x 896 x 896 42 us, 24 % busy.
#include "mfma_common.h"
#include <algorithm>
#include <type_traits>

namespace tr {

struct TileArgs {
    const uint4 *Wt;      // tiled weights [tile][KS][64]
    const uint4 *pack;    // packed activations [64-row group][KS][4][64]
    int KS, kwg, ksw;     // K / 16; k-steps per workgroup (gridDim.y of them along K); k-steps per split of the sum
    int spw;              // splits per workgroup (TilePartial, TileResidualParts)
    int n_tiles, groups;  // 32-feature tiles, 64-row groups
    int M;
    int n_mblk, n_nblk;   // row blocks, feature blocks
    int gm;               // row blocks per group of the walk
    int items, per_xcd;   // n_mblk * n_nblk, and its eighth rounded up
};

// one wavefront: 64 x 16 bytes from base + lane's offset to LDS bytes lds .. lds + 1023. The compiler writes M0, which must be one wait state before an LDS
// load uses it.
__device__ __forceinline__ void load_to_lds(uint32_t lds, uint32_t lane_off, const char *base)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"{m0}"(lds), "v"(lane_off), "s"(base) : "memory");
}
// own loads but the youngest N have landed, own LDS reads are done, then the workgroup's barrier. (Built-ins rather than assembly for the wait: the
// compiler then knows that no LDS read is outstanding and adds no waits of its own for the operands read a step earlier.)
template <int N> __device__ __forceinline__ void wait_and_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));   // vmcnt N, expcnt 7 (no wait), lgkmcnt 0
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ------------------------------------------------------------------ epilogues
// init(): once per workgroup, m[mi] = this lane's row of accumulator row mi. start(): the value the split sums are added to, 8 consecutive features
// from n0 on of row mi. store(): the finished value of the same 8 features (tile t, features i0 .. i0 + 7 of it). pair(): in place of store for
// gate/up tiles. fini(): after the last block (lds: the kernel's whole LDS buffer, free by then).

struct TilePartial {   // split-K partial sums: part[split][m][n]
    static constexpr bool pairs = false;
    float *part;
    int N, M;
    template <int WM> struct State { __device__ void init(const TilePartial &, const int (&)[WM], int) {} };
    __device__ __forceinline__ void store(int split, int m, int t, int i0, const float (&v)[8]) const
    {
        const int n = t * 32 + i0;
        if (m < M && n < N) {
            float *dst = part + ((size_t)split * M + m) * N + n;
            *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
            *reinterpret_cast<float4 *>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
        }
    }
};

template <typename KT>
struct TileQkv {       // bias, rotary embedding, q out, cache append
    static constexpr bool pairs = false;
    QkvOut<KT> out;
    const int *slot, *pos, *ptab;
    int M, n_tiles, page, maxp;
    template <int WM> struct State {
        int p[WM], unit[WM], up[WM];
        __device__ void init(const TileQkv &e, const int (&m)[WM], int)
        {
#pragma unroll
            for (int mi = 0; mi < WM; ++mi) {
                const int r = min(m[mi], e.M - 1);
                p[mi] = e.pos[r]; unit[mi] = e.slot[r]; up[mi] = p[mi];
                if (e.page) { unit[mi] = e.ptab[(size_t)unit[mi] * e.maxp + p[mi] / e.page]; up[mi] = p[mi] % e.page; }
            }
        }
    };
    template <int WM> __device__ __forceinline__ void start(State<WM> &, int, int, int n0, float (&v)[8]) const   // the bias, in the tile's order (pairs (j, j + dh/2))
    {
        const int t = min(n0 >> 5, n_tiles - 1), i0 = n0 & 31, tph = out.dh >> 5, half = out.dh >> 1, hh = t / tph, j0 = (t % tph) * 16 + (i0 >> 1);
        const float4 ba = *reinterpret_cast<const float4 *>(out.bias + hh * out.dh + j0), bb = *reinterpret_cast<const float4 *>(out.bias + hh * out.dh + half + j0);
        v[0] = ba.x; v[1] = bb.x; v[2] = ba.y; v[3] = bb.y; v[4] = ba.z; v[5] = bb.z; v[6] = ba.w; v[7] = bb.w;
    }
    template <int WM> __device__ __forceinline__ void store(State<WM> &st, int mi, int m, int t, int i0, const float (&v)[8]) const
    {
        if (m < M && t < n_tiles) qkv_emit<true>(out, t, m, i0, v, st.p[mi], st.unit[mi], st.up[mi]);
    }
};

struct TileSwiglu {    // tiles alternate gate, up; h = silu(gate) * up, written as packed activations of the down projection
    static constexpr bool pairs = true;
    const float *rstd; // rstd[row * SS_STRIDE]: factor on gate and up (deferred RMSNorm), or NULL
    uint4 *hpack;      // [group][F/16][4][64]
    int M, F;
    template <int WM> struct State {
        float rs[WM];
        __device__ void init(const TileSwiglu &e, const int (&m)[WM], int)
        {
#pragma unroll
            for (int mi = 0; mi < WM; ++mi) rs[mi] = e.rstd ? e.rstd[(size_t)min(m[mi], e.M - 1) * SS_STRIDE] : 1.0f;
        }
    };
    template <int WM> __device__ __forceinline__ void start(State<WM> &, int, int, int, float (&v)[8]) const
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.f;
    }
    template <int WM> __device__ __forceinline__ void pair(State<WM> &st, int mi, int m, int t, int i0, const float (&g)[8], const float (&u)[8]) const
    {
        const float r = st.rs[mi];
        float h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float gt = g[e] * r;
            h[e] = gt * __frcp_rn(1.0f + __expf(-gt)) * (u[e] * r);
        }
        const int f0 = (t >> 1) * 32 + i0;
        if (m < M && f0 < F) store_packed(hpack + (size_t)(m >> 6) * (F / 16) * 4 * 64, 4, m & 63, f0 >> 3, h);
    }
};

// x += tile; with `pack` the input of the next linear layer is written as x * gain (hi/lo split, no 1/rms) and the rows' sums of squares over each
// tile of 32 features as sumsq[row][tile] (a tile's four bands of 8 features, each summed in order, added pairwise): the consumer applies 1/rms.
struct TileResidual {
    static constexpr bool pairs = false;
    float *x;              // residual stream [M][d], updated in place
    const bf16_t *gain;    // gain of the norm that follows
    uint4 *pack;           // packed activations of the next linear layer [group][d/16][4][64], or NULL
    float *sumsq;
    int M, d;
    template <int WM> struct State {
        float first;       // sum of squares of the tile's lower band of this lane
        __device__ void init(const TileResidual &, const int (&)[WM], int) {}
    };
    template <int WM> __device__ __forceinline__ void start(State<WM> &, int, int m, int n0, float (&v)[8]) const
    {
        const float *xr = x + (size_t)min(m, M - 1) * d + min(n0, d - 8);
        const float4 p = *reinterpret_cast<const float4 *>(xr), q = *reinterpret_cast<const float4 *>(xr + 4);
        v[0] = p.x; v[1] = p.y; v[2] = p.z; v[3] = p.w; v[4] = q.x; v[5] = q.y; v[6] = q.z; v[7] = q.w;
    }
    template <int WM> __device__ __forceinline__ void store(State<WM> &st, int, int m, int t, int i0, const float (&xn)[8]) const
    {
        const int n0 = t * 32 + i0;
        if (pack) {   // the lanes l and l + 32 hold the same row
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) ss = fmaf(xn[e], xn[e], ss);
            if (n0 >= d) ss = 0.f;
            if (i0 < 16) st.first = ss;
            else {
                const float a = st.first + __shfl_xor(st.first, 32, 64), b = ss + __shfl_xor(ss, 32, 64);
                if (i0 == 16 && m < M && t * 32 < d) sumsq[(size_t)m * SS_STRIDE + t] = a + b;
            }
        }
        if (m >= M || n0 >= d) return;
        float *xr = x + (size_t)m * d + n0;
        *reinterpret_cast<float4 *>(xr) = make_float4(xn[0], xn[1], xn[2], xn[3]);
        *reinterpret_cast<float4 *>(xr + 4) = make_float4(xn[4], xn[5], xn[6], xn[7]);
        if (pack) {
            const uint4 gbits = *reinterpret_cast<const uint4 *>(gain + n0);
            const uint32_t gw[4] = {gbits.x, gbits.y, gbits.z, gbits.w};
            float gx[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) gx[e] = xn[e] * __uint_as_float((e & 1) ? (gw[e >> 1] & 0xffff0000u) : (gw[e >> 1] << 16));
            store_packed(pack + (size_t)(m >> 6) * (d / 16) * 4 * 64, 4, m & 63, n0 >> 3, gx);
        }
    }
};

// The same for a product whose K several workgroups share: those of the first part add their splits to x, the others leave theirs apart for the consumer
// to add in order (x as the first part left it, then the partials), which gives the sums of TileResidual.
struct TileResidualParts : TileResidual {
    TilePartial rest;      // splits from the second part on
};

// LM head over more than 64 rows (139.6 GFLOP of bf16 work at 256 rows and 152 k features: 142 -> 129 us with the norm and the final kernel;
// below that one 64-row group streams the weights at HBM speed). Softmax statistics of a block's features per row: part[feature block][m] = {max, lowest index that attains it, sum exp(z - max)}. The tiles from vt on are
// the router's first layer: their sums go to r1 and stay out of the statistics (see EpiLmHead). logits: also written, or NULL.
struct TileHead {
    static constexpr bool pairs = false;
    float4 *part;
    float *logits, *r1;
    const int *live;   // device-side row count or NULL: with zero live rows the launch returns at once
    int M, V, vt, r1_stride, n_tiles;
    template <int WM> struct State { __device__ void init(const TileHead &, const int (&)[WM], int) {} };
    template <int GM, int GN, int WM, int WN>
    __device__ __forceinline__ void whole(const f32x16 (&acc)[WM][WN], const int (&m)[WM], int t0, int nb, int wm, int wn, float4 *lds) const
    {
        const int lane = threadIdx.x & 63, hf = lane >> 5;
#pragma unroll
        for (int mi = 0; mi < WM; ++mi) {
            float mx = -INFINITY, sum = 0.f;
            int idx = 0x7fffffff;
            auto each = [&](auto f) {   // the lane's features of the vocabulary, ascending
#pragma unroll
                for (int ni = 0; ni < WN; ++ni)
#pragma unroll
                    for (int r = 0; r < 16; ++r) f(ni, (t0 + ni) * 32 + 16 * (r >> 3) + 8 * hf + (r & 7), acc[mi][ni][r]);
            };
            each([&](int ni, int n, float z) {
                if (t0 + ni < vt && n < V && z > mx) { mx = z; idx = n; }   // strict: the lowest index wins ties
            });
            const float ref = mx == -INFINITY ? 0.f : mx;
            each([&](int ni, int n, float z) { sum += t0 + ni < vt && n < V ? __expf(z - ref) : 0.f; });
            if (logits && m[mi] < M)
                each([&](int ni, int n, float z) { if (t0 + ni < vt && n < V) logits[(size_t)m[mi] * V + n] = z; });
            if (m[mi] < M)
                each([&](int ni, int n, float z) { if (t0 + ni >= vt && t0 + ni < n_tiles) r1[(size_t)m[mi] * r1_stride + n - vt * 32] = z; });
            const float mo = __shfl_xor(mx, 32, 64), so = __shfl_xor(sum, 32, 64);
            const int io = __shfl_xor(idx, 32, 64);
            const float top = fmaxf(mx, mo), rt = top == -INFINITY ? 0.f : top;
            const int it = mx > mo || (mx == mo && idx < io) ? idx : io;
            if (hf == 0) lds[wn * (GM * WM * 32) + (wm * WM + mi) * 32 + lane] = make_float4(top, __int_as_float(it), sum * __expf(mx - rt) + so * __expf(mo - rt), 0.f);
        }
        __syncthreads();
        const int row = threadIdx.x;                                       // a row of the block; its waves' shares in ascending feature order
        const int r0 = m[0] - ((wm * WM) * 32 + (lane & 31)) + row;        // the block's first row, plus row
        if (row < GM * WM * 32 && r0 < M) {
            float top = -INFINITY, sum = 0.f;
            int idx = 0x7fffffff;
#pragma unroll
            for (int w = 0; w < GN; ++w) {
                const float4 p = lds[w * (GM * WM * 32) + row];
                if (p.x > top) { top = p.x; idx = __float_as_int(p.y); }
            }
#pragma unroll
            for (int w = 0; w < GN; ++w) {
                const float4 p = lds[w * (GM * WM * 32) + row];
                if (p.x > -INFINITY) sum += p.z * __expf(p.x - top);
            }
            part[(size_t)nb * M + r0] = make_float4(top, __int_as_float(idx), sum, 0.f);
        }
    }
};

__device__ __forceinline__ const TilePartial &partial_of(const TilePartial &e) { return e; }
__device__ __forceinline__ const TilePartial &partial_of(const TileResidualParts &e) { return e.rest; }

// ------------------------------------------------------------------ the kernel

// GM x GN wavefronts of WM x WN accumulators; ST: stages of one k-step in the ring; OCC: wavefronts per SIMD the registers must leave room for.
// Sums are formed in the order of the skinny kernels: the k-steps of a split (ksw of them) fall into four runs of `per` = ksw / 4 rounded up, each
// accumulated from zero by the matrix instructions (hi product, then lo product, k-step by k-step); the four runs of a split are added in order,
// and the splits are added in order to the epilogue's starting value. Where several workgroups share K (TilePartial, TileResidualParts) the splits are left
// apart for the next kernel to add in the same order, however many of them one workgroup walks. A pass over many rows then leaves the same bits in the cache as one over few: a bf16 cache turns another order
// of the same sums into other roundings, which 28 layers amplify to 1.3e-3 of the hidden rows (prompts of 39 to 71 tokens).
// SPLITS: more than one split is walked (or the start is not zero), which takes a third set of sums.
template <int GM, int GN, int WM, int WN, int ST, int OCC, bool SPLITS, class Epi>
__global__ __launch_bounds__(64 * GM *GN, OCC) void tile_gemm_kernel(TileArgs a, Epi epi)
{
    constexpr bool PLAIN = std::is_same_v<Epi, TileHead>;   // nothing depends on the order of the sum: one run
    constexpr bool APART = std::is_same_v<Epi, TilePartial>, CHAIN = std::is_same_v<Epi, TileResidualParts>;
    const bool apart = APART || (CHAIN && blockIdx.y > 0);   // this workgroup leaves its splits apart (uniform)
    if constexpr (PLAIN)
        if (epi.live && *epi.live == 0) return;   // uniform over the launch
    constexpr int NWV = GM * GN, BT = GN * WN, RB = GM * WM, CH = BT + 2 * RB;   // wavefronts, weight tiles, 32-row blocks, 1 KiB operands per k-step
    constexpr int L = CH / NWV, STG = CH * 64, P = ST - 1;
    static_assert(CH % NWV == 0 && (P - 1) * L < 64, "every wavefront copies the same number of operands; the wait counter has 6 bits");
    __shared__ __attribute__((aligned(1024))) uint4 sm[ST * STG];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, hf = lane >> 5, wm = wave % GM, wn = wave / GM;
    const int lin = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);   // workgroups are dealt to the 8 XCDs round-robin
    if (lin >= a.items) return;
    const int per_group = a.gm * a.n_nblk, mg = lin / per_group, rest = lin - mg * per_group, gsz = min(a.gm, a.n_mblk - mg * a.gm);
    const int mblk = mg * a.gm + rest % gsz, nb = rest / gsz;
    const int ks0 = blockIdx.y * a.kwg, ks1 = min(a.KS, ks0 + a.kwg), nstep = ks1 - ks0;

    // ---- loads: this wavefront copies operands wave, wave + NWV, ... of a step. Past the range the last step is loaded again (and not used), so that
    // the number of loads in flight is a constant.
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4 *)sm, lane_off = lane * 16;
    const char *src[L];
    uint32_t inc[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
        const int idx = wave + NWV * i;
        if (idx < BT) {
            const int t = min(nb * BT + idx, a.n_tiles - 1);
            src[i] = reinterpret_cast<const char *>(a.Wt + ((size_t)t * a.KS + ks0) * 64); inc[i] = 1024;
        } else {
            const int j = idx - BT, r32 = mblk * RB + (j >> 1), g = min(r32 >> 1, a.groups - 1);
            src[i] = reinterpret_cast<const char *>(a.pack + (((size_t)g * a.KS + ks0) * 4 + (j & 1) * 2 + (r32 & 1)) * 64); inc[i] = 4096;
        }
    }
    int more = nstep - 1;   // steps after the next one to be loaded
    uint32_t lbuf = lds0 + wave * 1024;
    auto issue = [&]() {
#pragma unroll
        for (int i = 0; i < L; ++i) {
            load_to_lds(lbuf + i * (NWV * 1024), lane_off, src[i]);
            src[i] += more > 0 ? inc[i] : 0;
        }
        --more;
        lbuf = lbuf + STG * 16 < lds0 + ST * STG * 16 ? lbuf + STG * 16 : lds0 + wave * 1024;
    };
#pragma unroll
    for (int p = 0; p < P; ++p) issue();

    int m[WM];
#pragma unroll
    for (int mi = 0; mi < WM; ++mi) m[mi] = (mblk * RB + wm * WM + mi) * 32 + (lane & 31);
    typename Epi::template State<WM> st;
    st.init(epi, m, hf);

    f32x16 acc[WM][WN], sum[WM][WN], tot[SPLITS ? WM : 1][SPLITS ? WN : 1];
    const int t0 = nb * BT + wn * WN;
    auto each = [&](auto f) {
#pragma unroll
        for (int mi = 0; mi < WM; ++mi)
#pragma unroll
            for (int ni = 0; ni < WN; ++ni) f(mi, ni);
    };
    auto run8 = [&](const f32x16 &c, int h, float (&v)[8]) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = c[8 * h + e];
    };
    if constexpr (SPLITS)
        if (!apart) each([&](int mi, int ni) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float v[8];
                epi.start(st, mi, m[mi], (t0 + ni) * 32 + 16 * h + 8 * hf, v);
#pragma unroll
                for (int e = 0; e < 8; ++e) tot[mi][ni][8 * h + e] = v[e];
            }
        });
    // At the barrier of step s every wavefront holds the operands of step s in registers, so that step's buffer is free for step s + ST.
    struct Operands { bf16x8 w[WN], h[WM], l[WM]; };
    Operands even, odd;
    const uint4 *const S0 = sm + lane;
    int rd = 0;
    auto fetch = [&](Operands &o) {
        const uint4 *S = S0 + rd;
#pragma unroll
        for (int mi = 0; mi < WM; ++mi) o.h[mi] = __builtin_bit_cast(bf16x8, S[(BT + 2 * (wm * WM + mi)) * 64]);
#pragma unroll
        for (int ni = 0; ni < WN; ++ni) o.w[ni] = __builtin_bit_cast(bf16x8, S[(wn * WN + ni) * 64]);
#pragma unroll
        for (int mi = 0; mi < WM; ++mi) o.l[mi] = __builtin_bit_cast(bf16x8, S[(BT + 2 * (wm * WM + mi) + 1) * 64]);
        rd = rd + STG < ST * STG ? rd + STG : 0;
    };
    // matrix instructions of the step held in `cur` while the next step's operands are read; nothing conditional in here
    auto step = [&](Operands &cur, Operands &nxt) {
        wait_and_barrier<(P - 1) * L>();
        issue();
        fetch(nxt);
        each([&](int mi, int ni) { acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.w[ni], cur.h[mi], acc[mi][ni], 0, 0, 0); });
        each([&](int mi, int ni) { acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.w[ni], cur.l[mi], acc[mi][ni], 0, 0, 0); });
        __builtin_amdgcn_sched_barrier(0);
    };
    auto clear = [&](f32x16 (&c)[WM][WN]) {
        each([&](int mi, int ni) {
#pragma unroll
            for (int r = 0; r < 16; ++r) c[mi][ni][r] = 0.f;
        });
    };
    wait_and_barrier<(P - 1) * L>();
    issue();                                                    // the ring is full
    fetch(even);
    int left = nstep, split = (CHAIN ? blockIdx.y - 1 : blockIdx.y) * a.spw;
    if constexpr (PLAIN) {
        clear(acc);
#pragma unroll 1
        for (; left >= 2; left -= 2) {
            step(even, odd);
            step(odd, even);
        }
        if (left) step(even, odd);
        wait_and_barrier<0>();                                  // no load may be in flight into LDS when it is used otherwise
        epi.template whole<GM, GN, WM, WN>(acc, m, t0, nb, wm, wn, reinterpret_cast<float4 *>(sm));
        return;
    }
#pragma unroll 1
    while (left > 0) {                                          // one split
        int in_split = min(left, a.ksw);
        const int per = (in_split + 3) / 4;
        left -= in_split;
        clear(sum);
#pragma unroll 1
        while (in_split > 0) {                                  // one run; the operands of its first step are in `even`
            int n = min(in_split, per);
            in_split -= n;
            clear(acc);
#pragma unroll 1
            for (; n >= 2; n -= 2) {
                step(even, odd);
                step(odd, even);
            }
            if (n) {
                step(even, odd);
                even = odd;
            }
            each([&](int mi, int ni) {
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[mi][ni][r] += acc[mi][ni][r];
            });
        }
        if constexpr (SPLITS)
            if (!apart) each([&](int mi, int ni) {
#pragma unroll
                for (int r = 0; r < 16; ++r) tot[mi][ni][r] += sum[mi][ni][r];
            });
        if constexpr (APART || CHAIN) if (apart) {   // (stores only make the waits of the next steps stricter: loads land in order)
            each([&](int mi, int ni) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float v[8];
                    run8(sum[mi][ni], h, v);
                    partial_of(epi).store(split, m[mi], t0 + ni, 16 * h + 8 * hf, v);
                }
            });
            ++split;
        }
    }
    wait_and_barrier<0>();                                      // no load may be in flight into LDS when the workgroup ends
    if constexpr (PLAIN || APART) return;
    else {
    if (apart) return;
    // one split: the starting value joins last (the same sum)
    auto value = [&](int mi, int ni, int h, float (&v)[8]) {
        if constexpr (SPLITS) run8(tot[mi][ni], h, v);
        else {
            float b[8];
            epi.start(st, mi, m[mi], (t0 + ni) * 32 + 16 * h + 8 * hf, b);
            run8(sum[mi][ni], h, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = b[e] + v[e];
        }
    };
    if constexpr (Epi::pairs) {
        static_assert(WN % 2 == 0, "whole gate/up pairs");
#pragma unroll
        for (int mi = 0; mi < WM; ++mi)
#pragma unroll
            for (int ni = 0; ni < WN; ni += 2)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float g[8], u[8];
                    value(mi, ni, h, g); value(mi, ni + 1, h, u);
                    epi.pair(st, mi, m[mi], t0 + ni, 16 * h + 8 * hf, g, u);
                }
    } else {
        each([&](int mi, int ni) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float v[8];
                value(mi, ni, h, v);
                epi.store(st, mi, m[mi], t0 + ni, 16 * h + 8 * hf, v);
            }
        });
    }
    }
}

// ------------------------------------------------------------------ launches

// Two block shapes: 128 x 128 (two workgroups per compute unit) and 64 x 128 (three). The smaller one moves half as many operand bytes again per
// product, the larger one leaves more of the chip idle in its last round, so the choice is by the rounds each takes, a small block costing 0.6 of a large
// one. Measured (us, 128 x 128 / 64 x 128): 8192 x 9728 x 896 253 / 264, 8192 x 1152 x 896 54 / 47, 8192 x 896 x 4864 141 / 153, 4096 x 896 x 4864
// 88 / 78, 512 x 37888 x 3584 244 / 266, 256 x 37888 x 3584 149 / 142, 1152 x 3584 x 18944 342 / 317, 2048 x 3584 x 18944 514 / 609.
static bool large_blocks(int M, int n_tiles, int nsplit)
{
    auto rounds = [&](int bm, int slots) { return ((M + bm - 1) / bm * ((n_tiles + 3) / 4) * nsplit + slots - 1) / slots; };
    return rounds(128, 512) * 512 <= rounds(64, 768) * 768 * 0.6;
}

template <bool SPLITS, class Epi>
static void launch_tile(hipStream_t s, TileArgs a, int nsplit, const Epi &epi)
{
    const bool large = large_blocks(a.M, a.n_tiles, nsplit);
    const int bm = large ? 128 : 64;
    a.groups = (a.M + 63) / 64;
    a.n_mblk = (a.M + bm - 1) / bm; a.n_nblk = (a.n_tiles + 3) / 4;
    const int walks = (a.n_mblk + 11) / 12;   // groups of up to 12 row blocks, all about the same size
    a.gm = (a.n_mblk + walks - 1) / walks;
    a.items = a.n_mblk * a.n_nblk; a.per_xcd = (a.items + 7) / 8;
    const dim3 grid(a.per_xcd * 8, nsplit);
    if (large) hipLaunchKernelGGL((tile_gemm_kernel<2, 2, 2, 2, 6, 2, SPLITS, Epi>), grid, dim3(256), 0, s, a, epi);
    else hipLaunchKernelGGL((tile_gemm_kernel<2, 2, 1, 2, 6, 3, SPLITS, Epi>), grid, dim3(256), 0, s, a, epi);
}

static TileArgs tile_args(const void *Wt, const void *pack, int K, int n_tiles, int M, int ksw)
{
    TileArgs a{};
    a.Wt = (const uint4 *)Wt; a.pack = (const uint4 *)pack; a.KS = a.kwg = K / 16; a.ksw = ksw; a.n_tiles = n_tiles; a.M = M;
    return a;
}

bool tile_fills_chip(int N, int M, int blocks) { return (M + 63) / 64 * (((N + 31) / 32 + 3) / 4) >= blocks; }

void launch_tile_qkv(hipStream_t s, int kdt, const Dims &D, const void *Wt, const void *pack, const float *bias, Rows rows, const float2 *rope, float *q,
                     void *kc, void *vc, int ksw)
{
    const TileArgs a = tile_args(Wt, pack, D.d, (D.qw + 2 * D.kvw) / 32, rows.n, ksw);
    auto go = [&](auto kt) {
        using KT = decltype(kt);
        const TileQkv<KT> e{{bias, rope, q, (KT *)kc, (KT *)vc, D.Hq, D.Hkv, D.dh, kv_unit_len(D), D.qw, kv_unit_vts(D)},
                            rows.slot, rows.pos, D.ptab, rows.n, a.n_tiles, D.page, D.maxp};
        if (ksw >= a.KS) launch_tile<false>(s, a, 1, e);
        else launch_tile<true>(s, a, 1, e);
    };
    if (kdt == DT_F32) go(float{}); else go(bf16_t{});
}

void launch_tile_swiglu(hipStream_t s, const Dims &D, const void *Wt, const void *pack, int M, void *hpack, const float *rstd, int ksw)
{
    const TileArgs a = tile_args(Wt, pack, D.d, 2 * ((D.F + 31) / 32), M, ksw);
    const TileSwiglu e{rstd, (uint4 *)hpack, M, D.F};
    if (ksw >= a.KS) launch_tile<false>(s, a, 1, e);
    else launch_tile<true>(s, a, 1, e);
}

void launch_tile_residual(hipStream_t s, const void *Wt, const void *pack, int K, int N, int M, float *x, const void *gain, void *pack_out, float *sumsq, int ksw)
{
    const TileArgs a = tile_args(Wt, pack, K, (N + 31) / 32, M, ksw);
    const TileResidual e{x, (const bf16_t *)gain, (uint4 *)pack_out, sumsq, M, N};
    if (ksw >= a.KS) launch_tile<false>(s, a, 1, e);
    else launch_tile<true>(s, a, 1, e);
}

// Workgroups along K for a product of few blocks: as many as leave every block of 64 x 128 a compute unit of its own, at least two, each with whole splits of
// the sum. Returns the number of splits.
static int share_splits(TileArgs &a, int N, int M)
{
    const int S = (a.KS + a.ksw - 1) / a.ksw, blocks = (M + 63) / 64 * ((N + 127) / 128), P = std::min(S, std::max(2, 256 / blocks));
    a.spw = (S + P - 1) / P;
    a.kwg = a.spw * a.ksw;
    return S;
}

void launch_tile_partial(hipStream_t s, const void *Wt, const void *pack, int K, int N, int M, float *part, int *nsplit)
{
    TileArgs a = tile_args(Wt, pack, K, (N + 31) / 32, M, gemm_split_steps(K, N, M));
    *nsplit = share_splits(a, N, M);
    launch_tile<false>(s, a, (*nsplit + a.spw - 1) / a.spw, TilePartial{part, N, M});
}

void launch_tile_residual_parts(hipStream_t s, const void *Wt, const void *pack, int K, int N, int M, float *x, float *part, int *nsplit)
{
    TileArgs a = tile_args(Wt, pack, K, (N + 31) / 32, M, gemm_split_steps(K, N, M));
    const int S = share_splits(a, N, M);
    *nsplit = S - a.spw;
    launch_tile<true>(s, a, (S + a.spw - 1) / a.spw, TileResidualParts{{x, nullptr, nullptr, nullptr, M, N}, {part, N, M}});
}

int tile_head_blocks(int V, int router_tiles) { return ((V + 31) / 32 + router_tiles + 7) / 8; }

// 128 x 256 blocks by 8 wavefronts, two workgroups per compute unit; where that leaves half a block of rows empty, 64 x 256 blocks by 4, three per
// compute unit. Whole tail of the 0.5B-class model at 256 / 160 / 100 rows: large blocks 130 / 118 / 76 us, small ones 137 / 99 / 74 us; at 256 rows with
// 4 wavefronts of 64 x 128 a block 131 us (one workgroup per compute unit: 168 us), with 256 x 256 blocks 163 us.
void launch_tile_head(hipStream_t s, const Dims &D, const void *Wt, const void *pack, int M, float *part, float *logits, float *r1, int router_tiles,
                      const int *live)
{
    const int vt = (D.V + 31) / 32;
    TileArgs a = tile_args(Wt, pack, D.d, vt + router_tiles, M, D.d / 16);
    const TileHead e{(float4 *)part, logits, r1, live, M, D.V, router_tiles > 0 ? vt : 0x7fffffff, router_tiles * 32, a.n_tiles};
    a.groups = (M + 63) / 64;
    const bool large = a.groups % 2 == 0;
    a.n_mblk = large ? a.groups / 2 : a.groups; a.n_nblk = tile_head_blocks(D.V, router_tiles);
    a.gm = a.n_mblk;   // the row blocks of a feature block next to each other: its weights come from HBM once
    a.items = a.n_mblk * a.n_nblk; a.per_xcd = (a.items + 7) / 8;
    if (large) hipLaunchKernelGGL((tile_gemm_kernel<2, 4, 2, 2, 5, 2, false, TileHead>), dim3(a.per_xcd * 8), dim3(512), 0, s, a, e);
    else hipLaunchKernelGGL((tile_gemm_kernel<1, 4, 2, 2, 4, 3, false, TileHead>), dim3(a.per_xcd * 8), dim3(256), 0, s, a, e);
}

// 1/rms of the rows from their sums of squares, in place: sumsq[row][0] = 1/rms. The order is that of EpiSwiglu: four groups of eight, added pairwise. One
// line of memory per row (8192 rows: 4.7 us; reading the rows themselves took 12). In the blocks of gate and up it would be done once per block, which cost
// more than this launch (64 prompts 69.7 ms against 68.3).
__global__ __launch_bounds__(64) void row_rstd_kernel(float *sumsq, int M, int n_ss, float eps, float inv_d)
{
    const int m = blockIdx.x * 64 + threadIdx.x;
    if (m >= M) return;
    const float4 *sp = reinterpret_cast<const float4 *>(sumsq + (size_t)m * SS_STRIDE);
    float p[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const float4 u = sp[2 * b], v = sp[2 * b + 1];
        const float r[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
        p[b] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) p[b] += 8 * b + i < n_ss ? r[i] : 0.f;
    }
    sumsq[(size_t)m * SS_STRIDE] = 1.0f / sqrtf(((p[0] + p[1]) + (p[2] + p[3])) * inv_d + eps);
}

void launch_row_rstd(hipStream_t s, float *sumsq, int M, int d, int n_ss, float eps)
{
    hipLaunchKernelGGL(row_rstd_kernel, dim3((M + 63) / 64), dim3(64), 0, s, sumsq, M, n_ss, eps, 1.0f / (float)d);
}

}  // namespace tr
