// All layers of a decode step of 9 to 64 rows in ONE launch (bf16 models of up to 896 columns, bf16 cache).
//
// The tasks, the way outputs are handed on and the order that lets the launch end are those of flow_kernels.hip. What differs is the work of a task: with this many rows a
// compute unit is bound by the activations it has to fetch (229 KB for 64 rows of 896 columns as hi and lo parts), so a task takes 16 rows (gate and up: 16 or 32) and few
// weight rows, and the operands need no conversion and no LDS on their way:
//   * Rows come in groups of 16, the columns of one v_mfma_f32_16x16x32_bf16. A producer leaves its outputs as the hi and lo operand of the next product: 16 bytes a lane,
//     1 KB a step of 32 columns and part, which a wavefront of the consumer loads straight into the registers the product reads.
//   * The norms are deferred: what is handed on is x * gain, with the sums of squares of each 16 columns of a row beside it; the consumer scales its sums by 1/rms.
//   * Work is split over workgroups by rows and features alone, so no sum is put together by a task of its own: the 8 wavefronts of a task share K and add up through the LDS.
//     Only long contexts are split (flow_rows_split), merged by tasks of their own.
// What bounds it: five or six hand-overs a layer and the rows that each task brings from the L2; 64 rows take 28 us a layer where their bytes take 10 at the copy rate.
// 0.5B-class model, a launch per link / here: 64 rows after 128 to 1024 keys 1132 / 760 us a step.
#include "flow_attention.h"
#include <algorithm>
#include <numeric>
#include <type_traits>
#include <utility>
#include <vector>

namespace tr {

constexpr int FR_W = FLOW_WAVES;   // wavefronts of a workgroup
constexpr int FR_NS = 4;       // steps of 32 columns per wavefront: up to 1024 columns
constexpr int FR_NSO = 4;      // of the output projection: up to 1024
constexpr int FR_NSD = 20;     // of the FFN output, per round: 5120 columns
constexpr int FR_BATCH = 10;    // of these, activations in flight
template <int DH> constexpr int FR_U = DH == 64 ? 3 : 1;   // blocks of 32 keys per wavefront

struct FlowRowsArgs {
    const char *wt;                   // tiled weights of layer 0
    size_t wt_stride;                 // bytes from layer to layer
    uint32_t wt_qkv, wt_o, wt_gu, wt_d;
    const float *bias; size_t bias_stride;
    const bf16_t *ln1[FLOW_MAX_LAYERS], *ln2[FLOW_MAX_LAYERS];
    char *kc, *vc; size_t k_layer, v_layer;   // bytes from layer to layer
    const int *slot, *pos;
    const float2 *rope;
    Dims D;
    float inv_d;                      // 1 / d
    int R, U, P;                      // rows; blocks of 32 keys per wavefront; most parts of a row's context
    int nG16, nPair;                  // groups of 16 rows; of 16 * PAIR rows
    float *buf;                       // the hand-over buffers, offsets and strides in words of 4 bytes
    uint32_t buf_bytes;
    // xa, pa, sa: a layer's input: residual rows, times the norm's gain as operands, sums of squares; x1, p1, s1: the same behind the output projection; q, kvn: query, new
    // key and value; ap: attention of parts of a context; at: attention; h: FFN activations as operands; out: the last layer's rows
    uint32_t o_xa, o_pa, o_sa, o_x1, o_p1, o_s1, o_q, o_kvn, o_ap, o_at, o_h, o_out, s_in, s_q, s_kvn, s_ap, s_at, s_h;
    int nQ, nA, nM, nO, nG, nD;       // tasks of a layer (nM: rows whose contexts are in parts)
    int uG;                           // groups of 8 gate and 8 up rows of a layer
    int *ticket, *given_up;           // next task; set when a wait was given up
    // the parts of all rows' contexts, row + 256 * part: first parts of the rows, those of several parts first, then the other parts
    uint32_t part[FLOW_ROWS_PARTS];
};
static_assert(sizeof(FlowRowsArgs) <= 4096, "kernel arguments");

// What values whose squares add up to sq (with others of their row) are handed on by: where that overflows, the row's 1/rms is 0 and they count for 0. Handed on as they are,
// their products with the gain or with a weight could be infinite, and infinity times 0 is a NaN. (Infinities become NaNs here.)
__device__ __forceinline__ float flow_rows_by(float sq) { return sq < INFINITY ? 1.f : 0.f; }

// QU, OU: groups of 16 weight rows of a q|k|v and of an output projection task; PAIR: groups of 16 rows of a gate/up task; GU: its groups of 8 gate and 8 up rows; DR: rows of an FFN output task (16 or 8)
template <int DH, int QU, int OU, int PAIR, int GU, int DR>
struct FlowRows : FlowAttention<FlowRows<DH, QU, OU, PAIR, GU, DR>, DH, 256, 2, FR_U<DH>> {
    static constexpr int MOST = PAIR * GU;
    union Lds {
        struct { f32x4 red[FR_W][MOST][64]; float ss[PAIR][FR_W][16]; } g;
        FlowAttentionLds<DH> att;
    };
    static_assert(PAIR == 1 || PAIR == 2, "");
    static_assert(MOST >= QU && MOST >= OU, "");
    typedef FlowPiece<u32x4, 1, 2 * FR_NS> Operands;          // a wavefront's steps of one group of rows, hi and lo
    const FlowRowsArgs &a;
    Lds &lds;
    __amdgpu_buffer_rsrc_t buf;
    int wave, lane, col, o;

    __device__ __forceinline__ FlowRows(const FlowRowsArgs &args, Lds &l) : a(args), lds(l)
    {
        buf = buffer_of(a.buf, a.buf_bytes);
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); lane = threadIdx.x & 63;
        col = lane & 15; o = lane >> 4;
    }
    __device__ __forceinline__ FlowWait wait() const { return FlowWait{a.given_up}; }
    __device__ __forceinline__ const char *layer(int l) const { return a.wt + (size_t)l * a.wt_stride; }

    struct Share { int s0, ns; };   // a wavefront's steps s0 .. s0 + ns - 1
    __device__ __forceinline__ Share share(int n32) const
    {
        const int s0 = wave * n32 / FR_W;
        return Share{s0, (wave + 1) * n32 / FR_W - s0};
    }
    // this lane's 16 bytes of a step: row col of a group
    __device__ __forceinline__ uint32_t row_off(uint32_t tile, uint32_t row, int n32) const { return tile * (uint32_t)n32 * 2048 + (o >> 1) * 1024 + (o & 1) * 512 + row * 16; }
    __device__ __forceinline__ uint32_t group_off(int unit, int n32) const { return row_off(unit >> 1, 16 * (unit & 1) + col, n32); }
    template <int N> __device__ __forceinline__ static void weights(uint4 (&w)[N], const char *base, uint32_t off, Share sh)   // past the share: its last step again
    {
#pragma unroll
        for (int s = 0; s < N; ++s) {
            const char *p = base + (size_t)(sh.s0 + min(s, max(sh.ns, 1) - 1)) * 2048;
            asm("" : "+s"(p));
            w[s] = *reinterpret_cast<const uint4 *>(p + off);
        }
    }
    // operands of rows 16 rg .. as a producer left them at `base` (bytes, of this group): steps of the share, hi and lo of each (past the share: its last step again); rows
    // that do not exist: zeros
    template <int N> __device__ __forceinline__ void operand_places(FlowPiece<u32x4, 1, N> &x, uint32_t base, int rg, int s0, int ns) const
    {
        x.off[0] = 16 * rg + col < a.R ? base + s0 * 2048 + lane * 16 : BUFFER_NOWHERE;
#pragma unroll
        for (int i = 0; i < N; ++i) x.set[i] = min(i / 2, max(ns, 1) - 1) * 2048 + (i & 1) * 1024;
    }
    template <int N> __device__ __forceinline__ static void multiply(f32x4 &c, const uint4 *w, const FlowPiece<u32x4, 1, N> &x, int ns)
    {
#pragma unroll
        for (int s = 0; s < N / 2; ++s) {
            if (s < ns) {   // (uniform)
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[s]), __builtin_bit_cast(bf16x8, x.v[2 * s][0]), c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[s]), __builtin_bit_cast(bf16x8, x.v[2 * s + 1][0]), c, 0, 0, 0);
            }
        }
    }
    // Sums of squares of the rows of a group, left per 16 columns: [tile][row]. A wavefront brings those of its share, four lanes a row.
    typedef FlowPiece<uint32_t, FR_NS / 2> Norm;
    __device__ __forceinline__ void norm_places(Norm &n, uint32_t base, int rg, Share sh) const
    {
#pragma unroll
        for (int i = 0; i < FR_NS / 2; ++i) n.off[i] = 16 * rg + col < a.R && 4 * i + o < 2 * sh.ns ? base + ((2 * sh.s0 + 4 * i + o) * 16 + col) * 4 : BUFFER_NOWHERE;
    }
    __device__ __forceinline__ void add_squares(const Norm &n, int p) const
    {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < FR_NS / 2; ++i) s += __uint_as_float(n.v[0][i]);
        s = flow_sum4(s);
        if (o == 0) lds.g.ss[p][wave][col] = s;
    }
    __device__ __forceinline__ float rstd(int p, float inv_d, float eps) const   // of row col (after the barrier)
    {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < FR_W; ++w) s += lds.g.ss[p][w][col];
        return flow_rsqrt(fmaf(s, inv_d, eps));
    }
    // combination c of a task's sums (16 weight rows x 16 rows), over the wavefronts
    __device__ __forceinline__ f32x4 sum(int c) const
    {
        f32x4 v = lds.g.red[0][c][lane];
#pragma unroll
        for (int w = 1; w < FR_W; ++w) v += lds.g.red[w][c][lane];
        return v;
    }
    // first of the 4 consecutive features that a lane's results of a group of 16 are (tile_feature)
    __device__ __forceinline__ int feature4(int unit) const { return 16 * unit + 8 * (o & 1) + 4 * (o >> 1); }
    // bytes of group rg: residual rows and operands (both 64 bytes a column); sums of squares
    __device__ __forceinline__ uint32_t at_group(uint32_t words, int rg, int K) const { return words * 4 + rg * K * 64; }
    __device__ __forceinline__ uint32_t at_squares(uint32_t words, int rg) const { return words * 4 + rg * a.D.d * 4; }
    __device__ __forceinline__ uint32_t at_tile(uint32_t words, int rg, int unit, int row) const { return at_group(words, rg, a.D.d) + unit * 1024 + (o * 16 + row) * 16; }   // residual rows: as the products leave them
    // a layer's rows handed on: residual, operand of the next product, sums of squares; row `row` of group rg, if `on`
    __device__ __forceinline__ void leave(uint32_t x, uint32_t p, uint32_t s, int rg, int row, bool on, int unit, f32x4 v, uint2 gain) const
    {
        float sq = v.x * v.x;
        sq = fmaf(v.y, v.y, sq); sq = fmaf(v.z, v.z, sq); sq = fmaf(v.w, v.w, sq);
        sq = flow_sum4(sq);
        if (!on) return;
        uint32_t h0, h1, l0, l1;
        const f32x4 n = v * flow_rows_by(sq);
        split_hi_lo(n.x * __uint_as_float(gain.x << 16), n.y * __uint_as_float(gain.x & 0xffff0000u), h0, l0);
        split_hi_lo(n.z * __uint_as_float(gain.y << 16), n.w * __uint_as_float(gain.y & 0xffff0000u), h1, l1);
        const uint32_t at = at_group(p, rg, a.D.d) + (unit >> 1) * 2048 + ((2 * (unit & 1) + (o & 1)) * 16 + row) * 16 + (o >> 1) * 8;
        flow_store_pair(buf, at, h0, h1);
        flow_store_pair(buf, at + 1024, l0, l1);
        if (o == 0) flow_store(buf, at_squares(s, rg) + (unit * 16 + row) * 4, sq);
        flow_store(buf, at_tile(x, rg, unit, row), v);
    }

    // ---- tasks
    __device__ __forceinline__ void qkv(int l, int task) const
    {
        const int rg = task % a.nG16, u0 = task / a.nG16 * QU, n32 = a.D.d / 32, unit = u0 + min(wave, QU - 1), m = min(16 * rg + col, a.R - 1);
        const Share sh = share(n32);
        uint4 w[QU][FR_NS];
#pragma unroll
        for (int u = 0; u < QU; ++u) weights(w[u], layer(l) + a.wt_qkv, group_off(u0 + u, n32), sh);
        const bool fin = wave < QU;
        const int half = DH / 2, Hq = flow_now(a.D.Hq), Hkv = flow_now(a.D.Hkv);
        const int f = feature4(unit), tph = DH >> 5, hh = (f >> 5) / tph, j = ((f >> 5) % tph) * 16 + ((f & 31) >> 1);   // rotary pairs j, j + 1 of head hh
        const int pos = a.pos[m], slot = a.slot[m];
        const float *bias = a.bias + l * a.bias_stride + hh * DH + j;
        const float2 ba = *reinterpret_cast<const float2 *>(bias), bb = *reinterpret_cast<const float2 *>(bias + half);
        const float4 cs = *reinterpret_cast<const float4 *>(a.rope + (size_t)pos * half + j);
        const KvPlace at = kv_place(a.D, slot, pos);
        const bool key = hh < Hq + Hkv;
        const int head = key ? hh - Hq : hh - Hq - Hkv;
        bf16_t *cache = key ? reinterpret_cast<bf16_t *>(a.kc + (size_t)l * a.k_layer) + k_offset(a.D, at.unit, max(head, 0), at.pos, j)
                            : reinterpret_cast<bf16_t *>(a.vc + (size_t)l * a.v_layer) + v_offset(a.D, at.unit, max(head, 0), at.pos, j);
        const uint32_t at_q = (a.o_q + l * a.s_q) * 4 + ((rg * Hq + hh) * 3 * (DH / 8) + (j >> 3)) * 256 + col * 16 + (j & 7) * 2;
        const uint32_t at_n = (a.o_kvn + l * a.s_kvn) * 4 + ((rg * Hkv + head) * 2 * (DH / 8) + (key ? 0 : DH / 8) + (j >> 3)) * 256 + col * 16 + (j & 7) * 2;
        const float inv_d = flow_now(a.inv_d), eps = flow_now(a.D.eps);
        Operands x;
        Norm n;
        const uint32_t base = at_group(a.o_pa + l * a.s_in, rg, a.D.d);
        operand_places(x, base, rg, sh.s0, sh.ns);
        norm_places(n, at_squares(a.o_sa + l * a.s_in, rg), rg, sh);
        Sample sample;
        sample_rows(sample, base, sh, 1, 0);
        flow_await(buf, l > 0 ? at_group(a.o_h + (l - 1) * a.s_h, rg, a.D.F) + task % (a.D.F / 32) * 2048 : base, wait(), sample);
        flow_fetch(buf, wait(), x, n);
        add_squares(n, 0);
#pragma unroll
        for (int u = 0; u < QU; ++u) {
            f32x4 c = {0.f, 0.f, 0.f, 0.f};
            multiply(c, w[u], x, sh.ns);
            lds.g.red[wave][u][lane] = c;
        }
        __syncthreads();
        if (!fin) return;
        const float rs = rstd(0, inv_d, eps);
        const f32x4 v = sum(wave);
        if (16 * rg + col >= a.R) return;
        const float a0 = fmaf(v.x, rs, ba.x), b0 = fmaf(v.y, rs, bb.x), a1 = fmaf(v.z, rs, ba.y), b1 = fmaf(v.w, rs, bb.y);
        float lo0 = a0, hi0 = b0, lo1 = a1, hi1 = b1;
        if (key) {   // (queries too)
            lo0 = a0 * cs.x - b0 * cs.y; hi0 = b0 * cs.x + a0 * cs.y;
            lo1 = a1 * cs.z - b1 * cs.w; hi1 = b1 * cs.z + a1 * cs.w;
        }
        if (hh < Hq) {   // three parts of the scaled query
            const float scale = 1.0f / sqrtf((float)DH);
            lo0 *= scale; lo1 *= scale; hi0 *= scale; hi1 *= scale;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const uint32_t wl = flow_part(lo0, lo1), wh = flow_part(hi0, hi1);
                flow_store_pair(buf, at_q + p * DH * 32, wl);
                flow_store_pair(buf, at_q + p * DH * 32 + half * 32, wh);
            }
            return;
        }
        const uint32_t plo = flow_part(lo0, lo1), phi = flow_part(hi0, hi1);
        flow_store_pair(buf, at_n, plo);   // the values that the cache will hold, for this step's attention
        flow_store_pair(buf, at_n + half * 32, phi);
        if (key) {
            *reinterpret_cast<uint32_t *>(cache) = plo;
            *reinterpret_cast<uint32_t *>(cache + half) = phi;
        } else {
            cache[0] = (bf16_t)plo; cache[32] = (bf16_t)(plo >> 16);
            cache[half * 32] = (bf16_t)phi; cache[half * 32 + 32] = (bf16_t)(phi >> 16);
        }
    }
    // One word of the last part of what each producer left of a share: 16 columns each (the rows' operands; `groups` of 16 rows, `stride` bytes apart) ..
    typedef FlowPiece<uint32_t, 1> Sample;
    __device__ __forceinline__ void sample_rows(Sample &x, uint32_t base, Share sh, int groups, uint32_t stride) const
    {
        static_assert(2 * FR_NS * PAIR <= 64, "");
        const int p = lane / (2 * FR_NS), s = lane / 2 % FR_NS;
        x.off[0] = p < groups && s < sh.ns ? base + p * stride + (sh.s0 + s) * 2048 + 1024 + (lane & 1) * 512 : BUFFER_NOWHERE;
    }
    // .. or 8 columns each (FFN activations)
    static constexpr int HS = (4 * FR_NSD + 63) / 64;
    __device__ __forceinline__ void sample_ffn(FlowPiece<uint32_t, HS> &x, uint32_t base, Share sh) const
    {
#pragma unroll
        for (int i = 0; i < HS; ++i) {
            const int s = lane / 4 + 16 * i;
            x.off[i] = s < min(sh.ns, FR_NSD) ? base + (sh.s0 + s) * 2048 + 1024 + (lane & 3) * 256 : BUFFER_NOWHERE;
        }
    }

    // ---- attention: where its input and output lie (bytes): queries, keys and values of 16 rows side by side, 8 dims each; its output row by row
    __device__ __forceinline__ uint32_t q_at(int l, int r, int head) const { return (a.o_q + l * a.s_q) * 4 + ((r >> 4) * a.D.Hq + head) * 3 * DH * 32 + (r & 15) * 16; }
    __device__ __forceinline__ uint32_t kvn_at(int l, int r, int g) const { return (a.o_kvn + l * a.s_kvn) * 4 + ((r >> 4) * a.D.Hkv + g) * 2 * DH * 32 + (r & 15) * 16; }
    __device__ __forceinline__ uint32_t vn_behind() const { return DH * 32; }
    __device__ __forceinline__ uint32_t plane() const { return a.R * a.D.qw * 2; }
    __device__ __forceinline__ uint32_t out_of(int l, int r, int g) const { return (a.o_at + l * a.s_at) * 4 + (r * a.D.qw + g * a.D.G * DH) * 2; }
    __device__ __forceinline__ uint32_t attention_gate(int l, int r) const { return at_group(a.o_pa + l * a.s_in, r >> 4, a.D.d) + r % (a.D.d / 32) * 2048; }
    __device__ __forceinline__ uint32_t merge_gate(int l, int r) const { return kvn_at(l, r, 0); }

    // x1 = x + Wo . attention
    __device__ __forceinline__ void oproj(int l, int task) const
    {
        const int rg = task % a.nG16, u0 = task / a.nG16 * OU, nU = a.D.d / 16, unit = min(u0 + min(wave, OU - 1), nU - 1), n32 = a.D.qw / 32, m = 16 * rg + col;
        const Share sh = share(n32);
        uint4 w[OU][FR_NSO];
#pragma unroll
        for (int u = 0; u < OU; ++u) weights(w[u], layer(l) + a.wt_o, group_off(min(u0 + u, nU - 1), n32), sh);
        const uint2 gain = *reinterpret_cast<const uint2 *>(a.ln2[l] + feature4(unit));
        FlowPiece<u32x4, 1> old;
        old.off[0] = wave < OU && m < a.R ? at_tile(a.o_xa + l * a.s_in, rg, unit, col) : BUFFER_NOWHERE;
        const uint32_t base = (a.o_at + l * a.s_at) * 4, plane = a.R * a.D.qw * 2;
        FlowPiece<u32x4, 1, 2 * FR_NSO> x;
        x.off[0] = m < a.R ? base + (m * a.D.qw + 32 * sh.s0 + 8 * o) * 2 : BUFFER_NOWHERE;
#pragma unroll
        for (int i = 0; i < 2 * FR_NSO; ++i) x.set[i] = (i & 1) * plane + min(i / 2, max(sh.ns, 1) - 1) * 64;
        // one word of the last part of each row and head of the share (at most five heads)
        FlowPiece<uint32_t, 2> sample;
        const int first = 32 * sh.s0, last = 32 * (sh.s0 + max(sh.ns, 1)) - 1;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = max(first, min((first / DH + o + 4 * i) * DH, last)) & ~1;
            sample.off[i] = m < a.R ? base + plane + (m * a.D.qw + k) * 2 : BUFFER_NOWHERE;
        }
        const uint32_t out_x = a.o_x1 + l * a.s_in, out_p = a.o_p1 + l * a.s_in, out_s = a.o_s1 + l * a.s_in;
        flow_await(buf, (a.o_q + l * a.s_q) * 4 + (rg * a.D.Hq + unit % a.D.Hq) * 3 * DH * 32, wait(), sample);
        flow_fetch(buf, wait(), x, old);
#pragma unroll
        for (int u = 0; u < OU; ++u) {
            f32x4 c = {0.f, 0.f, 0.f, 0.f};
            multiply(c, w[u], x, sh.ns);
            lds.g.red[wave][u][lane] = c;
        }
        __syncthreads();
        if (wave >= OU || u0 + wave >= nU) return;
        leave(out_x, out_p, out_s, rg, col, m < a.R, unit, sum(wave) + __builtin_bit_cast(f32x4, old.v[0][0]), gain);
    }

    // 8 gate rows and the 8 up rows of the same features in one operand
    __device__ __forceinline__ void gateup(int l, int task) const
    {
        const int rg0 = task % a.nPair * PAIR, u0 = task / a.nPair * GU, n32 = a.D.d / 32;
        const Share sh = share(n32);
        uint4 w[GU][FR_NS];
#pragma unroll
        for (int u = 0; u < GU; ++u) {   // features 8 t .. + 7 of gate and of up
            const int t = min(u0 + u, a.uG - 1);
            weights(w[u], layer(l) + a.wt_gu, row_off(2 * (t >> 2) + (col >> 3), 16 * ((t & 3) >> 1) + 4 * (t & 1) + 8 * ((col >> 2) & 1) + (col & 3), n32), sh);
        }
        const float inv_d = flow_now(a.inv_d), eps = flow_now(a.D.eps);
        const uint32_t base = at_group(a.o_p1 + l * a.s_in, rg0, a.D.d);
        Operands x[PAIR];
        Norm n[PAIR];
#pragma unroll
        for (int p = 0; p < PAIR; ++p) {
            operand_places(x[p], base + p * a.D.d * 64, rg0 + p, sh.s0, sh.ns);
            norm_places(n[p], at_squares(a.o_s1 + l * a.s_in, rg0 + p), rg0 + p, sh);
        }
        const int mine = rg0 + wave % PAIR;   // the rows that the wavefront finishes
        Sample sample;
        sample_rows(sample, base, sh, min(PAIR, a.nG16 - rg0), a.D.d * 64);
        flow_await(buf, (a.o_at + l * a.s_at) * 4 + (min(16 * rg0 + task % (16 * PAIR), a.R - 1) * a.D.qw) * 2, wait(), sample);
        if constexpr (PAIR == 2) flow_fetch(buf, wait(), x[0], x[1], n[0], n[1]);
        else flow_fetch(buf, wait(), x[0], n[0]);
#pragma unroll
        for (int p = 0; p < PAIR; ++p) add_squares(n[p], p);
#pragma unroll
        for (int u = 0; u < GU; ++u)
#pragma unroll
            for (int p = 0; p < PAIR; ++p) {
                f32x4 c = {0.f, 0.f, 0.f, 0.f};
                multiply(c, w[u], x[p], sh.ns);
                lds.g.red[wave][u * PAIR + p][lane] = c;
            }
        const uint32_t out = at_group(a.o_h + l * a.s_h, mine, a.D.F) + (o >> 1) * 1024 + col * 16 + (o & 1) * 8;
        __syncthreads();
        const float rs = rstd(wave % PAIR, inv_d, eps);
#pragma unroll
        for (int i = 0; i < (MOST + FR_W - 1) / FR_W; ++i) {
            const int c = wave + i * FR_W, unit = u0 + c / PAIR;
            if (c >= MOST || unit >= a.uG) break;   // (uniform)
            const f32x4 v = sum(c);
            float t[4], h[4];
            f32x4 up;
#pragma unroll
            for (int e = 0; e < 4; ++e) { const FlowTwo two = flow_halves(v[e]); t[e] = two.a * rs; up[e] = two.b * rs; }   // gate rows: lanes 0 to 31, up rows: 32 to 63
            flow_silu(t, h);
            uint32_t h0, h1, l0, l1;
            split_hi_lo(h[0] * up[0], h[1] * up[1], h0, l0);
            split_hi_lo(h[2] * up[2], h[3] * up[3], h1, l1);
            if (16 * mine + col < a.R) flow_store_pair(buf, out + (unit >> 2) * 2048 + (unit & 3) * 256, o < 2 ? h0 : l0, o < 2 ? h1 : l1);
        }
    }

    // x of the next layer = x1 + Wd . h, of 16 rows, or of 8: their hi and lo parts side by side in the 16 columns of one product
    template <int ROWS> __device__ __forceinline__ void down(int l, int task) const
    {
        constexpr int PARTS = ROWS / 8, GROUPS = 16 / ROWS, BATCH = ROWS == 16 ? FR_BATCH : FR_NSD;
        const int n8 = (a.R + ROWS - 1) / ROWS, r0 = task % n8 * ROWS, rg = r0 >> 4, unit = task / n8, n32 = a.D.F / 32;
        const int row = (r0 & 15) + col % ROWS, m = 16 * rg + row;
        const bool in = m < a.R;
        const Share sh = share(n32);
        const char *wbase = layer(l) + a.wt_d;
        const uint32_t woff = group_off(unit, n32);
        uint4 w[FR_NSD];
        weights(w, wbase, woff, sh);
        const bool last = l == a.D.L - 1;
        const uint2 gain = *reinterpret_cast<const uint2 *>(a.ln1[last ? l : l + 1] + feature4(unit));
        const uint32_t base = at_group(a.o_h + l * a.s_h, rg, a.D.F) + (r0 & 15) * 16, out = (a.o_out + m * a.D.d + feature4(unit)) * 4;
        const uint32_t out_x = a.o_xa + (l + 1) * a.s_in, out_p = a.o_pa + (l + 1) * a.s_in, out_s = a.o_sa + (l + 1) * a.s_in;
        FlowPiece<u32x4, 1> old;
        old.off[0] = wave == 0 && in ? at_tile(a.o_x1 + l * a.s_in, rg, unit, row) : BUFFER_NOWHERE;
        const uint32_t gate = at_group(a.o_p1 + l * a.s_in, rg, a.D.d) + task % (a.D.d / 32) * 2048;
        f32x4 c = {0.f, 0.f, 0.f, 0.f};
        for (int done = 0; done == 0 || done < sh.ns; done += FR_NSD) {   // (one round up to 5120 FFN columns)
            if (done > 0) weights(w, wbase, woff, Share{sh.s0 + done, sh.ns - done});
            const int ns = min(sh.ns - done, FR_NSD);
            FlowPiece<uint32_t, HS> sample;
            sample_ffn(sample, base, Share{sh.s0 + done, ns});
            flow_await(buf, gate, wait(), sample, old);
#pragma unroll
            for (int b = 0; b < FR_NSD; b += BATCH) {
                if (b < ns) {   // (uniform)
                    FlowPiece<u32x4, 1, PARTS * BATCH> x;
                    const uint32_t at = base + (sh.s0 + done + b) * 2048 + o * 256 + col % ROWS * 16;
                    x.off[0] = in ? ROWS == 16 ? at : at + (col >> 3) * 1024 : BUFFER_NOWHERE;
#pragma unroll
                    for (int i = 0; i < PARTS * BATCH; ++i) x.set[i] = min(i / PARTS, ns - b - 1) * 2048 + i % PARTS * 1024;
                    flow_fetch(buf, wait(), x);
#pragma unroll
                    for (int i = 0; i < PARTS * BATCH; ++i)
                        if (i / PARTS < ns - b) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[b + i / PARTS]), __builtin_bit_cast(bf16x8, x.v[i][0]), c, 0, 0, 0);
                }
            }
        }
        lds.g.red[wave][0][lane] = c;
        __syncthreads();
        if (wave > 0) return;
        f32x4 v = sum(0);
        if (GROUPS > 1)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += flow_next<8>(v[e]);
        v += __builtin_bit_cast(f32x4, old.v[0][0]);
        const bool on = in && col < ROWS;
        if (!last) leave(out_x, out_p, out_s, rg, row, on, unit, v, gain);
        else if (on) flow_store(buf, out, v);
    }
};

template <int DH, int QU, int OU, int PAIR, int GU, int DR>
__global__ __launch_bounds__(64 * FR_W, 2) void flow_rows_kernel(FlowRowsArgs args)
{
    __shared__ typename FlowRows<DH, QU, OU, PAIR, GU, DR>::Lds lds;
    __shared__ int s_task[2];
    if (threadIdx.x == 0) s_task[0] = atomicAdd(args.ticket, 1);
    __syncthreads();
    for (int it = 0;; it ^= 1) {
        const int t = __builtin_amdgcn_readfirstlane(s_task[it]);
        // (the arguments are read again for every task: kept in registers over the loop they would not fit)
        auto kernarg = __builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(kernarg));
        const FlowRowsArgs &a = *(const FlowRowsArgs *)kernarg;
        const int per_layer = a.nQ + a.nA + a.nM + a.nO + a.nG + a.nD;
        if (t >= per_layer * a.D.L) break;   // uniform over the workgroup
        FlowRows<DH, QU, OU, PAIR, GU, DR> f(a, lds);
        const int l = t / per_layer;
        int i = t - l * per_layer;
        if (i < a.nQ) f.qkv(l, i);
        else if ((i -= a.nQ) < a.nA) { const uint32_t p = a.part[i / a.D.Hkv]; f.attention(l, p & 0xff, i % a.D.Hkv, p >> 8); }
        else if ((i -= a.nA) < a.nM) { f.merge(l, a.part[i] & 0xff, 0, a.D.Hq); __syncthreads(); }   // (not all of its wavefronts have something to wait for)
        else if ((i -= a.nM) < a.nO) f.oproj(l, i);
        else if ((i -= a.nO) < a.nG) f.gateup(l, i);
        else f.template down<DR>(l, i - a.nG);
        // (see flow_kernel)
        if (threadIdx.x == 64 * (FR_W - 1)) s_task[it ^ 1] = atomicAdd(a.ticket, 1);
        __syncthreads();   // also: the LDS is free for the next task
    }
}

// ------------------------------------------------------------------ set-up

struct FlowRowsSetup { int slot[FLOW_ROWS_MAX], tok[FLOW_ROWS_MAX], pos[FLOW_ROWS_MAX]; };

// Row tables and the first layer's input (blocks 0 .. R - 1: a row each), the other hand-over buffers to SENT (the others), task counter to zero
__global__ __launch_bounds__(256) void flow_rows_setup_kernel(FlowRowsSetup a, int R, int *d_slot, int *d_tok, int *d_pos, const bf16_t *E, const bf16_t *gain, int d, int vocab,
                                                              const int *dev_tok, char *x, char *pack, char *squares, uint4 *fill, uint32_t n_fill, uint32_t skip, int *ticket)
{
    const int b = blockIdx.x;
    if (b < R) {
        const int tok = dev_tok ? min(max(dev_tok[b], 0), vocab - 1) : a.tok[b], rg = b >> 4, col = b & 15;
        if (threadIdx.x == 0) { d_slot[b] = a.slot[b]; d_tok[b] = tok; d_pos[b] = a.pos[b]; }
        if (b == 0 && threadIdx.x == 0) *ticket = 0;
        for (int t = threadIdx.x; t < d / 16; t += 256) {   // 16 columns
            const uint4 *e = reinterpret_cast<const uint4 *>(E + (size_t)tok * d + 16 * t), *gp = reinterpret_cast<const uint4 *>(gain + 16 * t);
            float sq = 0.f;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint4 u = e[h], g = gp[h];
                float v[8], n[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t ui = i == 0 ? u.x : i == 1 ? u.y : i == 2 ? u.z : u.w, gi = i == 0 ? g.x : i == 1 ? g.y : i == 2 ? g.z : g.w;
                    v[2 * i] = __uint_as_float(ui << 16); v[2 * i + 1] = __uint_as_float(ui & 0xffff0000u);
                    n[2 * i] = v[2 * i] * flow_rows_by(v[2 * i] * v[2 * i]) * __uint_as_float(gi << 16);
                    n[2 * i + 1] = v[2 * i + 1] * flow_rows_by(v[2 * i + 1] * v[2 * i + 1]) * __uint_as_float(gi & 0xffff0000u);
                    sq = fmaf(v[2 * i], v[2 * i], sq); sq = fmaf(v[2 * i + 1], v[2 * i + 1], sq);
                }
                uint4 hi, lo;
                split_hi_lo(n, hi, lo);
                hi = make_uint4(flow_pair(hi.x), flow_pair(hi.y), flow_pair(hi.z), flow_pair(hi.w));
                lo = make_uint4(flow_pair(lo.x), flow_pair(lo.y), flow_pair(lo.z), flow_pair(lo.w));
                char *at = pack + (size_t)rg * d * 64 + (t >> 1) * 2048 + ((2 * (t & 1) + h) * 16 + col) * 16;
                *reinterpret_cast<uint4 *>(at) = hi;
                *reinterpret_cast<uint4 *>(at + 1024) = lo;
                char *ax = x + (size_t)rg * d * 64 + t * 1024 + (h * 16 + col) * 16;   // columns 8 h + 4 q: lanes of quarter h + 2 q
                *reinterpret_cast<float4 *>(ax) = make_float4(v[0], v[1], v[2], v[3]);
                *reinterpret_cast<float4 *>(ax + 512) = make_float4(v[4], v[5], v[6], v[7]);
            }
            reinterpret_cast<uint32_t *>(squares + (size_t)rg * d * 4)[t * 16 + col] = flow_word(sq);
        }
        return;
    }
    for (uint32_t i = skip + (b - R) * 256 + threadIdx.x; i < n_fill; i += (gridDim.x - R) * 256) fill[i] = make_uint4(SENT, SENT, SENT, SENT);
}

// ------------------------------------------------------------------ launches

// parts of a context of `pos` cached keys, U blocks of 32 keys to a wavefront
static int flow_rows_parts(int pos, int U) { return std::max(1, (pos + 32 * FR_W * U - 1) / (32 * FR_W * U)); }
static int flow_rows_most(int R) { return FLOW_ROWS_PARTS / R; }

// One part of every context where the registers hold the longest (768 keys; 256 of 128-wide heads): a part and its merge cost more than the blocks that they save. Against the
// rule below, which splits from 257 keys on: 16 rows after 200 to 600 keys 476 us a step and 490, 32 after 128 to 700 559 and 577, 64 after 128 to 512 709 and 744.
// Else the smallest parts that make no more tasks than can be under way while their queries are computed; false: more parts than there is room for. Blocks per wavefront
// 1 / 2 / 3: 16 rows after 100 to 1900 keys 542 / 512 / 540 us, 32 rows after 128 to 1024 616 / 590 / 594, 64 rows 834 / 765 / 771.
static bool flow_rows_split(const Dims &D, int R, const int *poss, FlowRowsPlan *p)
{
    const int umax = D.dh == 64 ? FR_U<64> : FR_U<128>, longest = *std::max_element(poss, poss + R);
    p->P = 1;
    for (p->U = 1; p->U <= umax; ++p->U)
        if (flow_rows_parts(longest, p->U) == 1) return true;
    for (p->U = 1;; ++p->U) {
        p->P = flow_rows_parts(longest, p->U);
        int tasks = 0;
        for (int r = 0; r < R; ++r) tasks += flow_rows_parts(poss[r], p->U) * D.Hkv;
        if (p->P <= flow_rows_most(R) && (tasks <= (R <= 32 ? 128 : 256) || p->U == umax)) return true;
        if (p->U == umax) return false;
    }
}

// words that the buffers take; *first: the first layer's input, at the front; *filled: what is to be SENT or that
static size_t flow_rows_layout(const Dims &D, int R, int P, FlowRowsArgs &a, size_t *first, size_t *filled)
{
    const size_t rows = (size_t)(R + 15) / 16 * 16;
    size_t at = 0;
    auto take = [&](size_t per, int layers, uint32_t &off, uint32_t &stride) {
        stride = (uint32_t)((per + 31) / 32 * 32); off = (uint32_t)at; at += (size_t)stride * layers;
    };
    const size_t x = rows * D.d, in = 2 * x + x / 16;   // residual rows, operands, sums of squares
    take(in, D.L, a.o_xa, a.s_in); take(in, D.L, a.o_x1, a.s_in);
    a.o_pa = a.o_xa + (uint32_t)x; a.o_sa = a.o_pa + (uint32_t)x; a.o_p1 = a.o_x1 + (uint32_t)x; a.o_s1 = a.o_p1 + (uint32_t)x;
    *first = a.s_in;
    take(rows * D.qw * 3 / 2, D.L, a.o_q, a.s_q);   // three bf16 parts
    take(rows * D.kvw, D.L, a.o_kvn, a.s_kvn);
    take((size_t)R * D.qw, D.L, a.o_at, a.s_at);    // hi and lo
    take(rows * D.F, D.L, a.o_h, a.s_h);
    take((size_t)R * D.Hq * P * (D.dh + 4), P > 1 ? D.L : 0, a.o_ap, a.s_ap);
    *filled = at;
    uint32_t none;
    take((size_t)R * D.d, 1, a.o_out, none);
    return at;
}

// A wavefront takes its share of an FFN output in rounds of FR_NSD steps (5120 columns in all), one after another; from the third or fourth round on a launch per link is faster, which
// splits these columns over workgroups. 4 layers after 23 keys, launch per link / here: 896 columns, FFN of 9728 64 rows 1.05, 16 rows 1.41; FFN of 12288 64 rows 0.95, 33 rows 1.00, 32 rows
// 1.10, 16 rows 1.26; of 15360 0.88, 0.94, 1.04, 1.21; 512 columns, 12288: 0.93, 1.02, 1.02, 1.18; 256 columns, 9728: 1.06, 1.13, 1.08, 1.27; 12288: 0.92, 1.00, 0.97, 1.12; 128 columns, 16384: 0.78,
// 0.80, 0.83, 0.97; 896 columns, 20480: 0.81, 0.92, 0.96, 1.13.
static bool flow_rows_ffn(const Dims &D, int R)
{
    const int round = 32 * FR_W * FR_NSD;
    return D.F <= round * (2 + (R <= 16) + (R <= 32 && D.d >= 512));
}

constexpr size_t FR_MOST_WORDS = (size_t)1 << 29;   // 32-bit offsets in bytes

size_t flow_rows_floats(const Dims &D, int max_rows)
{
    size_t most = 0, first, filled;
    FlowRowsArgs a;
    for (int R = FLOW_MAX_ROWS + 1; R <= std::min(max_rows, FLOW_ROWS_MAX); ++R) {
        if (!flow_rows_ffn(D, R)) continue;
        for (int P = std::min(flow_rows_most(R), flow_rows_parts(D.max_seq - 1, 1)); P > 0; --P) {   // (a row's own key is in no block)
            const size_t n = flow_rows_layout(D, R, P, a, &first, &filled);
            if (n >= FR_MOST_WORDS) continue;
            most = std::max(most, n);
            break;
        }
    }
    return most;
}

// FLOW_ROWS_PARTS is what the table of parts has room for: the launch is still the faster one there. 6 layers, all rows after as many keys, a launch per link / here: 896 columns with
// 2 kv heads, 9 rows after 16 keys 206 / 117 us, 64 after 3071 374 / 307; 128-wide heads, 64 rows after 1023 326 / 235; 256 columns with 16 kv heads, 64 rows after 769 481 / 431,
// after 2312 886 / 879 (a merge per kv head and not per row: 498, 946), 9 rows after 21503 1215 / 991. Not so only where 14 to 16 rows of 1024 key columns all have more than 9000 keys
// (3900 of 128-wide heads) and both are bound by the cache: 16 rows after 12287 987 / 1012, with contexts of 1500 to 12287 809 / 636; and for 64 rows of 32 columns with two rounds
// of the FFN output (0.97 after 23 keys, 1.03 after 253).
bool flow_rows_takes(const Dims &D, int R, const int *poss, FlowRowsPlan *p)
{
    if (R <= FLOW_MAX_ROWS || R > FLOW_ROWS_MAX || !flow_rows_ffn(D, R) || !flow_rows_split(D, R, poss, p)) return false;
    FlowRowsArgs a;
    size_t first, filled;
    return flow_rows_layout(D, R, p->P, a, &first, &filled) < FR_MOST_WORDS;
}

void launch_flow_rows_setup(hipStream_t s, const Dims &D, const FlowRowsPlan &plan, const void *tok_emb, const void *gain, int R, const int *slots, const int *toks, const int *poss,
                            const int *dev_toks, int *d_slot, int *d_tok, int *d_pos, float *buf, int *ticket)
{
    FlowRowsArgs a;
    size_t first, filled;
    flow_rows_layout(D, R, plan.P, a, &first, &filled);
    FlowRowsSetup su{};
    for (int i = 0; i < R; ++i) { su.slot[i] = slots[i]; su.tok[i] = toks ? toks[i] : 0; su.pos[i] = poss[i]; }
    const uint32_t skip = (uint32_t)(first / 4), n_fill = (uint32_t)(filled / 4);   // 16-byte words
    hipLaunchKernelGGL(flow_rows_setup_kernel, dim3(R + std::min<uint32_t>(2048, (n_fill - skip + 255) / 256)), dim3(256), 0, s, su, R, d_slot, d_tok, d_pos,
                       (const bf16_t *)tok_emb, (const bf16_t *)gain, D.d, D.V, dev_toks, (char *)(buf + a.o_xa), (char *)(buf + a.o_pa), (char *)(buf + a.o_sa),
                       reinterpret_cast<uint4 *>(buf), n_fill, skip, ticket);
}

float *launch_flow_rows(hipStream_t s, const Dims &D, const FlowRowsPlan &plan, const FlowModel &m, int R, const int *poss, const int *d_slot, const int *d_pos, float *buf, int *ticket, int *given_up)
{
    FlowRowsArgs a{};
    size_t first, filled;
    a.U = plan.U; a.P = plan.P;
    const size_t n = flow_rows_layout(D, R, a.P, a, &first, &filled);
    a.wt = m.wt; a.wt_stride = m.wt_stride; a.wt_qkv = (uint32_t)m.wt_qkv; a.wt_o = (uint32_t)m.wt_o; a.wt_gu = (uint32_t)m.wt_gu; a.wt_d = (uint32_t)m.wt_d;
    a.bias = m.bias; a.bias_stride = m.bias_stride;
    for (int l = 0; l < D.L; ++l) { a.ln1[l] = (const bf16_t *)m.layers[l].ln1; a.ln2[l] = (const bf16_t *)m.layers[l].ln2; }
    a.kc = m.kc; a.vc = m.vc; a.k_layer = m.k_layer; a.v_layer = m.v_layer;
    a.slot = d_slot; a.pos = d_pos; a.rope = m.rope; a.D = D; a.inv_d = 1.0f / (float)D.d; a.R = R; a.buf = buf; a.buf_bytes = (uint32_t)(n * 4); a.ticket = ticket; a.given_up = given_up;
    int n_parts = 0, n_split = 0;
    {
        std::vector<int> rows(R);
        std::iota(rows.begin(), rows.end(), 0);
        std::stable_sort(rows.begin(), rows.end(), [&](int i, int j) { return poss[i] > poss[j]; });
        for (int c = 0; c < a.P; ++c)
            for (int r : rows)
                if (c < flow_rows_parts(poss[r], a.U)) a.part[n_parts++] = r + 256 * c;
        for (int r : rows) n_split += flow_rows_parts(poss[r], a.U) > 1;
    }
    auto go = [&](auto kern, int qu, int ou, int pair, int gu, int dr) {
        a.nG16 = (R + 15) / 16; a.nPair = (a.nG16 + pair - 1) / pair; a.uG = D.F / 8;
        a.nQ = (D.qw + 2 * D.kvw) / 16 / qu * a.nG16; a.nA = n_parts * D.Hkv; a.nM = n_split; a.nO = (D.d / 16 + ou - 1) / ou * a.nG16; a.nD = D.d / 16 * ((R + dr - 1) / dr);
        a.nG = (a.uG + gu - 1) / gu * a.nPair;
        hipLaunchKernelGGL(kern, dim3(256), dim3(64 * FR_W), 0, s, a);
    };
    auto rows = [&](auto dh) {
        constexpr int DH = decltype(dh)::value;
        // Tasks as small as keep the links of a layer, of which two or three are under way, to about the 256 workgroups: smaller ones queue, larger ones take longer each. us a step,
        // as here / smaller / larger. 16 rows after 200 to 600 keys, gate/up of 5, 4, 6 groups: 476 / 514 / 479, FFN output of 8, 16 rows: 476 / 510. 32 rows after 128 to 700,
        // gate/up of 16 rows by 8, 10 groups: 558 / 587 / 557, q|k|v of 1 group: 605, FFN output of 8 rows: 618. 64 rows after 128 to 1024, gate/up of 6, 5, 7, 8 groups: 763 / 781 /
        // 762, 784, of 16 rows by 8 groups: 888, q|k|v of 2, 6: 768 / 784, output projection of 7: 793.
        if (R <= 16) go(flow_rows_kernel<DH, 1, 2, 1, 5, 8>, 1, 2, 1, 5, 8);
        else if (R <= 32) go(flow_rows_kernel<DH, 2, 2, 2, 5, 16>, 2, 2, 2, 5, 16);
        else go(flow_rows_kernel<DH, 4, 4, 2, 6, 16>, 4, 4, 2, 6, 16);
    };
    if (D.dh == 64) rows(std::integral_constant<int, 64>{}); else rows(std::integral_constant<int, 128>{});
    return buf + a.o_out;
}

}  // namespace tr
