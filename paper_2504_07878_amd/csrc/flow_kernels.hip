// All layers of a decode step of up to 8 rows in ONE launch (bf16 models of up to 896 columns, bf16 cache).
//
// A decode step of few rows is a chain of small dependent products. As a launch each, a link costs 2.6 us before its kernel does anything, the weights of a
// link are not requested before the link before it has ended, and the chip is empty at both ends of every kernel. Here the links are TASKS of one launch:
//   * Tasks are numbered in the order of the chain: layer by layer q|k|v, attention (and a merge of its parts), output projection, gate/up, down. A workgroup takes the next number from a
//     counter, requests the task's weights (keys and values) into registers, waits for the task's input, computes, leaves its output and takes the next number. A
//     task waits only for tasks of lower numbers, which were taken before by workgroups that are running: whatever part of the grid is resident, the lowest
//     unfinished task can go on. A layer of the 0.5B-class model is 242 tasks at one row (18 q|k|v, 2 attention, 14 output projection, 152 gate/up, 56
//     FFN output), so 256 workgroups have the weights of a whole layer in flight.
//   * Outputs are handed on as data that tell by themselves that they are there: every layer has its own buffers, filled with SENT (a NaN that no product
//     stores) before the launch; a consumer loads what it needs and loads it again until no word of it is SENT. One store and one load, both past the L2 of the
//     XCD (sc1), lie between two tasks: 1.25 to 1.4 us from task to task, against 3.7 us of kernel + 2.6 us between two kernels.
//   * A task far ahead of the chain polls one word of the link before its own input, and its whole input only from then on.
// Products: v_mfma_f32_16x16x32_bf16, weights as the tiles of repack_kernel, one wavefront per 16 weight rows. The 16 columns are parts of the fp32
// activations: 3 bf16 parts (all 24 bits) of up to 4 rows, or hi and lo parts of up to 8 (as in few_kernels.hip). Attention: 3 parts of the query and of the
// probabilities (hi and middle in columns 0-7 and 8-15, lo in a second product).
// What bounds it: the hand-overs of a layer, 11 us against 4.3 us for its bytes. 0.5B-class model, a launch per link / here: 1 row after 256 keys 636 / 322 us a step,
// 7 rows in pages after 100 to 1900 keys 944 / 483, 1 to 8 rows after 16 to 2000 keys 625-926 / 319-510. Error of the hidden rows against 64 bits after 256 keys 1.4e-6 /
// 1.3e-6 (1 row), 2.5e-5 / 1.3e-6 (4 rows), 2.6e-5 / 2.4e-5 (8 rows).
#include "flow_attention.h"
#include <algorithm>
#include <type_traits>
#include <utility>

namespace tr {

constexpr int FLOW_UNITS = 4;    // groups of 16 weight rows per task
constexpr int FLOW_NS = 4;       // steps of 32 of the reduction dimension per wavefront: up to 1024 columns
constexpr int FLOW_NSD = 5;      // its steps in flight per wavefront: 5120 columns in one round

struct FlowArgs {
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
    float *buf;                       // the hand-over buffers, offsets and strides in words of 4 bytes
    uint32_t buf_bytes;
    // x1: residual rows behind the output projection of a layer, xp: what its FFN adds, FLOW_KQ sums over parts of the FFN's columns (layer - 1: the embedding and zeros);
    // q, kvn: query, new key and value; ap: attention of parts of a context; at: attention; h: FFN activations
    uint32_t o_x1, o_xp, o_q, o_kvn, o_ap, o_at, o_h, s_x1, s_xp, s_q, s_kvn, s_ap, s_at, s_h;
    int nQ, nA, nM, nO, nG, nD;       // tasks of a layer
    int uQ, uO, uG;                   // groups of 16 rows of a layer
    int *ticket, *given_up;           // next task; set when a wait was given up
};

// RC: rows the operands are laid out for (1, 2, 4, 8); a.R of them exist
template <int RC, int DH>
struct Flow : FlowAttention<Flow<RC, DH>, DH, 16, RC <= 4 ? 3 : 2, DH == 64 ? 3 : 1> {
    static constexpr int NP = RC <= 4 ? 3 : 2;            // parts
    static constexpr int NC = NP * RC;                     // columns of a stored operand: part * RC + row
    static constexpr int PV = RC == 1 ? 2 : 4;             // columns of a piece: what a lane brings of a row at a time
    static constexpr int LPR = 64 / RC, NU = (32 * FLOW_NS / PV + LPR - 1) / LPR;   // lanes per row; pieces per lane
    static constexpr int AS = 4 * FLOW_NSD + 1;            // 16-byte words of a column of a stored operand (one more: no bank conflicts)
    static constexpr int RPW = RC == 1 ? 1 : 2, NF = RC / RPW, GR = 4 / RPW;   // finishing: rows per wavefront, wavefronts, lanes that share a sum
    typedef std::conditional_t<PV == 2, u32x2, u32x4> Piece;
    // From 4 rows on a workgroup's input is up to 140 KB: past the L2 a compute unit gets 45 bytes a ns. It polls one word of each store that its share comes from,
    // then fetches the share through the L2.
    static constexpr bool FETCH = RC >= 4;
    union Lds {
        struct {
            uint4 act[FLOW_WAVES][NC * AS];                // a wavefront's operands
            f32x4 red[FLOW_WAVES][FLOW_UNITS][4][NC | 1];  // sums of a wavefront's share (odd: no bank conflicts)
            float ss[RC][FLOW_WAVES];                      // sums of squares of a wavefront's share
        } g;
        FlowAttentionLds<DH> att;
    };
    const FlowArgs &a;
    Lds &lds;
    __amdgpu_buffer_rsrc_t buf;
    int wave, lane, col, o, cidx;                          // cidx: column of the stored operand that this lane's column reads
    // finishing a task's sums: lane = (one of GR, row fm, group of 16 weight rows fu, results 4 fo .. + 3)
    int fm, fu, fo, fg;
    bool fin;

    __device__ __forceinline__ Flow(const FlowArgs &args, Lds &l) : a(args), lds(l)
    {
        buf = buffer_of(a.buf, a.buf_bytes);
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); lane = threadIdx.x & 63;
        col = lane & 15; o = lane >> 4;
        cidx = min(col / RC, NP - 1) * RC + min(col % RC, a.R - 1);
        const int row = wave * RPW + (RPW == 2 ? (lane >> 4) & 1 : 0);
        fo = lane & 3; fu = (lane >> 2) & 3; fm = min(row, a.R - 1); fg = RPW == 2 ? lane >> 5 : lane >> 4;
        fin = wave < NF && row < a.R;
    }
    __device__ __forceinline__ FlowWait wait() const { return FlowWait{a.given_up}; }
    // what the lanes of a wavefront wrote to the LDS is read by others of them: its LDS operations are carried out in order, the compiler is to leave them so
    __device__ __forceinline__ static void wave_fence() { asm volatile("" ::: "memory"); __builtin_amdgcn_wave_barrier(); }
    __device__ __forceinline__ const char *layer(int l) const { return a.wt + (size_t)l * a.wt_stride; }

    // ---- products of FLOW_UNITS groups of 16 weight rows over n32 steps of 32 columns, shared by the wavefronts
    struct Share { int s0, ns; };   // a wavefront's steps s0 .. s0 + ns - 1
    __device__ __forceinline__ Share share(int from, int n32) const
    {
        const int s0 = wave * n32 / FLOW_WAVES;
        return Share{from + s0, (wave + 1) * n32 / FLOW_WAVES - s0};
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
    // A wavefront brings its own share of the rows: pieces of PV columns, converted and turned into operands through its own part of the LDS, without a barrier.
    // Pieces past the share are zeros.
    __device__ __forceinline__ int my_row() const { return lane / LPR; }
    __device__ __forceinline__ int piece(int i) const { return lane % LPR + i * LPR; }
    __device__ __forceinline__ void put(int j, float (&v)[PV]) const
    {
        if (my_row() >= a.R || j >= 32 * FLOW_NS / PV) return;
        char *dst = reinterpret_cast<char *>(&lds.g.act[wave][my_row() * AS]) + j * PV * 2;
#pragma unroll
        for (int p = 0; p < NP; ++p, dst += RC * AS * 16) {
            if constexpr (PV == 2) *reinterpret_cast<uint32_t *>(dst) = flow_part(v[0], v[1]);
            else {
                const uint32_t w0 = flow_part(v[0], v[1]), w1 = flow_part(v[2], v[3]);
                *reinterpret_cast<uint2 *>(dst) = make_uint2(w0, w1);
            }
        }
    }
    // rows = x1 + the FLOW_KQ sums of xp (NX = 1 + FLOW_KQ), or x1 alone, times the norm's gain; the sums of squares go to lds.g.ss
    template <int NX> __device__ __forceinline__ void stage_norm(uint32_t x1, uint32_t xp, const bf16_t *gain, Share sh, uint32_t gate) const
    {
        const int row = my_row(), K = a.D.d;
        uint32_t g[NU][PV / 2];
        FlowPiece<Piece, NU, NX> x;   // set 0: x1, the others: xp
#pragma unroll
        for (int q = 1; q < NX; ++q) x.set[q] = (xp + (q - 1) * a.R * K - x1) * 4;
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            const int k = 32 * sh.s0 + PV * piece(i);
            const bool in = PV * piece(i) < 32 * sh.ns && row < a.R;
#pragma unroll
            for (int e = 0; e < PV / 2; ++e) g[i][e] = in ? reinterpret_cast<const uint32_t *>(gain + k)[e] : 0;
            x.off[i] = in ? (x1 + row * K + k) * 4 : BUFFER_NOWHERE;
        }
        flow_gate(buf, gate * 4, wait());
        if constexpr (FETCH) {   // stores of x1 and xp: two rows, 64 columns
            constexpr int PER = 3 * RC / 2;
            const int q = lane / PER, first = 32 * sh.s0, k = max(first, min((first / 64 + lane % 3) * 64, 32 * (sh.s0 + max(sh.ns, 1) - 1))), r2 = min(lane % PER / 3 * 2, a.R - 1);
            FlowPiece<uint32_t, 1> sample;
            sample.off[0] = q >= NX ? BUFFER_NOWHERE : ((q == 0 ? x1 + r2 * K : xp + ((q - 1) * a.R + r2) * K) + k) * 4;
            flow_poll(buf, wait(), sample);
            flow_fetch(buf, wait(), x);
        } else flow_poll(buf, wait(), x);
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            float v[PV];
#pragma unroll
            for (int e = 0; e < PV; ++e) {
                v[e] = __uint_as_float(x.v[0][i][e]);
#pragma unroll
                for (int q = 1; q < NX; ++q) v[e] += __uint_as_float(x.v[q][i][e]);
                ss = fmaf(v[e], v[e], ss);
                v[e] *= __uint_as_float(e & 1 ? g[i][e / 2] & 0xffff0000u : g[i][e / 2] << 16);
            }
            put(piece(i), v);
        }
        wave_fence();
        ss = flow_sum<LPR>(ss);
        if (lane % LPR == 0) lds.g.ss[row][wave] = ss;
    }
    __device__ __forceinline__ float rstd(float inv_d, float eps) const   // of row fm (after the barrier in product)
    {
        const f32x4 t = *reinterpret_cast<const f32x4 *>(&lds.g.ss[fm][0]) + *reinterpret_cast<const f32x4 *>(&lds.g.ss[fm][4]);
        return flow_rsqrt(fmaf((t.x + t.y) + (t.z + t.w), inv_d, eps));   // (0 where the sum overflows, as in the other kernels)
    }
    template <int N> __device__ __forceinline__ void accumulate(f32x4 (&c)[FLOW_UNITS], const uint4 (&w)[FLOW_UNITS][N]) const
    {
        const uint4 *b = &lds.g.act[wave][cidx * AS + o];
        uint4 x[N];
#pragma unroll
        for (int s = 0; s < N; ++s) x[s] = b[4 * s];
#pragma unroll
        for (int s = 0; s < N; ++s)
#pragma unroll
            for (int u = 0; u < FLOW_UNITS; ++u) c[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(flow_bf(w[u][s]), flow_bf(x[s]), c[u], 0, 0, 0);
    }
    // the sums over wavefronts and parts, in all lanes that share a sum (only wavefronts below NF)
    __device__ __forceinline__ f32x4 finish(const f32x4 (&c)[FLOW_UNITS]) const
    {
        if (col < NC)
#pragma unroll
            for (int u = 0; u < FLOW_UNITS; ++u) lds.g.red[wave][u][o][col] = c[u];
        __syncthreads();
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (wave < NF) {
#pragma unroll
            for (int q = 0; q < FLOW_WAVES / GR; ++q)
#pragma unroll
                for (int p = 0; p < NP; ++p) v += lds.g.red[q * GR + fg][fu][fo][p * RC + fm];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = GR == 4 ? flow_sum4(v[e]) : flow_sum2(v[e]);
        }
        return v;
    }
    __device__ __forceinline__ static void clear(f32x4 (&c)[FLOW_UNITS])
    {
#pragma unroll
        for (int u = 0; u < FLOW_UNITS; ++u) c[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // first of the 4 consecutive features that results 4 q .. + 3 of 16 rows of a matrix are (tile_feature)
    __device__ __forceinline__ static int feature4(int unit, int q) { return (unit >> 1) * 32 + 16 * (unit & 1) + 8 * (q & 1) + 4 * (q >> 1); }

    // ---- tasks
    __device__ __forceinline__ void qkv(int l, int task) const
    {
        const int u0 = task * FLOW_UNITS, n32 = a.D.d / 32, unit = min(u0 + fu, a.uQ - 1);
        const Share sh = share(0, n32);
        uint4 w[FLOW_UNITS][FLOW_NS];
#pragma unroll
        for (int u = 0; u < FLOW_UNITS; ++u) weights(w[u], layer(l) + a.wt_qkv, group_off(min(u0 + u, a.uQ - 1), n32), sh);
        const bool on = fin && u0 + fu < a.uQ && fg == 0;
        const int half = DH / 2, Hq = flow_now(a.D.Hq), Hkv = flow_now(a.D.Hkv);
        const int f = feature4(unit, fo), tph = DH >> 5, hh = (f >> 5) / tph, j = ((f >> 5) % tph) * 16 + ((f & 31) >> 1);   // rotary pairs j, j + 1 of head hh
        const int pos = a.pos[fm], slot = a.slot[fm];
        const float *bias = a.bias + l * a.bias_stride + hh * DH + j;
        const float2 ba = *reinterpret_cast<const float2 *>(bias), bb = *reinterpret_cast<const float2 *>(bias + half);
        const float4 cs = *reinterpret_cast<const float4 *>(a.rope + (size_t)pos * half + j);
        const KvPlace at = kv_place(a.D, slot, pos);
        const bool key = hh < Hq + Hkv;
        const int head = key ? hh - Hq : hh - Hq - Hkv;
        bf16_t *cache = key ? reinterpret_cast<bf16_t *>(a.kc + (size_t)l * a.k_layer) + k_offset(a.D, at.unit, max(head, 0), at.pos, j)
                            : reinterpret_cast<bf16_t *>(a.vc + (size_t)l * a.v_layer) + v_offset(a.D, at.unit, max(head, 0), at.pos, j);
        const uint32_t at_q = (a.o_q + l * a.s_q + (fm * Hq + hh) * (3 * DH / 2) + j / 2) * 4;
        const uint32_t at_n = (a.o_kvn + l * a.s_kvn + ((fm * 2 + (key ? 0 : 1)) * a.D.kvw + head * DH + j) / 2) * 4;
        const float inv_d = flow_now(a.inv_d), eps = flow_now(a.D.eps);
        stage_norm<1 + FLOW_KQ>(a.o_x1 + l * a.s_x1, a.o_xp + l * a.s_xp, a.ln1[l], sh, l > 0 ? a.o_h + (l - 1) * a.s_h : a.o_x1);
        f32x4 c[FLOW_UNITS];
        clear(c);
        accumulate(c, w);
        const f32x4 v = finish(c);
        if (!on) return;
        const float rs = rstd(inv_d, eps);
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
                flow_store_pair(buf, at_q + p * DH * 2, wl);
                flow_store_pair(buf, at_q + p * DH * 2 + half * 2, wh);
            }
            return;
        }
        const uint32_t plo = flow_part(lo0, lo1), phi = flow_part(hi0, hi1);
        flow_store_pair(buf, at_n, plo);   // the values that the cache will hold, for this step's attention
        flow_store_pair(buf, at_n + half * 2, phi);
        if (key) {
            *reinterpret_cast<uint32_t *>(cache) = plo;
            *reinterpret_cast<uint32_t *>(cache + half) = phi;
        } else {
            cache[0] = (bf16_t)plo; cache[32] = (bf16_t)(plo >> 16);
            cache[half * 32] = (bf16_t)phi; cache[half * 32 + 32] = (bf16_t)(phi >> 16);
        }
    }

    // ---- attention: where its input and output lie (bytes)
    __device__ __forceinline__ uint32_t q_at(int l, int r, int head) const { return (a.o_q + l * a.s_q + (r * a.D.Hq + head) * (3 * DH / 2)) * 4; }
    __device__ __forceinline__ uint32_t kvn_at(int l, int r, int g) const { return (a.o_kvn + l * a.s_kvn + (r * 2 * a.D.kvw + g * DH) / 2) * 4; }
    __device__ __forceinline__ uint32_t vn_behind() const { return a.D.kvw * 2; }
    __device__ __forceinline__ uint32_t plane() const { return RC * a.D.qw * 2; }
    __device__ __forceinline__ uint32_t attention_gate(int l, int) const { return (a.o_xp + l * a.s_xp) * 4; }
    __device__ __forceinline__ uint32_t merge_gate(int l, int) const { return (a.o_kvn + l * a.s_kvn) * 4; }
    __device__ __forceinline__ uint32_t out_of(int l, int r, int g) const { return (a.o_at + l * a.s_at) * 4 + (r * a.D.qw + g * a.D.G * DH) * 2; }

    // A wavefront's share of rows that are operand parts already, K columns a plane: NL pieces of 8 columns per lane, to its part of the LDS
    static constexpr int NL = (NC * FLOW_NSD * 4 + 63) / 64;
    template <class... More> __device__ __forceinline__ void stage_parts(uint32_t base, uint32_t K, Share sh, uint32_t sample_at, More &...more) const
    {
        FlowPiece<u32x4, NL> x;
#pragma unroll
        for (int i = 0; i < NL; ++i) {   // column cc of the operand, columns 8 k8 .. of the share; past it: zeros
            const int cc = (i * 64 + lane) / (FLOW_NSD * 4), k8 = (i * 64 + lane) % (FLOW_NSD * 4);
            x.off[i] = cc < NC && cc % RC < a.R && k8 < 4 * sh.ns ? base + (cc * K + sh.s0 * 32 + 8 * k8) * 2 : BUFFER_NOWHERE;
        }
        if constexpr (FETCH) {
            FlowPiece<uint32_t, 1> sample;
            sample.off[0] = sample_at;
            flow_poll(buf, wait(), sample);
            flow_fetch(buf, wait(), x, more...);
        } else flow_poll(buf, wait(), x, more...);
        wave_fence();
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int cc = (i * 64 + lane) / (FLOW_NSD * 4), k8 = (i * 64 + lane) % (FLOW_NSD * 4);
            if (cc < NC) lds.g.act[wave][cc * AS + k8] = __builtin_bit_cast(uint4, x.v[0][i]);
        }
        wave_fence();
    }

    // x1 = x + Wo . attention
    __device__ __forceinline__ void oproj(int l, int task) const
    {
        const int u0 = task * FLOW_UNITS, n32 = a.D.qw / 32, unit = min(u0 + fu, a.uO - 1);
        const Share sh = share(0, n32);
        uint4 w[FLOW_UNITS][FLOW_NS];
#pragma unroll
        for (int u = 0; u < FLOW_UNITS; ++u) weights(w[u], layer(l) + a.wt_o, group_off(min(u0 + u, a.uO - 1), n32), sh);
        const bool on = fin && u0 + fu < a.uO && fg == 0;
        FlowPiece<u32x4, 1, 1 + FLOW_KQ> old;   // x1 and the sums of xp
        const uint32_t at = feature4(unit, fo), out = (a.o_x1 + (l + 1) * a.s_x1 + fm * a.D.d + at) * 4;
        old.off[0] = on ? (a.o_x1 + l * a.s_x1 + fm * a.D.d + at) * 4 : BUFFER_NOWHERE;
#pragma unroll
        for (int q = 0; q < FLOW_KQ; ++q) old.set[1 + q] = (a.o_xp + l * a.s_xp + q * a.R * a.D.d - a.o_x1 - l * a.s_x1) * 4;
        const uint32_t base = (a.o_at + l * a.s_at) * 4;
        // one word of the last part of each row and head of the share (at most three heads)
        const int first = 32 * sh.s0, last = 32 * (sh.s0 + max(sh.ns, 1)) - 1, r = lane / 3, k = max(first, min((first / DH + lane % 3) * DH, last)) & ~1;
        const uint32_t sample = r < a.R ? base + (((NP - 1) * RC + r) * a.D.qw + k) * 2 : BUFFER_NOWHERE;
        flow_gate(buf, (a.o_q + l * a.s_q) * 4, wait());
        stage_parts(base, a.D.qw, sh, sample, old);
        f32x4 c[FLOW_UNITS];
        clear(c);
        accumulate(c, w);
        f32x4 v = finish(c);
        if (!on) return;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float x = __uint_as_float(old.v[0][0][e]);
#pragma unroll
            for (int q = 0; q < FLOW_KQ; ++q) x += __uint_as_float(old.v[1 + q][0][e]);
            v[e] += x;
        }
        flow_store(buf, out, v);
    }

    // 8 gate rows and the 8 up rows of the same features in one operand
    __device__ __forceinline__ void gateup(int l, int task) const
    {
        const int u0 = task * FLOW_UNITS, n32 = a.D.d / 32, unit = u0 + fu;
        const Share sh = share(0, n32);
        uint4 w[FLOW_UNITS][FLOW_NS];
#pragma unroll
        for (int u = 0; u < FLOW_UNITS; ++u) {   // features 8 t .. + 7 of gate and of up
            const int t = min(u0 + u, a.uG - 1);
            weights(w[u], layer(l) + a.wt_gu, row_off(2 * (t >> 2) + (col >> 3), 16 * ((t & 3) >> 1) + 4 * (t & 1) + 8 * ((col >> 2) & 1) + (col & 3), n32), sh);
        }
        const bool on = fin && unit < a.uG && fo < 2;
        const uint32_t F = flow_now(a.D.F), out = (a.o_h + l * a.s_h) * 4 + (fm * F + 8 * unit + 4 * fo) * 2;
        const float inv_d = flow_now(a.inv_d), eps = flow_now(a.D.eps);
        stage_norm<1>(a.o_x1 + (l + 1) * a.s_x1, 0, a.ln2[l], sh, a.o_at + l * a.s_at);
        f32x4 c[FLOW_UNITS];
        clear(c);
        accumulate(c, w);
        const f32x4 v = finish(c);
        if (wave >= NF) return;
        const float rs = rstd(inv_d, eps);
        float t[4], h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = v[e] * rs;
        flow_silu(t, h);
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] *= flow_dpp<0x4e>(v[e]) * rs;   // gate rows: fo 0 and 1, up rows: 2 lanes on
        // each of the lanes that share a sum stores a part
        uint32_t w0[NP], w1[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) { w0[p] = flow_part(h[0], h[1]); w1[p] = flow_part(h[2], h[3]); }
        if constexpr (GR >= NP) {
            const uint32_t s0 = fg == 0 ? w0[0] : fg == 1 ? w0[1] : w0[NP - 1], s1 = fg == 0 ? w1[0] : fg == 1 ? w1[1] : w1[NP - 1];
            if (on && fg < NP) flow_store_pair(buf, out + fg * RC * F * 2, s0, s1);
        } else {
            const uint32_t s0 = fg == 0 ? w0[0] : w0[1], s1 = fg == 0 ? w1[0] : w1[1];
            if (on) flow_store_pair(buf, out + fg * RC * F * 2, s0, s1);
            if (on && fg == 0) flow_store_pair(buf, out + 2 * RC * F * 2, w0[NP - 1], w1[NP - 1]);
        }
    }

    // FLOW_UNITS groups of 16 rows of the FFN output over one of FLOW_KQ parts of the FFN's columns
    __device__ __forceinline__ void down(int l, int task) const
    {
        const int u0 = task / FLOW_KQ * FLOW_UNITS, kq = task % FLOW_KQ, n32 = a.D.F / 32, unit = min(u0 + fu, a.uO - 1);
        const int from = kq * n32 / FLOW_KQ, to = (kq + 1) * n32 / FLOW_KQ;
        Share sh = share(from, to - from);
        sh.s0 = min(sh.s0, n32 - 1);
        const char *base = layer(l) + a.wt_d;
        uint32_t woff[FLOW_UNITS];
        uint4 w[FLOW_UNITS][FLOW_NSD];
#pragma unroll
        for (int u = 0; u < FLOW_UNITS; ++u) { woff[u] = group_off(min(u0 + u, a.uO - 1), n32); weights(w[u], base, woff[u], sh); }
        const bool on = fin && u0 + fu < a.uO && fg == 0;
        const uint32_t out = (a.o_xp + (l + 1) * a.s_xp + (kq * a.R + fm) * a.D.d + feature4(unit, fo)) * 4;
        const uint32_t hbase = (a.o_h + l * a.s_h) * 4;
        f32x4 c[FLOW_UNITS];
        clear(c);
        flow_gate(buf, (a.o_x1 + (l + 1) * a.s_x1) * 4, wait());
        for (int done = 0; done < sh.ns; done += FLOW_NSD) {   // (one round up to 5120 FFN columns)
            if (done > 0)
#pragma unroll
                for (int u = 0; u < FLOW_UNITS; ++u) weights(w[u], base, woff[u], Share{sh.s0 + done, sh.ns - done});
            // one word of the last part of each two rows and 32 columns
            const int t = lane % FLOW_NSD, r2 = lane / FLOW_NSD * 2;
            const uint32_t sample = r2 < a.R && t < sh.ns - done ? hbase + (((NP - 1) * RC + r2) * a.D.F + (sh.s0 + done + t) * 32) * 2 : BUFFER_NOWHERE;
            stage_parts(hbase, a.D.F, Share{sh.s0 + done, min(sh.ns - done, FLOW_NSD)}, sample);
            accumulate(c, w);
        }
        const f32x4 v = finish(c);
        if (on) flow_store(buf, out, v);
    }
};

template <int RC, int DH>
__global__ __launch_bounds__(64 * FLOW_WAVES, 2) void flow_kernel(FlowArgs args)
{
    __shared__ typename Flow<RC, DH>::Lds lds;
    __shared__ int s_task[2];
    if (threadIdx.x == 0) s_task[0] = atomicAdd(args.ticket, 1);
    __syncthreads();
    for (int it = 0;; it ^= 1) {
        const int t = __builtin_amdgcn_readfirstlane(s_task[it]);
        // (the arguments are read again for every task: kept in registers over the loop they would not fit)
        auto kernarg = __builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(kernarg));
        const FlowArgs &a = *(const FlowArgs *)kernarg;
        const int per_layer = a.nQ + a.nA + a.nM + a.nO + a.nG + a.nD;
        if (t >= per_layer * a.D.L) break;   // uniform over the workgroup
        Flow<RC, DH> f(a, lds);
        const int l = t / per_layer;
        int i = t - l * per_layer;
        if (i < a.nQ) f.qkv(l, i);
        else if ((i -= a.nQ) < a.nA) f.attention(l, i / (a.D.Hkv * a.P), (i / a.P) % a.D.Hkv, i % a.P);
        else if ((i -= a.nA) < a.nM) { f.merge(l, i / a.D.Hkv, i % a.D.Hkv * a.D.G, a.D.G); __syncthreads(); }   // (not all of its wavefronts have something to wait for)
        else if ((i -= a.nM) < a.nO) f.oproj(l, i);
        else if ((i -= a.nO) < a.nG) f.gateup(l, i);
        else f.down(l, i - a.nG);
        // the next task is asked for when this one is over but for its last stores, by a wavefront that has none of these: a number held during a wait would be a
        // task nobody has begun
        if (threadIdx.x == 64 * (FLOW_WAVES - 1)) s_task[it ^ 1] = atomicAdd(a.ticket, 1);
        __syncthreads();   // also: the LDS is free for the next task
    }
}

// ------------------------------------------------------------------ launches

// Blocks of 32 cached keys per wavefront (U), and parts that gives the longest row. One part as long as the registers hold its blocks: a block more costs 11 us
// a step of the 0.5B-class model, parts and their merge 24 (one row) to 38 (8 rows). Past that as few blocks as make 6 parts (1 / 2 / 3 blocks: one row after 1000
// keys 351 / 362 / 371 us, after 2000 keys 365 / 364 / 374; 8 rows 476 / 483 / 492 and 498 / 495 / 503).
static void flow_split(const Dims &D, int max_ctx, int *U, int *P)
{
    const int umax = D.dh == 64 ? 3 : 1, blocks = std::max(1, (max_ctx - 1 + 31) / 32);
    auto per = [&](int parts) { return (blocks + FLOW_WAVES * parts - 1) / (FLOW_WAVES * parts); };
    *U = per(1) <= umax ? per(1) : std::min(umax, per(6));
    *P = (blocks + FLOW_WAVES * *U - 1) / (FLOW_WAVES * *U);
}

static int flow_row_class(int R) { return R <= 2 ? R : R <= 4 ? 4 : 8; }

static size_t flow_layout(const Dims &D, int R, int P, FlowArgs &a)
{
    const int RC = flow_row_class(R), NC = RC * (RC <= 4 ? 3 : 2);
    size_t at = 0;
    auto take = [&](size_t per, int layers, uint32_t &off, uint32_t &stride) {
        stride = (uint32_t)((per + 31) / 32 * 32); off = (uint32_t)at; at += (size_t)stride * layers;
    };
    take((size_t)R * D.d, D.L + 1, a.o_x1, a.s_x1);   // the first of these two are the embedding and zeros
    take((size_t)R * D.d * FLOW_KQ, D.L + 1, a.o_xp, a.s_xp);
    take((size_t)R * D.qw * 3 / 2, D.L, a.o_q, a.s_q);   // three bf16 parts
    take((size_t)R * D.kvw, D.L, a.o_kvn, a.s_kvn);
    take((size_t)D.qw * NC / 2, D.L, a.o_at, a.s_at);   // bf16 parts, column after column
    take((size_t)D.F * NC / 2, D.L, a.o_h, a.s_h);   // bf16 parts, column after column
    at = (at + 31) / 32 * 32;
    a.s_ap = (uint32_t)((size_t)R * D.Hq * P * (D.dh + 4)); a.o_ap = (uint32_t)at; at += (size_t)a.s_ap * D.L;
    return at;
}

size_t flow_floats(const Dims &D, int max_rows)
{
    size_t most = 0;
    FlowArgs a;
    for (int R = 1; R <= std::min(max_rows, FLOW_MAX_ROWS); ++R) most = std::max(most, flow_layout(D, R, FLOW_MAX_PARTS, a));
    return most;
}

bool flow_supported(const Dims &D, int wdt, int kdt)
{
    return wdt == DT_BF16 && kdt == DT_BF16 && D.L <= FLOW_MAX_LAYERS && D.d % 32 == 0 && D.d <= 32 * FLOW_NS * FLOW_WAVES && D.qw % 32 == 0 && D.qw <= 32 * FLOW_NS * FLOW_WAVES && D.F % 32 == 0 &&
           (D.dh == 64 || D.dh == 128) && D.G <= 8 && (size_t)D.F * D.d < (size_t)1 << 30 &&
           flow_floats(D, FLOW_MAX_ROWS) < (size_t)1 << 29;
}

// FLOW_MAX_PARTS is what the buffers are sized for, 12288 cached keys (4096 of 128-wide heads): the launch is still the faster one there. 6 layers of 896 columns, 1 / 2 /
// 4 / 8 rows after 12200 keys: a launch per link 175 / 221 / 267 / 293 us, here 110 / 122 / 142 / 182; 128-wide heads (768 columns) after 4000 keys 184 / 208 / 242 / 269 and
// 106 / 114 / 132 / 161; the closest, 3 layers of 256 columns with 16 kv heads, 8 rows after 12200 keys, 298 and 272.
bool flow_takes(const Dims &D, int R, int max_ctx)
{
    int U, P;
    flow_split(D, max_ctx, &U, &P);
    return R <= FLOW_MAX_ROWS && P <= FLOW_MAX_PARTS;
}

void launch_flow_setup(hipStream_t s, const Dims &D, const void *tok_emb, int R, int max_ctx, const int *slots, const int *toks, const int *poss, const int *dev_toks,
                       int *d_slot, int *d_tok, int *d_pos, float *buf, int *ticket)
{
    FlowArgs a{};
    flow_split(D, max_ctx, &a.U, &a.P);
    const size_t n = flow_layout(D, R, a.P, a);
    flow_setup(s, flow_tables(R, slots, toks, poss), R, d_slot, d_tok, d_pos, (const bf16_t *)tok_emb, D, dev_toks, buf, n, a.s_x1, a.o_xp, a.o_xp + a.s_xp, ticket);
}

float *launch_flow(hipStream_t s, const Dims &D, const FlowModel &m, int R, int max_ctx, const int *d_slot, const int *d_pos, float *buf, int *ticket, int *given_up, float **partials)
{
    FlowArgs a{};
    flow_split(D, max_ctx, &a.U, &a.P);
    const size_t n = flow_layout(D, R, a.P, a);
    a.wt = m.wt; a.wt_stride = m.wt_stride; a.wt_qkv = (uint32_t)m.wt_qkv; a.wt_o = (uint32_t)m.wt_o; a.wt_gu = (uint32_t)m.wt_gu; a.wt_d = (uint32_t)m.wt_d;
    a.bias = m.bias; a.bias_stride = m.bias_stride;
    for (int l = 0; l < D.L; ++l) { a.ln1[l] = (const bf16_t *)m.layers[l].ln1; a.ln2[l] = (const bf16_t *)m.layers[l].ln2; }
    a.kc = m.kc; a.vc = m.vc; a.k_layer = m.k_layer; a.v_layer = m.v_layer;
    a.slot = d_slot; a.pos = d_pos; a.rope = m.rope; a.D = D; a.inv_d = 1.0f / (float)D.d; a.R = R; a.buf = buf; a.buf_bytes = (uint32_t)(n * 4); a.ticket = ticket; a.given_up = given_up;
    a.uQ = (D.qw + 2 * D.kvw) / 16; a.uO = D.d / 16; a.uG = D.F / 8;
    auto tasks = [](int units) { return (units + FLOW_UNITS - 1) / FLOW_UNITS; };
    a.nQ = tasks(a.uQ); a.nA = R * D.Hkv * a.P; a.nM = a.P > 1 ? R * D.Hkv : 0; a.nO = tasks(a.uO); a.nG = tasks(a.uG); a.nD = a.nO * FLOW_KQ;
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(256), dim3(64 * FLOW_WAVES), 0, s, a); };
    auto rows = [&](auto dh) {
        constexpr int DH = decltype(dh)::value;
        switch (flow_row_class(R)) {
        case 1: go(flow_kernel<1, DH>); break;
        case 2: go(flow_kernel<2, DH>); break;
        case 4: go(flow_kernel<4, DH>); break;
        default: go(flow_kernel<8, DH>);
        }
    };
    if (D.dh == 64) rows(std::integral_constant<int, 64>{}); else rows(std::integral_constant<int, 128>{});
    *partials = buf + a.o_xp + (size_t)a.s_xp * D.L;
    return buf + a.o_x1 + (size_t)a.s_x1 * D.L;
}

}  // namespace tr
