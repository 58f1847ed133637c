// A decode step of up to 4 rows of an fp32 model (fp32 cache) in ONE launch: all layers, the LM head's slices and the router's first layer.
//
// What bounds such a step is the number of dependent links, five a layer, not bytes: a launch each, they take 3 to 5 us of kernel and 1 between two kernels. The
// links are tasks as in flow_kernels.hip (numbers from a counter, weights requested before the input is waited for, outputs handed on as words that are no longer
// SENT), with products in plain fp32: a wavefront multiplies FLOW32_UNIT weight rows by the activation rows, each of its lanes 4 columns of every 256, fetches the
// activation rows by itself (no LDS, no barrier before the product) and adds up its lanes' sums. The sums of the 8 wavefronts meet in LDS, where a few threads
// finish the task, so that its output leaves in runs of 64 bytes or more.
// Whole steps, a launch per link / here: 2 layers of 256 columns (FFN 1024, 4096 words), 2 rows, 16 / 190 / 1000 / 2000 cached keys 57 / 61 / 66 / 68 us -> 30 / 31 /
// 42 / 57, 4 rows 78 / 81 / 88 / 88 -> 34 / 35 / 47 / 62; 12 layers of 512 columns (FFN 2048) 2 rows 316 -> 156 at 190 keys; 24 layers of 1024 columns (FFN 4096), 1 / 4
// rows 800 / 1255 -> 400 / 565. In the first of these the launch takes 22 us: ten hand-overs of 1.4 us, the products and sums between them, the first numbers.
#include "flow_common.h"

namespace tr {

constexpr int FLOW32_UNIT = 4;   // weight rows per wavefront: two rotary pairs, two gate/up pairs, or 4 output features
constexpr int FLOW32_STEPS = 8;  // steps of 256 / head width keys per wavefront in flight

struct Flow32Args {
    LayerW layers[FLOW32_MAX_LAYERS];
    float *kc, *vc; size_t k_layer, v_layer;   // floats from layer to layer
    const int *slot, *pos;
    const float2 *rope;
    Dims D;
    float inv_d;
    int R, wk;                        // rows; wavefronts that share the columns of the FFN output
    float *buf;                       // the hand-over buffers, offsets and strides in words: residual rows before a layer (and after the last) and behind its output
    uint32_t buf_bytes;               // projection, query, new key and value, attention, FFN activations
    uint32_t o_x, o_x1, o_q, o_kvn, o_at, o_h, s_x, s_x1, s_q, s_kvn, s_at, s_h;
    int nQ, nA, nO, nG, nD;           // tasks of a layer
    int nV, nR;                       // tasks of the LM head and of the router's first layer
    const float *head, *final_norm, *r_w1;
    float *hn, *hidden, *logits, *r1; // tail: normalised rows, the exposed ones, logits (or NULL), sums of the router's first layer [R][rh]
    float4 *part;                     // [nV][R]: maximum, its lowest index, sum of exponentials
    int tap;
    int *ticket, *given_up;
};

// RC: rows the registers are laid out for (1, 2, 4); KC: 256-column pieces per row (1, 4); DH: head width (64, 128)
template <int RC, int KC, int DH>
struct Flow32 {
    static constexpr int U = FLOW32_UNIT, N = U * RC, HALF = DH / 2;
    static constexpr int LK = DH / 4, KPW = 64 / LK, NS = FLOW32_STEPS;   // lanes per key, keys per step of a wavefront
    union Lds {
        struct { float red[FLOW_WAVES][N], ss[RC]; } g;
        struct { float o[FLOW_WAVES][DH], m[FLOW_WAVES], l[FLOW_WAVES]; } att;
    };
    struct Weights { uint4 v[U][KC]; };
    typedef FlowPiece<u32x4, RC * KC> Rows4;
    const Flow32Args &a;
    Lds &lds;
    __amdgpu_buffer_rsrc_t buf;
    int wave, lane;

    __device__ __forceinline__ Flow32(const Flow32Args &args, Lds &l) : a(args), lds(l)
    {
        buf = buffer_of(a.buf, a.buf_bytes);
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); lane = threadIdx.x & 63;
    }
    __device__ __forceinline__ FlowWait wait() const { return FlowWait{a.given_up}; }
    // A task far ahead of the chain: one wavefront waits for a word of the link before its own input. Tasks take different ones of n runs of 32 words.
    __device__ __forceinline__ void gate(uint32_t words, int n, int task) const
    {
        if (wave == 0) flow_gate(buf, (words + (uint32_t)(task % max(n, 1)) * 32) * 4, wait());
        __syncthreads();
    }
    __device__ __forceinline__ int column(int c) const { return c * 256 + lane * 4; }
    // row `row` of W[rows][K], this lane's columns from k0 on (past the row or the matrix: zeros)
    __device__ __forceinline__ void request(uint4 (&w)[KC], const void *W, int row, int rows, int K, int k0 = 0) const
    {
        const __amdgpu_buffer_rsrc_t b = buffer_of(W, (uint32_t)rows * (uint32_t)K * 4);
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            const int k = k0 + column(c);
            w[c] = buffer_load16(b, row < rows && k < K ? (uint32_t)row * K * 4 + k * 4 : BUFFER_NOWHERE, 0);
        }
    }
    __device__ __forceinline__ void gains(uint4 (&g)[KC], const void *gain) const { request(g, gain, 0, 1, a.D.d); }
    __device__ __forceinline__ void place(Rows4 &x, uint32_t words, int K, int k0 = 0) const
    {
#pragma unroll
        for (int r = 0; r < RC; ++r)
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                const int k = k0 + column(c);
                x.off[r * KC + c] = r < a.R && k < K ? (words + (uint32_t)(r * K + k)) * 4 : BUFFER_NOWHERE;
            }
    }
    // the rows times the norm's gain; the sums of their squares go to lds.g.ss (every wavefront has them)
    __device__ __forceinline__ void norm(Rows4 &x, const uint4 (&g)[KC]) const
    {
        const bool first = threadIdx.x == 0;
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                u32x4 &p = x.v[0][r * KC + c];
                const uint32_t ge[4] = {g[c].x, g[c].y, g[c].z, g[c].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v = __uint_as_float(p[e]);
                    s = fmaf(v, v, s);
                    p[e] = __float_as_uint(v * __uint_as_float(ge[e]));
                }
            }
            s = flow_sum<64>(s);
            if (first) lds.g.ss[r] = s;
        }
    }
    // this wavefront's U x RC sums to lds.g.red[wave][weight row * RC + activation row]: halves, then rows of 16 lanes, take half of the sums each
    __device__ __forceinline__ void dots(const Weights &w, const Rows4 &x) const
    {
        float v[N];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < RC; ++r) {
                float s = 0.f;
#pragma unroll
                for (int c = 0; c < KC; ++c) {
                    const uint32_t we[4] = {w.v[u][c].x, w.v[u][c].y, w.v[u][c].z, w.v[u][c].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) s = fmaf(__uint_as_float(we[e]), __uint_as_float(x.v[0][r * KC + c][e]), s);
                }
                v[u * RC + r] = s;
            }
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + N / 2]), false, false);
            v[i] = __uint_as_float(t[0]) + __uint_as_float(t[1]);
        }
#pragma unroll
        for (int i = 0; i < N / 4; ++i) {
            const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + N / 4]), false, false);
            v[i] = flow_sum<16>(__uint_as_float(t[0]) + __uint_as_float(t[1]));
        }
        if ((lane & 15) == 0)
#pragma unroll
            for (int i = 0; i < N / 4; ++i) lds.g.red[wave][i + N / 2 * (lane >> 5) + N / 4 * (lane >> 4 & 1)] = v[i];
    }
    __device__ __forceinline__ float rstd(int r) const { return 1.0f / sqrtf(lds.g.ss[r] * a.inv_d + a.D.eps); }

    // ---- links
    // 16 rotary pairs of one head: wavefront w has the pairs 2 w and 2 w + 1, thread 16 r + p finishes pair p of row r
    __device__ __forceinline__ void qkv(int l, int task) const
    {
        const LayerW &lw = a.layers[l];
        const int d = a.D.d, Hq = a.D.Hq, Hkv = a.D.Hkv, pair0 = task * 16, hh = pair0 / HALF, j0 = pair0 - hh * HALF;
        const bool isq = hh < Hq, isk = !isq && hh < Hq + Hkv;
        const int head = isq ? hh : isk ? hh - Hq : hh - Hq - Hkv;
        const void *W = isq ? lw.wq : isk ? lw.wk : lw.wv;
        const float *bias = (const float *)(isq ? lw.bq : isk ? lw.bk : lw.bv);
        Weights w;
#pragma unroll
        for (int u = 0; u < U; ++u) request(w.v[u], W, head * DH + j0 + 2 * wave + (u >> 1) + (u & 1) * HALF, (isq ? Hq : Hkv) * DH, d);
        uint4 g[KC];
        gains(g, lw.ln1);
        const int r = min((int)threadIdx.x >> 4, a.R - 1), j = j0 + (threadIdx.x & 15), n1 = head * DH + j;
        const bool fin = (int)threadIdx.x >> 4 < a.R;
        const int pos = a.pos[r];
        const int slot = a.slot[r];
        const float2 cs = a.rope[(size_t)pos * HALF + j];
        const float b1 = bias ? bias[n1] : 0.f, b2 = bias ? bias[n1 + HALF] : 0.f;
        Rows4 x;
        place(x, a.o_x + l * a.s_x, d);
        if (l > 0) gate(a.o_h + (l - 1) * a.s_h, a.D.F / 32, task);
        flow_poll(buf, wait(), x);
        norm(x, g);
        dots(w, x);
        __syncthreads();
        if (!fin) return;
        const int p = threadIdx.x & 15, u = (p & 1) * 2;
        const float rs = rstd(r);
        float y1 = lds.g.red[p >> 1][u * RC + r] * rs + b1, y2 = lds.g.red[p >> 1][(u + 1) * RC + r] * rs + b2;
        if (isq || isk) {
            const float t1 = y1 * cs.x - y2 * cs.y, t2 = y2 * cs.x + y1 * cs.y;
            y1 = t1; y2 = t2;
        }
        const uint32_t out = isq ? (a.o_q + l * a.s_q + r * a.D.qw + n1) * 4 : (a.o_kvn + l * a.s_kvn + (r * 2 + (isk ? 0 : 1)) * a.D.kvw + n1) * 4;
        flow_store(buf, out, y1);
        flow_store(buf, out + HALF * 4, y2);
        if (isq) return;
        float *dst = (isk ? a.kc + l * a.k_layer : a.vc + l * a.v_layer) + k_offset(a.D, slot, head, pos, j);   // (an fp32 cache has no pages and holds V like K)
        dst[0] = y1;
        dst[HALF] = y2;
    }
    // one row and query head: the wavefronts share the cached keys, KPW keys a step; the new key is wavefront 0's
    __device__ __forceinline__ void attention(int l, int task) const
    {
        const int Hq = a.D.Hq, r = task / Hq, hh = task % Hq, g = hh / a.D.G, dim = lane % LK * 4, kk = lane / LK;
        const int pos = a.pos[r], slot = a.slot[r];
        const float *kc = a.kc + l * a.k_layer, *vc = a.vc + l * a.v_layer;
        uint4 k[NS], v[NS];
        auto key_of = [&](int from, int i) { return from + (i * FLOW_WAVES + wave) * KPW + kk; };
        auto fetch = [&](int from) {   // (past the context: its last key again)
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const size_t o = k_offset(a.D, slot, g, max(min(key_of(from, i), pos - 1), 0), dim);
                k[i] = *reinterpret_cast<const uint4 *>(kc + o);
                v[i] = *reinterpret_cast<const uint4 *>(vc + o);
            }
        };
        fetch(0);
        FlowPiece<u32x4, 1> q, kn, vn;
        q.off[0] = (a.o_q + l * a.s_q + r * a.D.qw + hh * DH + dim) * 4;
        kn.off[0] = (a.o_kvn + l * a.s_kvn + r * 2 * a.D.kvw + g * DH + dim) * 4;
        vn.off[0] = kn.off[0] + a.D.kvw * 4;
        if (l > 0) gate(a.o_x + l * a.s_x, a.D.d / 32, task);
        flow_poll(buf, wait(), q, kn, vn);
        const float scale = 1.0f / sqrtf((float)DH);
        auto score = [&](float4 kv) {
            float s = __uint_as_float(q.v[0][0].x) * kv.x;
            s = fmaf(__uint_as_float(q.v[0][0].y), kv.y, s);
            s = fmaf(__uint_as_float(q.v[0][0].z), kv.z, s);
            s = fmaf(__uint_as_float(q.v[0][0].w), kv.w, s);
            return flow_sum<LK>(s) * scale;
        };
        const bool own = wave == 0 && kk == 0;
        const float s_own = own ? score(__builtin_bit_cast(float4, kn.v[0][0])) : -INFINITY;
        float M = flow_max4(s_own), L = own ? expf(s_own - M) : 0.f;
        float4 acc = own ? __builtin_bit_cast(float4, vn.v[0][0]) : make_float4(0.f, 0.f, 0.f, 0.f);
        acc.x *= L; acc.y *= L; acc.z *= L; acc.w *= L;
        for (int from = 0; from < pos; from += NS * FLOW_WAVES * KPW) {   // uniform over the workgroup
            if (from > 0) fetch(from);
            float s[NS], top = M;
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                s[i] = key_of(from, i) < pos ? score(__builtin_bit_cast(float4, k[i])) : -INFINITY;
                top = fmaxf(top, s[i]);
            }
            top = flow_max4(top);
            const float c = M == -INFINITY ? 0.f : expf(M - top);
            L *= c; acc.x *= c; acc.y *= c; acc.z *= c; acc.w *= c;
            M = top;
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                if (key_of(from, i) >= pos) continue;
                const float p = expf(s[i] - M);
                const float4 e = __builtin_bit_cast(float4, v[i]);
                L += p;
                acc.x = fmaf(p, e.x, acc.x); acc.y = fmaf(p, e.y, acc.y); acc.z = fmaf(p, e.z, acc.z); acc.w = fmaf(p, e.w, acc.w);
            }
        }
        auto keys = [&](float t) { if constexpr (LK == 16) return flow_sum4(t); else return flow_sum2(t); };   // over the keys of a step
        L = keys(L); acc.x = keys(acc.x); acc.y = keys(acc.y); acc.z = keys(acc.z); acc.w = keys(acc.w);
        if (kk == 0) *reinterpret_cast<float4 *>(&lds.att.o[wave][dim]) = acc;
        if (lane == 0) { lds.att.m[wave] = M; lds.att.l[wave] = L; }
        __syncthreads();
        const int t = threadIdx.x;
        if (t >= DH) return;
        float top = -INFINITY, sum = 0.f, o = 0.f;
#pragma unroll
        for (int w = 0; w < FLOW_WAVES; ++w) top = fmaxf(top, lds.att.m[w]);
#pragma unroll
        for (int w = 0; w < FLOW_WAVES; ++w) {
            const float c = lds.att.m[w] == -INFINITY ? 0.f : expf(lds.att.m[w] - top);
            sum = fmaf(lds.att.l[w], c, sum);
            o = fmaf(lds.att.o[w][t], c, o);
        }
        flow_store(buf, (a.o_at + l * a.s_at + r * a.D.qw + hh * DH + t) * 4, o / sum);
    }
    // out[r][n] = old[r][n] + W . in: WK wavefronts share the columns, the others take further groups of U features
    __device__ __forceinline__ void residual(const void *W, int K, int wk, uint32_t in, uint32_t old, uint32_t out, uint32_t before, int n_before, int task) const
    {
        const int d = a.D.d, groups = FLOW_WAVES / wk, nf = groups * U, n0 = task * nf, k0 = wave % wk * 256 * KC;
        Weights w;
#pragma unroll
        for (int u = 0; u < U; ++u) request(w.v[u], W, n0 + wave / wk * U + u, d, K, k0);
        Rows4 x;
        place(x, in, K, k0);
        const int r = threadIdx.x / nf, f = threadIdx.x % nf;
        const bool fin = r < a.R && n0 + f < d;
        FlowPiece<uint32_t, 1> res;
        res.off[0] = fin ? (old + r * d + n0 + f) * 4 : BUFFER_NOWHERE;
        gate(before, n_before, task);
        flow_poll(buf, wait(), x, res);
        dots(w, x);
        __syncthreads();
        if (!fin) return;
        float s = 0.f;
        for (int i = 0; i < wk; ++i) s += lds.g.red[f / U * wk + i][f % U * RC + r];
        flow_store(buf, (out + r * d + n0 + f) * 4, __uint_as_float(res.v[0][0]) + s);
    }
    __device__ __forceinline__ void oproj(int l, int task) const
    {
        residual(a.layers[l].wo, a.D.qw, 1, a.o_at + l * a.s_at, a.o_x + l * a.s_x, a.o_x1 + l * a.s_x1, a.o_q + l * a.s_q, a.D.qw / 32, task);
    }
    __device__ __forceinline__ void down(int l, int task) const
    {
        residual(a.layers[l].wd, a.D.F, a.wk, a.o_h + l * a.s_h, a.o_x1 + l * a.s_x1, a.o_x + (l + 1) * a.s_x, a.o_x1 + l * a.s_x1, a.D.d / 32, task);
    }
    // 16 FFN features: wavefront w has 2 w and 2 w + 1
    __device__ __forceinline__ void gateup(int l, int task) const
    {
        const int F = a.D.F, f0 = task * 16;
        Weights w;
#pragma unroll
        for (int u = 0; u < U; ++u) request(w.v[u], u & 1 ? a.layers[l].wu : a.layers[l].wg, f0 + 2 * wave + (u >> 1), F, a.D.d);
        uint4 g[KC];
        gains(g, a.layers[l].ln2);
        Rows4 x;
        place(x, a.o_x1 + l * a.s_x1, a.D.d);
        gate(a.o_at + l * a.s_at, a.D.qw / 32, task);
        flow_poll(buf, wait(), x);
        norm(x, g);
        dots(w, x);
        __syncthreads();
        const int r = threadIdx.x >> 4, p = threadIdx.x & 15, u = (p & 1) * 2;
        if (r >= a.R || f0 + p >= F) return;
        const float rs = rstd(r), gt = lds.g.red[p >> 1][u * RC + r] * rs, up = lds.g.red[p >> 1][(u + 1) * RC + r] * rs;
        flow_store(buf, (a.o_h + l * a.s_h + r * F + f0 + p) * 4, gt / (1.0f + expf(-gt)) * up);
    }
    // 32 rows of the LM head (task < nV) or of the router's first layer, which reads the tapped rows
    __device__ __forceinline__ void tail(int task) const
    {
        const int d = a.D.d, V = a.D.V;
        const bool router = task >= a.nV, plain = router && a.tap != 0;
        const int rows = router ? a.D.rh : V, n0 = (router ? task - a.nV : task) * 32;
        Weights w;
#pragma unroll
        for (int u = 0; u < U; ++u) request(w.v[u], router ? a.r_w1 : a.head, n0 + wave * U + u, rows, d);
        uint4 g[KC];
        gains(g, a.final_norm);
        Rows4 x;
        place(x, a.o_x + a.D.L * a.s_x, d);
        gate(a.o_h + (a.D.L - 1) * a.s_h, a.D.F / 32, task);
        flow_poll(buf, wait(), x);
        if (plain)
#pragma unroll
            for (int c = 0; c < KC; ++c) g[c] = make_uint4(0x3f800000u, 0x3f800000u, 0x3f800000u, 0x3f800000u);
        Rows4 raw = x;
        norm(x, g);
        dots(w, x);
        __syncthreads();
        if (task == 0 && wave < a.R) {   // the normalised rows for the last kernel and the caller: wavefront r leaves row r
#pragma unroll
            for (int r = 0; r < RC; ++r) {
                if (r != wave) continue;
                const float rs = rstd(r);
#pragma unroll
                for (int c = 0; c < KC; ++c) {
                    const int k = column(c);
                    if (k >= d) continue;
                    const float4 e = __builtin_bit_cast(float4, raw.v[0][r * KC + c]), ge = __builtin_bit_cast(float4, g[c]);
                    const float4 y = make_float4(e.x * rs * ge.x, e.y * rs * ge.y, e.z * rs * ge.z, e.w * rs * ge.w);
                    *reinterpret_cast<float4 *>(a.hn + (size_t)r * d + k) = y;
                    if (a.hidden) {
                        float *h = a.hidden + (size_t)r * d + k;   // (the caller's: any alignment)
                        const float4 z = a.tap == 0 ? y : e;
                        h[0] = z.x; h[1] = z.y; h[2] = z.z; h[3] = z.w;
                    }
                }
            }
        }
        const int r = threadIdx.x >> 5, f = threadIdx.x & 31;
        if (r >= a.R) return;
        const float z = lds.g.red[f / U][f % U * RC + r] * (plain ? 1.0f : rstd(r));
        if (router) {
            if (n0 + f < rows) a.r1[r * rows + n0 + f] = z;
            return;
        }
        const bool in = n0 + f < V;
        if (a.logits && in) a.logits[(size_t)r * V + n0 + f] = z;
        float mx = in && z > -INFINITY ? z : -INFINITY;   // (a NaN is no maximum)
        int idx = mx > -INFINITY ? n0 + f : 0x7fffffff;
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) {
            const float m2 = __shfl_xor(mx, o, 64);
            const int i2 = __shfl_xor(idx, o, 64);
            if (m2 > mx || (m2 == mx && i2 < idx)) { mx = m2; idx = i2; }
        }
        const float sum = flow_sum<32>(in ? expf(z - (mx == -INFINITY ? 0.f : mx)) : 0.f);
        if (f == 0) a.part[(size_t)task * a.R + r] = make_float4(mx, __int_as_float(idx), sum, 0.f);
    }
};

template <int RC, int KC, int DH>
__global__ __launch_bounds__(64 * FLOW_WAVES, 2) void flow32_kernel(Flow32Args args)
{
    __shared__ typename Flow32<RC, KC, DH>::Lds lds;
    __shared__ int s_task[2];
    if (threadIdx.x == 0) s_task[0] = atomicAdd(args.ticket, 1);
    __syncthreads();
    for (int it = 0;; it ^= 1) {
        const int t = __builtin_amdgcn_readfirstlane(s_task[it]);
        // (the arguments are read again for every task: kept in registers over the loop they would not fit)
        auto kernarg = __builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(kernarg));
        const Flow32Args &a = *(const Flow32Args *)kernarg;
        const int per_layer = a.nQ + a.nA + a.nO + a.nG + a.nD, all = per_layer * a.D.L;
        if (t >= all + a.nV + a.nR) break;   // uniform over the workgroup
        Flow32<RC, KC, DH> f(a, lds);
        const int l = t / per_layer;
        int i = t - l * per_layer;
        if (t >= all) f.tail(t - all);
        else if (i < a.nQ) f.qkv(l, i);
        else if ((i -= a.nQ) < a.nA) f.attention(l, i);
        else if ((i -= a.nA) < a.nO) f.oproj(l, i);
        else if ((i -= a.nO) < a.nG) f.gateup(l, i);
        else f.down(l, i - a.nG);
        // a number held during a wait would be a task nobody has begun: the next one is asked for when this one is over, by a wavefront that finishes none
        if (threadIdx.x == 64 * (FLOW_WAVES - 1)) s_task[it ^ 1] = atomicAdd(a.ticket, 1);
        __syncthreads();   // also: the LDS is free for the next task
    }
}

// ------------------------------------------------------------------ launches

static size_t flow32_layout(const Dims &D, int R, Flow32Args &a)
{
    size_t at = 0;
    auto take = [&](size_t per, int layers, uint32_t &off, uint32_t &stride) {
        stride = (uint32_t)((per + 31) / 32 * 32); off = (uint32_t)at; at += (size_t)stride * layers;
    };
    take((size_t)R * D.d, D.L + 1, a.o_x, a.s_x);   // the first of these is the embedding
    take((size_t)R * D.d, D.L, a.o_x1, a.s_x1);
    take((size_t)R * D.qw, D.L, a.o_q, a.s_q);
    take((size_t)R * 2 * D.kvw, D.L, a.o_kvn, a.s_kvn);
    take((size_t)R * D.qw, D.L, a.o_at, a.s_at);
    take((size_t)R * D.F, D.L, a.o_h, a.s_h);
    return at;
}

size_t flow32_floats(const Dims &D, int max_rows)
{
    Flow32Args a;
    return flow32_layout(D, std::min(max_rows, FLOW32_MAX_ROWS), a);
}
int flow32_slices(const Dims &D) { return (D.V + 31) / 32; }

bool flow32_supported(const Dims &D, int wdt, int kdt)
{
    const size_t most = std::max((size_t)D.F * D.d, std::max((size_t)D.V * D.d, (size_t)D.rh * D.d));
    return wdt == DT_F32 && kdt == DT_F32 && D.L <= FLOW32_MAX_LAYERS && D.d <= 1024 && D.qw <= 1024 && D.d % 8 == 0 && D.F % 8 == 0 && D.F <= 8192 && (D.dh == 64 || D.dh == 128) &&
           most < (size_t)1 << 29 && flow32_slices(D) <= 1024 && flow32_floats(D, FLOW32_MAX_ROWS) < (size_t)1 << 29;
}

// One workgroup reads a row's whole context for a query head, 2048 / 1024 keys of 64 / 128 wide heads in 8 rounds of what it holds. Past that the split attention of
// the general path wins: 2 layers of 256 columns, 1 row, 64 wide heads, after 2000 keys 60 us there / 54 here, after 4000 66 / 81; 8 layers of 1024 columns, 128 wide
// heads, after 1000 keys 402 / 346, after 2000 407 / 484.
bool flow32_takes(const Dims &D, int R, int max_ctx) { return R <= FLOW32_MAX_ROWS && max_ctx <= 8 * FLOW32_STEPS * FLOW_WAVES * 256 / D.dh; }

void launch_flow32_setup(hipStream_t s, const Dims &D, const void *tok_emb, int R, const int *slots, const int *toks, const int *poss, const int *dev_toks,
                         int *d_slot, int *d_tok, int *d_pos, float *buf, int *ticket)
{
    Flow32Args a{};
    const size_t n = flow32_layout(D, R, a);
    flow_setup(s, flow_tables(R, slots, toks, poss), R, d_slot, d_tok, d_pos, (const float *)tok_emb, D, dev_toks, buf, n, a.s_x, 0, 0, ticket);
}

void launch_flow32(hipStream_t s, const Dims &D, const Flow32Model &m, int R, const int *d_slot, const int *d_pos, float *buf, int *ticket, int *given_up, TailArgs &t, float *r1)
{
    Flow32Args a{};
    const size_t n = flow32_layout(D, R, a);
    for (int l = 0; l < D.L; ++l) a.layers[l] = m.layers[l];
    a.kc = (float *)m.kc; a.vc = (float *)m.vc; a.k_layer = m.k_layer / 4; a.v_layer = m.v_layer / 4;
    a.slot = d_slot; a.pos = d_pos; a.rope = m.rope; a.D = D; a.inv_d = 1.0f / (float)D.d; a.R = R; a.buf = buf; a.buf_bytes = (uint32_t)(n * 4); a.ticket = ticket; a.given_up = given_up;
    const bool wide = std::max(D.d, D.qw) > 256 || D.F > 2048;
    const int share = wide ? 1024 : 256;   // columns of a wavefront
    a.wk = 1;
    while (a.wk * share < D.F) a.wk *= 2;
    auto tasks = [](int n_, int per) { return (n_ + per - 1) / per; };
    a.nQ = (D.qw + 2 * D.kvw) / 32; a.nA = R * D.Hq; a.nO = tasks(D.d, FLOW_WAVES * FLOW32_UNIT); a.nG = tasks(D.F, 16); a.nD = tasks(D.d, FLOW_WAVES / a.wk * FLOW32_UNIT);
    a.nV = flow32_slices(D); a.nR = r1 ? tasks(D.rh, 32) : 0;
    a.head = (const float *)t.head; a.final_norm = (const float *)t.final_norm; a.r_w1 = (const float *)t.r_w1;
    a.hn = t.hn; a.hidden = t.hidden; a.logits = t.logits; a.r1 = r1; a.part = (float4 *)t.part; a.tap = t.hidden_tap;
    t.x = buf + a.o_x + (size_t)a.s_x * D.L;
    t.nslices = a.nV;
    if (r1) { t.r1 = r1; t.r1_stride = D.rh; }
    const int grid = std::min(256, (a.nQ + a.nA + a.nO + a.nG + a.nD) * D.L + a.nV + a.nR);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * FLOW_WAVES), 0, s, a); };
    auto rows = [&](auto kc, auto dh) {
        constexpr int KC = decltype(kc)::value, DH = decltype(dh)::value;
        if (R == 1) go(flow32_kernel<1, KC, DH>);
        else if (R == 2) go(flow32_kernel<2, KC, DH>);
        else go(flow32_kernel<4, KC, DH>);
    };
    auto heads = [&](auto kc) { if (D.dh == 64) rows(kc, std::integral_constant<int, 64>{}); else rows(kc, std::integral_constant<int, 128>{}); };
    if (wide) heads(std::integral_constant<int, 4>{}); else heads(std::integral_constant<int, 1>{});
}

}  // namespace tr
