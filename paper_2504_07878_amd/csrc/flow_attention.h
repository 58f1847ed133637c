// Attention of a decode step that runs in one launch: the tasks that flow_kernels.hip and flow_rows_kernels.hip share.
#pragma once
#include "flow_common.h"

namespace tr {

// two values as bf16, and what is left of them
__device__ __forceinline__ uint32_t flow_part(float &a, float &b)
{
    const f32x2 x = {a, b};
    const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    return h;
}
__device__ __forceinline__ uint4 flow_part(float (&v)[8])
{
    uint4 u;
    u.x = flow_part(v[0], v[1]); u.y = flow_part(v[2], v[3]); u.z = flow_part(v[4], v[5]); u.w = flow_part(v[6], v[7]);
    return u;
}
template <class T> __device__ __forceinline__ bf16x8 flow_bf(T u) { return __builtin_bit_cast(bf16x8, u); }
template <int DH> struct FlowAttentionLds { float o[FLOW_WAVES][8][DH + 4]; f32x4 m[8][FLOW_WAVES / 4], l[8][FLOW_WAVES / 4]; };

// K8: bytes from 8 dims to the next 8 of a query, key or value that is handed on; NP: parts of the attention output. F says where they lie (q_at, kvn_at, vn_behind, out_of,
// plane) and which word shows that the link before is on its way (attention_gate, merge_gate).
// UMAX: most blocks of 32 keys a wavefront takes.
template <class F, int DH, int K8, int NP, int UMAX>
struct FlowAttention {
    static constexpr int KS = DH / 32, DT = DH / 16;
    static constexpr int PSTR = DH + 4;
    static_assert(8 * DH / 2 <= 64 * FLOW_WAVES, "two dims of a head per thread");
    __device__ __forceinline__ const F &self() const { return static_cast<const F &>(*this); }

    // Parts of a row's context: blocks of 32 keys cached before this step, FLOW_WAVES U to a part
    __device__ __forceinline__ int parts_of(int pos) const { const int n = FLOW_WAVES * self().a.U; return max(1, ((pos + 31) / 32 + n - 1) / n); }
    // Part c of the keys of one row and kv head: wavefront w takes the blocks FLOW_WAVES U c + w + FLOW_WAVES i. The row's own key and value join in the last part, as a block of one.
    __device__ __forceinline__ void attention(int l, int r, int g, int c) const
    {
        const F &f = self();
        const auto &a = f.a;
        auto &lds = f.lds;
        const auto buf = f.buf;
        const int wave = f.wave, lane = f.lane, col = f.col, o = f.o;
        const int G = flow_now(a.D.G);
        const int pos = a.pos[r], slot = a.slot[r], nblk = (pos + 31) / 32, parts = parts_of(pos), b0 = c * FLOW_WAVES * a.U + wave;
        if (c >= parts) return;   // uniform over the workgroup
        const int ulen = kv_unit_len(a.D), uvts = kv_unit_vts(a.D);
        const bf16_t *kc = reinterpret_cast<const bf16_t *>(a.kc + (size_t)l * a.k_layer), *vc = reinterpret_cast<const bf16_t *>(a.vc + (size_t)l * a.v_layer);
        uint4 kr[UMAX][2][KS], vr[UMAX][DT];
        int nb = 0;   // the wavefront's blocks
        const int krow = 8 * (col >> 2) + (col & 3);   // row `col` of tile t holds key krow + 4 t: the probabilities come out as operands
#pragma unroll
        for (int i = 0; i < UMAX; ++i) {
            const int b = b0 + FLOW_WAVES * i;
            if (i >= a.U || b >= nblk) break;
            nb = i + 1;
            const int t = 32 * b, last = pos - 1 - t;   // keys from the row's own on: the last one again
            int unit = slot, tu = t;
            if (a.D.page) { const int pg = t / a.D.page; unit = a.D.ptab[(size_t)slot * a.D.maxp + pg]; tu = t - pg * a.D.page; }
            const bf16_t *kp = kc + ((size_t)unit * a.D.Hkv + g) * (size_t)ulen * DH + (size_t)tu * DH + 8 * o;
            const bf16_t *vp = vc + ((size_t)unit * a.D.Hkv + g) * (size_t)uvts * DH + (size_t)(tu >> 5) * DH * 32 + col * 32 + 8 * o;
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int s = 0; s < KS; ++s) kr[i][tt][s] = *reinterpret_cast<const uint4 *>(kp + min(krow + 4 * tt, last) * DH + 32 * s);
#pragma unroll
            for (int d = 0; d < DT; ++d) vr[i][d] = *reinterpret_cast<const uint4 *>(vp + d * 16 * 32);
        }
        const bool own = c == parts - 1 && wave == nblk % FLOW_WAVES;   // uniform over the wavefront
        FlowPiece<u32x4, KS> qhm, ql, kn;
        FlowPiece<uint32_t, DT> vn;
        const uint32_t at_q = f.q_at(l, r, g * G + min(col & 7, G - 1)) + o * K8, at_n = f.kvn_at(l, r, g), at_v = at_n + f.vn_behind();
        const uint32_t at_p = (a.o_ap + l * a.s_ap + ((r * a.D.Hq + g * G) * a.P + c) * PSTR) * 4, p_head = flow_now(a.P * PSTR * 4), at_o = flow_now(f.out_of(l, r, g)), o_plane = flow_now(f.plane());
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            qhm.off[s] = at_q + 4 * K8 * s + (col < 8 ? 0 : DH / 8 * K8);
            ql.off[s] = col < 8 ? at_q + 4 * K8 * s + DH / 4 * K8 : BUFFER_NOWHERE;   // columns 8 to 15: zeros
            kn.off[s] = own ? at_n + 4 * K8 * s + o * K8 : BUFFER_NOWHERE;
        }
#pragma unroll
        for (int d = 0; d < DT; ++d) vn.off[d] = own ? at_v + (2 * d + (col >> 3)) * K8 + (col & 6) * 2 : BUFFER_NOWHERE;
        flow_gate(buf, f.attention_gate(l, r), f.wait());
        flow_poll(buf, f.wait(), qhm, ql, kn, vn);
        auto scores = [&](auto &&k) {
            f32x4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(flow_bf(k(s)), flow_bf(qhm.v[0][s]), c0, 0, 0, 0);
                c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(flow_bf(k(s)), flow_bf(ql.v[0][s]), c1, 0, 0, 0);
            }
            return c0 + c1;
        };
        float sc[UMAX][8], s_own = -INFINITY;
        if (own) { const f32x4 c0 = scores([&](int s) { return kn.v[0][s]; }); s_own = c0.x + flow_next<8>(c0.x); }
        float mx = s_own;
#pragma unroll
        for (int i = 0; i < UMAX; ++i) {
            if (i >= nb) break;
            const int t = 32 * (b0 + FLOW_WAVES * i);
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                const f32x4 c0 = scores([&](int s) { return kr[i][tt][s]; });
#pragma unroll
                for (int e = 0; e < 4; ++e) sc[i][4 * tt + e] = c0[e] + flow_next<8>(c0[e]);   // key t + 8 o + 4 tt + e
            }
            if (t + 32 > pos) {
#pragma unroll
                for (int e = 0; e < 8; ++e) sc[i][e] = t + 8 * o + e < pos ? sc[i][e] : -INFINITY;
                // a probability of 0 does not make up for what an earlier sequence left there: infinities and NaNs go
                const int left = pos - t - 8 * o;   // of this lane's 8 values of a dim
                auto keep = [&](int w) { return left > 2 * w + 1 ? ~0u : left > 2 * w ? 0xffffu : 0u; };
#pragma unroll
                for (int d = 0; d < DT; ++d) { vr[i][d].x &= keep(0); vr[i][d].y &= keep(1); vr[i][d].z &= keep(2); vr[i][d].w &= keep(3); }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) mx = fmaxf(mx, sc[i][e]);
        }
        mx = flow_max4(mx);   // finite where the wavefront has a block: its first key is valid
        float sum = 0.f;
        f32x4 acc[DT];
#pragma unroll
        for (int d = 0; d < DT; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < UMAX; ++i) {
            if (i >= nb) break;
            float p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) { p[e] = __expf(sc[i][e] - mx); sum += p[e]; }
            const uint4 hi = flow_part(p), mid = flow_part(p), lo = flow_part(p);
            const uint4 phm = col < 8 ? hi : mid, pl = col < 8 ? lo : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int d = 0; d < DT; ++d) {
                acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(flow_bf(vr[i][d]), flow_bf(phm), acc[d], 0, 0, 0);
                acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(flow_bf(vr[i][d]), flow_bf(pl), acc[d], 0, 0, 0);
            }
        }
        if (own) {   // key 0 of a block of one
            float p = __expf(s_own - mx), none = 0.f;
            if (o == 0) sum += p;
            const uint32_t hi = flow_part(p, none), mid = flow_part(p, none), lo = flow_part(p, none);
            const uint4 phm = make_uint4(o == 0 ? (col < 8 ? hi : mid) : 0, 0, 0, 0), pl = make_uint4(o == 0 && col < 8 ? lo : 0, 0, 0, 0);
#pragma unroll
            for (int d = 0; d < DT; ++d) {
                const uint4 v = make_uint4(col & 1 ? vn.v[0][d] >> 16 : vn.v[0][d] & 0xffffu, 0, 0, 0);
                acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(flow_bf(v), flow_bf(phm), acc[d], 0, 0, 0);
                acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(flow_bf(v), flow_bf(pl), acc[d], 0, 0, 0);
            }
        }
        sum = flow_sum4(sum);
        const bool any = nb > 0 || own;
        if (any) {
#pragma unroll
            for (int d = 0; d < DT; ++d) {
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[d][e] + flow_next<8>(acc[d][e]);
                if (col < 8) *reinterpret_cast<f32x4 *>(&lds.att.o[wave][col][16 * d + 4 * o]) = v;
            }
        }
        if (lane < 8) {
            reinterpret_cast<float *>(&lds.att.m[lane])[wave] = any ? mx : -INFINITY;
            reinterpret_cast<float *>(&lds.att.l[lane])[wave] = any ? sum : 0.f;
        }
        __syncthreads();
        const int h = threadIdx.x / (DH / 2), d = 2 * (threadIdx.x % (DH / 2));
        if (h >= G) return;
        float M = -INFINITY, L = 0.f, O0 = 0.f, O1 = 0.f, mw[FLOW_WAVES], lw[FLOW_WAVES];
#pragma unroll
        for (int w = 0; w < FLOW_WAVES; ++w) { mw[w] = lds.att.m[h][w >> 2][w & 3]; lw[w] = lds.att.l[h][w >> 2][w & 3]; M = fmaxf(M, mw[w]); }
#pragma unroll
        for (int w = 0; w < FLOW_WAVES; ++w) {
            const float by = __expf(mw[w] - M);
            const float2 ow = *reinterpret_cast<const float2 *>(&lds.att.o[w][h][d]);
            const bool none = mw[w] == -INFINITY;   // a wavefront without keys: its sums are whatever the LDS held
            L = fmaf(lw[w], by, L);
            O0 = none ? O0 : fmaf(ow.x, by, O0); O1 = none ? O1 : fmaf(ow.y, by, O1);
        }
        if (parts > 1) {
            flow_store(buf, at_p + h * p_head + d * 4, O0, O1);
            if (d == 0) flow_store(buf, at_p + h * p_head + DH * 4, M, L);
        } else attention_out(f, at_o + (h * DH + d) * 2, o_plane, O0, O1, L);
    }
    // two dims of the attention output as operand parts
    __device__ __forceinline__ void attention_out(const F &f, uint32_t at, uint32_t plane, float O0, float O1, float L) const
    {
        const float inv = flow_rcp(L);
        O0 *= inv; O1 *= inv;
#pragma unroll
        for (int p = 0; p < NP; ++p) { const uint32_t w = flow_part(O0, O1); flow_store_pair(f.buf, at + p * plane, w); }
    }
    // the parts of `heads` heads of a row put together, two dims a thread (at most 1024)
    __device__ __forceinline__ void merge(int l, int r, int head, int heads) const
    {
        static_assert(2 * 64 * FLOW_WAVES >= 1024, "");
        const F &f = self();
        const auto &a = f.a;
        const auto buf = f.buf;
        const int parts = parts_of(a.pos[r]), k = 2 * (int)threadIdx.x, d = k % DH;
        if (parts == 1 || k >= heads * DH) return;
        const uint32_t at_p = (a.o_ap + l * a.s_ap + (r * a.D.Hq + head + k / DH) * a.P * PSTR) * 4, at_o = f.out_of(l, r, 0) + (head * DH + k) * 2, plane = flow_now(f.plane());
        flow_gate(buf, f.merge_gate(l, r), f.wait());
        float M = -INFINITY, L = 0.f, O0 = 0.f, O1 = 0.f;
        for (int c0 = 0; c0 < parts; c0 += 4) {
            FlowPiece<u32x2, 4> ml, po;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                ml.off[c] = c0 + c < parts ? at_p + ((c0 + c) * PSTR + DH) * 4 : BUFFER_NOWHERE;
                po.off[c] = c0 + c < parts ? at_p + ((c0 + c) * PSTR + d) * 4 : BUFFER_NOWHERE;
            }
            flow_poll(buf, f.wait(), ml, po);
            float m = M;
#pragma unroll
            for (int c = 0; c < 4; ++c) m = c0 + c < parts ? fmaxf(m, __uint_as_float(ml.v[0][c].x)) : m;
            const float old = __expf(M - m);   // 0 the first time
            L *= old; O0 *= old; O1 *= old; M = m;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float by = c0 + c < parts ? __expf(__uint_as_float(ml.v[0][c].x) - m) : 0.f;
                L = fmaf(__uint_as_float(ml.v[0][c].y), by, L);
                O0 = fmaf(__uint_as_float(po.v[0][c].x), by, O0); O1 = fmaf(__uint_as_float(po.v[0][c].y), by, O1);
            }
        }
        attention_out(f, at_o, plane, O0, O1, L);
    }
};

}  // namespace tr
