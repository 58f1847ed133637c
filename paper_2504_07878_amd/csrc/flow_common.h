// What the kernels that run a whole decode step in one launch share (flow_kernels.hip, flow_rows_kernels.hip, flow_f32_kernels.hip): words that tell by themselves that they are
// there, and how a task waits for them.
#pragma once
#include "mfma_common.h"
#include <algorithm>
#include <type_traits>
#include <utility>

namespace tr {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

constexpr uint32_t SENT = 0xffffffffu;
constexpr int FLOW_WAVES = 8;
constexpr int FLOW_SC1 = 16;     // cache policy of buffer loads and stores: past the L2 of the XCD
constexpr uint32_t FLOW_SPINS = 1u << 22;   // polls until a wait is given up (seconds): no wavefront waits for ever, whatever happens

struct FlowWait {
    int *gave_up;
    uint32_t spins = 0;
    __device__ __forceinline__ bool over()   // a wait that ends so leaves its mark, which the last kernel of the step and every later one report
    {
        asm volatile("" ::: "memory");
        ++spins;
        if ((spins & 1023) == 0 && __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return true;
        if (spins < FLOW_SPINS) return false;
        __hip_atomic_store(gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
};

// one word (or two, or four) of the hand-over buffers, past the L2; BUFFER_NOWHERE: zeros
template <int POLICY> __device__ __forceinline__ void flow_load(__amdgpu_buffer_rsrc_t b, uint32_t off, uint32_t uniform, u32x4 &v) { v = (u32x4)__builtin_amdgcn_raw_buffer_load_b128(b, (int)off, (int)uniform, POLICY); }
template <int POLICY> __device__ __forceinline__ void flow_load(__amdgpu_buffer_rsrc_t b, uint32_t off, uint32_t uniform, u32x2 &v) { v = (u32x2)__builtin_amdgcn_raw_buffer_load_b64(b, (int)off, (int)uniform, POLICY); }
template <int POLICY> __device__ __forceinline__ void flow_load(__amdgpu_buffer_rsrc_t b, uint32_t off, uint32_t uniform, uint32_t &v) { v = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(b, (int)off, (int)uniform, POLICY); }
__device__ __forceinline__ uint32_t flow_max(u32x4 v) { return max(max(v.x, v.y), max(v.z, v.w)); }   // SENT if any word is
__device__ __forceinline__ uint32_t flow_max(u32x2 v) { return max(v.x, v.y); }
__device__ __forceinline__ uint32_t flow_max(uint32_t v) { return v; }

// Words that are waited for: where (each of N places of the lane in each of M sets, a uniform distance apart), and what arrived
template <class T, int N, int M = 1> struct FlowPiece { uint32_t off[N], set[M]; T v[M][N]; };
template <int POLICY, class T, int N, int M> __device__ __forceinline__ void flow_request(__amdgpu_buffer_rsrc_t b, FlowPiece<T, N, M> &p)
{
#pragma unroll
    for (int q = 0; q < M; ++q)
#pragma unroll
        for (int i = 0; i < N; ++i) flow_load<POLICY>(b, p.off[i], q == 0 ? 0 : p.set[q], p.v[q][i]);
}
template <class T, int N, int M> __device__ __forceinline__ uint32_t flow_seen(const FlowPiece<T, N, M> &p)
{
    uint32_t m = 0;
#pragma unroll
    for (int q = 0; q < M; ++q)
#pragma unroll
        for (int i = 0; i < N; ++i) m = max(m, flow_max(p.v[q][i]));
    return m;
}
template <int POLICY, class... P> __device__ __forceinline__ bool flow_there(__amdgpu_buffer_rsrc_t b, P &...p)
{
    (flow_request<POLICY>(b, p), ...);
    uint32_t m = 0;
    ((m = max(m, flow_seen(p))), ...);
    asm volatile("" ::: "memory");
    return !__any(m == SENT);
}
// loads until every word has arrived
template <class... P> __device__ __forceinline__ void flow_poll(__amdgpu_buffer_rsrc_t b, FlowWait w, P &...p)
{
    while (!flow_there<FLOW_SC1>(b, p...) && !w.over()) {}
}
// Many words that are most likely there: through the L2, which serves all workgroups of an XCD that want them; no line of them has been in it during this launch but
// as somebody found it missing. Words that are not there yet are waited for as ever.
template <class... P> __device__ __forceinline__ void flow_fetch(__amdgpu_buffer_rsrc_t b, FlowWait w, P &...p)
{
    if (!flow_there<0>(b, p...)) flow_poll(b, w, p...);
}
// until one word (the same for all lanes) has arrived
__device__ __forceinline__ void flow_gate(__amdgpu_buffer_rsrc_t b, uint32_t off, FlowWait w)
{
    for (;;) {
        uint32_t v;
        flow_load<FLOW_SC1>(b, off, 0, v);
        if (v != SENT || w.over()) break;
        __builtin_amdgcn_s_sleep(4);
    }
}

// until every word has arrived; while they have not, one word of the link before is looked at
template <class... P> __device__ __forceinline__ void flow_await(__amdgpu_buffer_rsrc_t b, uint32_t gate, FlowWait w, P &...p)
{
    if (flow_there<FLOW_SC1>(b, p...)) return;
    flow_gate(b, gate, w);
    flow_poll(b, w, p...);
}

// what is handed on: never SENT
__device__ __forceinline__ uint32_t flow_word(float v)
{
    const uint32_t u = __float_as_uint(v);
    return u == SENT ? 0x7fc00000u : u;
}
__device__ __forceinline__ uint32_t flow_pair(uint32_t u) { return u == SENT ? 0x7fc07fc0u : u; }   // two bf16
__device__ __forceinline__ void flow_store(__amdgpu_buffer_rsrc_t b, uint32_t off, f32x4 v)
{
    const u32x4 u = {flow_word(v.x), flow_word(v.y), flow_word(v.z), flow_word(v.w)};
    __builtin_amdgcn_raw_buffer_store_b128(u, b, (int)off, 0, FLOW_SC1);
}
__device__ __forceinline__ void flow_store(__amdgpu_buffer_rsrc_t b, uint32_t off, float v) { __builtin_amdgcn_raw_buffer_store_b32(flow_word(v), b, (int)off, 0, FLOW_SC1); }
__device__ __forceinline__ void flow_store(__amdgpu_buffer_rsrc_t b, uint32_t off, float v0, float v1)
{
    const u32x2 u = {flow_word(v0), flow_word(v1)};
    __builtin_amdgcn_raw_buffer_store_b64(u, b, (int)off, 0, FLOW_SC1);
}
__device__ __forceinline__ void flow_store_pair(__amdgpu_buffer_rsrc_t b, uint32_t off, uint32_t u) { __builtin_amdgcn_raw_buffer_store_b32(flow_pair(u), b, (int)off, 0, FLOW_SC1); }
__device__ __forceinline__ void flow_store_pair(__amdgpu_buffer_rsrc_t b, uint32_t off, uint32_t u0, uint32_t u1)
{
    const u32x2 u = {flow_pair(u0), flow_pair(u1)};
    __builtin_amdgcn_raw_buffer_store_b64(u, b, (int)off, 0, FLOW_SC1);
}

template <int C> __device__ __forceinline__ float flow_dpp(float v) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), C, 0xf, 0xf, true)); }
template <int N> __device__ __forceinline__ float flow_next(float v) { return flow_dpp<0x120 + 16 - N>(v); }   // value of the lane N on, within 16 lanes
// a wavefront's halves: the values of lane % 32 and of lane % 32 + 32; rows of 16 lanes: of the even and of the odd row of a half
struct FlowTwo { float a, b; };
__device__ __forceinline__ FlowTwo flow_halves(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return FlowTwo{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ FlowTwo flow_rows(float v)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return FlowTwo{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ float flow_sum2(float v) { const FlowTwo t = flow_halves(v); return t.a + t.b; }   // lane % 32 + 32 i
__device__ __forceinline__ float flow_sum4(float v) { const FlowTwo t = flow_rows(v); return flow_sum2(t.a + t.b); }   // lane % 16 + 16 i
__device__ __forceinline__ float flow_max4(float v)
{
    const FlowTwo t = flow_rows(v), u = flow_halves(fmaxf(t.a, t.b));
    return fmaxf(u.a, u.b);
}
// sum over groups of N lanes
template <int N> __device__ __forceinline__ float flow_sum(float v)
{
    v += flow_dpp<0xb1>(v);                        // lane ^ 1
    v += flow_dpp<0x4e>(v);                        // lane ^ 2
    v += flow_dpp<0x141>(v);                       // the other four of eight
    if constexpr (N >= 16) v += flow_dpp<0x140>(v);   // the other eight of sixteen
    if constexpr (N >= 32) { const FlowTwo t = flow_rows(v); v = t.a + t.b; }
    if constexpr (N >= 64) v = flow_sum2(v);
    return v;
}
// reciprocal of a finite value: the hardware's and one Newton step (below 1 ulp; of infinity a NaN)
__device__ __forceinline__ float flow_rcp(float x)
{
    const float r = __builtin_amdgcn_rcpf(x), e = fmaf(-x, r, 1.0f);
    return fmaf(e, r, r);
}
// 1 / sqrt(x): the hardware's and one Newton step (below 1 ulp); zeros, subnormals, infinities and NaNs, which the step would spoil, by the definition
__device__ __forceinline__ float flow_rsqrt(float x)
{
    if (!__builtin_amdgcn_classf(x, 0x100)) return 1.0f / sqrtf(x);   // (0x100: positive and normal)
    const float r = __builtin_amdgcn_rsqf(x), e = fmaf(-x * r, r, 1.0f);
    return fmaf(0.5f * e, r, r);
}
// t / (1 + exp(-t)) of N values. exp(-t) = 2^n 2^f, n the whole number nearest to -t log2 e; the quotient is corrected by its remainder. Gates beyond 80, where a sum or
// a quotient leaves the normal range, by the definition, so that a saturated gate gives -0.
// Steps of the 0.5B-class model with expf, divisions and 1 / sqrtf throughout / with these two: 1 row 326.9 / 321.7 us, 7 rows 488.7 / 483.5; SwiGLU's error, gates of
// -20 to 0, mean 3.1e-8 / 3.2e-8, largest 1.0e-7 / 1.0e-7.
template <int N> __device__ __forceinline__ void flow_silu(const float (&t)[N], float (&s)[N])
{
    float most = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) most = fmaxf(most, fabsf(t[i]));
    if (!(most < 80.f)) {
#pragma unroll
        for (int i = 0; i < N; ++i) s[i] = t[i] / (1.0f + expf(-t[i]));
        return;
    }
    constexpr double LOG2E = 1.4426950408889634074;
    constexpr float L = (float)LOG2E, L_REST = (float)(LOG2E - (double)L);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float n = rintf(-t[i] * L), f = fmaf(-t[i], L_REST, fmaf(-t[i], L, -n)), den = 1.0f + ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
        const float r = __builtin_amdgcn_rcpf(den), q = t[i] * r;
        s[i] = fmaf(fmaf(-q, den, t[i]), r, q);
    }
}
// an argument that is wanted behind a wait: read before it, not when it is used
template <class T> __device__ __forceinline__ T flow_now(T v) { asm volatile("" : "+s"(v)); return v; }

// ------------------------------------------------------------------ set-up

struct FlowSetup { int slot[FLOW_MAX_ROWS], tok[FLOW_MAX_ROWS], pos[FLOW_MAX_ROWS]; };

// Row tables and embedding lookup (blocks 0 .. R - 1), hand-over buffers to SENT (the others), task counter to zero
template <class WT>
__global__ __launch_bounds__(256) void flow_setup_kernel(FlowSetup a, int R, int *d_slot, int *d_tok, int *d_pos, const WT *E, int d, int vocab, const int *dev_tok,
                                                         float *x0, uint4 *fill, uint32_t n_fill, uint32_t skip, uint32_t zero0, uint32_t zero1, int *ticket)
{
    const int b = blockIdx.x;
    if (b < R) {
        const int tok = dev_tok ? min(max(dev_tok[b], 0), vocab - 1) : a.tok[b];
        if (threadIdx.x == 0) { d_slot[b] = a.slot[b]; d_tok[b] = tok; d_pos[b] = a.pos[b]; }
        if (b == 0 && threadIdx.x == 0) *ticket = 0;
        const WT *e = E + (size_t)tok * d;
        for (int j = threadIdx.x; j < d; j += 256) {
            if constexpr (std::is_same_v<WT, float>) x0[(size_t)b * d + j] = __uint_as_float(flow_word(e[j]));   // (the first layer takes it as arrived)
            else x0[(size_t)b * d + j] = __uint_as_float((uint32_t)e[j] << 16);
        }
        return;
    }
    for (uint32_t i = skip + (b - R) * 256 + threadIdx.x; i < n_fill; i += (gridDim.x - R) * 256) {
        const uint32_t v = i >= zero0 && i < zero1 ? 0 : SENT;
        fill[i] = make_uint4(v, v, v, v);
    }
}

inline FlowSetup flow_tables(int R, const int *slots, const int *toks, const int *poss)
{
    FlowSetup su{};
    for (int i = 0; i < R; ++i) { su.slot[i] = slots[i]; su.tok[i] = toks ? toks[i] : 0; su.pos[i] = poss[i]; }
    return su;
}
// n words of hand-over buffers: the embedding in the first `first` of them, zeros in [zero0, zero1) (multiples of 4)
template <class WT>
void flow_setup(hipStream_t s, const FlowSetup &su, int R, int *d_slot, int *d_tok, int *d_pos, const WT *E, const Dims &D, const int *dev_toks, float *buf, size_t n,
                uint32_t first, uint32_t zero0, uint32_t zero1, int *ticket)
{
    const uint32_t skip = first / 4, n_fill = (uint32_t)(n / 4);   // 16-byte words
    hipLaunchKernelGGL(flow_setup_kernel<WT>, dim3(R + std::min<uint32_t>(1024, (n_fill - skip + 255) / 256)), dim3(256), 0, s, su, R, d_slot, d_tok, d_pos, E, D.d, D.V,
                       dev_toks, buf, reinterpret_cast<uint4 *>(buf), n_fill, skip, zero0 / 4, zero1 / 4, ticket);
}

}  // namespace tr
