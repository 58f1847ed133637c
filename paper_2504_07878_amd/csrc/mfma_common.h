// Types, operand layouts and packing shared by the matrix-core kernels (mfma_kernels.hip, tile_kernels.hip).
#pragma once
#include "tr_internal.h"

namespace tr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// value = hi + lo with hi = bf16(value), lo = bf16(value - hi), both rounded to nearest even by the hardware's packed
// conversion (two values per instruction)
__device__ __forceinline__ void split_hi_lo(float v0, float v1, uint32_t &h, uint32_t &l)
{
    const f32x2 x = {v0, v1};
    h = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
    const f32x2 rest = {v0 - __uint_as_float(h << 16), v1 - __uint_as_float(h & 0xffff0000u)};
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, bf16x2));
}
__device__ __forceinline__ void split_hi_lo(const float (&v)[8], uint4 &hi, uint4 &lo)
{
    split_hi_lo(v[0], v[1], hi.x, lo.x); split_hi_lo(v[2], v[3], hi.y, lo.y);
    split_hi_lo(v[4], v[5], hi.z, lo.z); split_hi_lo(v[6], v[7], hi.w, lo.w);
}

// Packed activations of one group of up to 64 rows: [k-step][column block][lane] of 16 bytes, column blocks =
// {hi rows 0-31, (hi rows 32-63), lo rows 0-31, (lo rows 32-63)}; lane = row%32 + 32*(k%16 / 8).
__device__ __forceinline__ void store_packed(uint4 *pack, int ncb, int row_in_group, int k8 /* index of the 8-column chunk */, uint4 hi, uint4 lo)
{
    const int ks = k8 >> 1, lane = (row_in_group & 31) + 32 * (k8 & 1), cb = row_in_group >> 5;
    pack[((size_t)ks * ncb + cb) * 64 + lane] = hi;
    pack[((size_t)ks * ncb + (ncb >> 1) + cb) * 64 + lane] = lo;
}
__device__ __forceinline__ void store_packed(uint4 *pack, int ncb, int row_in_group, int k8, const float (&v)[8])
{
    uint4 hi, lo;
    split_hi_lo(v, hi, lo);
    store_packed(pack, ncb, row_in_group, k8, hi, lo);
}

// MFMA row rho of a tile (the accumulator holds rows 8*qd + 4*hf + e in register 4*qd + e of the lanes with lane/32 = hf)
// carries the tile's feature tile_feature(rho): features are placed so that the accumulator registers {8a .. 8a+7} of
// one lane, a = 0 or 1, are 8 CONSECUTIVE features 16a + 8hf .. + 7. A wavefront can then hand half of its accumulator
// to another wavefront and keep, per lane, whole runs of 8 features.
__host__ __device__ __forceinline__ int tile_feature(int rho)
{
    const int qd = rho >> 3, hf = (rho >> 2) & 1, e = rho & 3;
    return 16 * (qd >> 1) + 8 * hf + 4 * (qd & 1) + e;
}

// A buffer of `bytes` bytes and a lane's 16 bytes of it, `off` bytes in (plus `uniform`): where off lies beyond the buffer the lane gets zeros and no
// memory is touched, but the load counts like any other, so that the number in flight stays known at compile time.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}
constexpr uint32_t BUFFER_NOWHERE = 0x80000000u;   // (buffers are smaller)
__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t b, uint32_t off, uint32_t uniform)
{
    typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
    return __builtin_bit_cast(uint4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(b, (int)off, (int)uniform, 0));
}

// four / one cache elements, rounded to nearest even where the cache is bf16
__device__ __forceinline__ void kv_store4(float *dst, const float (&v)[4]) { *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ void kv_store4(bf16_t *dst, const float (&v)[4])
{
    const f32x2 x0 = {v[0], v[1]}, x1 = {v[2], v[3]};
    *reinterpret_cast<uint2 *>(dst) = make_uint2(__builtin_bit_cast(uint32_t, __builtin_convertvector(x0, bf16x2)),
                                                 __builtin_bit_cast(uint32_t, __builtin_convertvector(x1, bf16x2)));
}
__device__ __forceinline__ void kv_store1(float *dst, float v) { *dst = v; }
__device__ __forceinline__ void kv_store1(bf16_t *dst, float v)
{
    const f32x2 x = {v, 0.f};
    *dst = (bf16_t)__builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}

// Where the outputs of a q|k|v projection go.
template <typename KT>
struct QkvOut {
    const float *bias;        // concatenated [qw + 2 kvw], natural feature order
    const float2 *rope;
    float *q;
    KT *kc, *vc;
    int Hq, Hkv, dh, unit_len, qw, vts;   // unit_len, vts: positions per storage unit of the cache (a slot or a page)
};

// Bias, rotation and store of 8 outputs of one row: features i0 .. i0+7 of tile t, which are the pairs (j, j + dh/2), j = 16*sub +
// i0/2 .. +3, as (first, partner) x 4 (see repack_kernel). pos: the row's position; its key and value go to position upos of storage unit `unit`.
// BIASED: v includes the bias.
template <bool BIASED, typename KT>
__device__ __forceinline__ void qkv_emit(const QkvOut<KT> &o, int t, int m, int i0, const float (&v)[8], int pos, int unit, int upos)
{
    const int tph = o.dh >> 5, half = o.dh >> 1, hh = t / tph, j0 = (t % tph) * 16 + (i0 >> 1);
    float4 ba = make_float4(0.f, 0.f, 0.f, 0.f), bb = ba;
    if (!BIASED) { ba = *reinterpret_cast<const float4 *>(o.bias + hh * o.dh + j0); bb = *reinterpret_cast<const float4 *>(o.bias + hh * o.dh + half + j0); }
    const float a[4] = {v[0] + ba.x, v[2] + ba.y, v[4] + ba.z, v[6] + ba.w}, b[4] = {v[1] + bb.x, v[3] + bb.y, v[5] + bb.z, v[7] + bb.w};
    float lo[4], hi[4];
    if (hh < o.Hq + o.Hkv) {
        const float4 *rp = reinterpret_cast<const float4 *>(o.rope + (size_t)pos * half + j0);   // 4 (cos, sin) pairs, 32 bytes, aligned
        const float4 c0 = rp[0], c1 = rp[1];
        const float cx[4] = {c0.x, c0.z, c1.x, c1.z}, sy[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            lo[e] = a[e] * cx[e] - b[e] * sy[e];
            hi[e] = b[e] * cx[e] + a[e] * sy[e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) { lo[e] = a[e]; hi[e] = b[e]; }
    }
    if (hh < o.Hq) {
        float *dst = o.q + (size_t)m * o.qw + hh * o.dh + j0;
        *reinterpret_cast<float4 *>(dst) = make_float4(lo[0], lo[1], lo[2], lo[3]);
        *reinterpret_cast<float4 *>(dst + half) = make_float4(hi[0], hi[1], hi[2], hi[3]);
    } else {
        const int head = hh < o.Hq + o.Hkv ? hh - o.Hq : hh - o.Hq - o.Hkv;
        if (hh < o.Hq + o.Hkv || o.vts == 0) {
            KT *dst = (hh < o.Hq + o.Hkv ? o.kc : o.vc) + (((size_t)unit * o.Hkv + head) * o.unit_len + upos) * o.dh + j0;
            kv_store4(dst, lo);
            kv_store4(dst + half, hi);
        } else {   // block-transposed V: one position of 8 dim rows
            KT *dst = o.vc + ((((size_t)unit * o.Hkv + head) * (o.vts >> 5) + (upos >> 5)) * o.dh + j0) * 32 + (upos & 31);
#pragma unroll
            for (int e = 0; e < 4; ++e) { kv_store1(dst + e * 32, lo[e]); kv_store1(dst + (half + e) * 32, hi[e]); }
        }
    }
}

}  // namespace tr
