/* Fused producers: the elementwise step that yields the bf16 input of a
 * BitLinear, evaluated inside the kernel that quantises it, so the bf16 tensor
 * never exists in HBM.  Each kind is exact elementwise fp32 work followed by a
 * round-to-nearest-even narrowing to bf16 (ReLU^2 in the FFN is the report's,
 * Section 2; the residual add and the context-length-1 attention are the
 * synthetic chain glue of this repository). */
#pragma once
#include "bl_device.h"

struct bl_prod_dev {
    int kind;            /* BL_PROD_* */
    const void* in0;
    const float* in1;
    float* aux_out;
    int voff, group, hd, in_stride;   /* ATTN_V geometry; in_stride = floats per source row */
    int norm;            /* RMS normalisation in front of the quantiser */
    const float* gain;   /* [K] or NULL */
    float eps;
};

/* fp32 values of k = 16u .. 16u+15 of token m, before narrowing (any kind).
 * store_aux: this caller also writes the fp32 by-product (RESIDUAL: the sum). */
__device__ __forceinline__ void bl_produce16_f32(const bl_prod_dev& pd, int m, int u, int K, bool store_aux,
                                                 float v[16]) {
    if (pd.kind == BL_PROD_BF16) {
        const bl_v4i BL_G* xr = bl_gc<bl_v4i>((const uint16_t*)pd.in0 + (int64_t)m * K);
        const bl_v4i lo = xr[2 * u], hi = xr[2 * u + 1];
        const uint32_t w[8] = {(uint32_t)lo[0], (uint32_t)lo[1], (uint32_t)lo[2], (uint32_t)lo[3],
                               (uint32_t)hi[0], (uint32_t)hi[1], (uint32_t)hi[2], (uint32_t)hi[3]};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            v[2 * j] = bl_bf16_to_f32(w[j] & 0xFFFFu);
            v[2 * j + 1] = bl_bf16_to_f32(w[j] >> 16);
        }
        return;
    }
    if (pd.kind == BL_PROD_RELU2_GATE) {
        const bl_v4f BL_G* g4 = bl_gc<bl_v4f>((const float*)pd.in0 + (int64_t)m * 2 * K + (int64_t)u * 16);
        const bl_v4f BL_G* u4 = bl_gc<bl_v4f>((const float*)pd.in0 + (int64_t)m * 2 * K + K + (int64_t)u * 16);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bl_v4f g = g4[j], up = u4[j];
            const float gg[4] = {g.x, g.y, g.z, g.w}, uu[4] = {up.x, up.y, up.z, up.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float r = fmaxf(gg[e], 0.0f);
                const float r2 = r * r;
                v[4 * j + e] = r2 * uu[e];
            }
        }
        return;
    }
    int64_t off;
    if (pd.kind == BL_PROD_ATTN_V) {
        const int k = u * 16;
        off = (int64_t)m * pd.in_stride + pd.voff + ((k / pd.hd) / pd.group) * pd.hd + (k % pd.hd);
    } else {
        off = (int64_t)m * K + (int64_t)u * 16;
    }
    const bl_v4f BL_G* a4 = bl_gc<bl_v4f>((const float*)pd.in0 + off);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const bl_v4f a = a4[j];
        v[4 * j] = a.x; v[4 * j + 1] = a.y; v[4 * j + 2] = a.z; v[4 * j + 3] = a.w;
    }
    if (pd.kind == BL_PROD_RESIDUAL) {
        const bl_v4f BL_G* b4 = bl_gc<bl_v4f>(pd.in1 + off);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bl_v4f b = b4[j];
            v[4 * j] += b.x; v[4 * j + 1] += b.y; v[4 * j + 2] += b.z; v[4 * j + 3] += b.w;
        }
        if (store_aux && pd.aux_out) {
            bl_v4f BL_G* o4 = (bl_v4f BL_G*)(pd.aux_out + off);
#pragma unroll
            for (int j = 0; j < 4; ++j) o4[j] = bl_v4f{v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]};
        }
    }
}

/* bf16 bit patterns of k = 16u .. 16u+15 of token m: lo = first eight, hi = last eight.
 * rn: the token's normalisation factor (used only if NORM and pd.norm).  NORM = false
 * compiles the normalisation out: kernels that never normalise keep their registers. */
template <bool NORM>
__device__ __forceinline__ void bl_produce16(const bl_prod_dev& pd, int m, int u, int K, bool store_aux, float rn,
                                             uint4& lo, uint4& hi) {
    if (pd.kind == BL_PROD_BF16 && !(NORM && pd.norm)) {
        const bl_v4i BL_G* xr = bl_gc<bl_v4i>((const uint16_t*)pd.in0 + (int64_t)m * K);
        lo = __builtin_bit_cast(uint4, xr[2 * u]);
        hi = __builtin_bit_cast(uint4, xr[2 * u + 1]);
        return;
    }
    float v[16];
    bl_produce16_f32(pd, m, u, K, store_aux, v);
    if (NORM && pd.norm) {
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = v[e] * rn;
        if (pd.gain) {
            const bl_v4f BL_G* g4 = bl_gc<bl_v4f>(pd.gain + (int64_t)u * 16);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bl_v4f g = g4[j];
                v[4 * j] *= g.x; v[4 * j + 1] *= g.y; v[4 * j + 2] *= g.z; v[4 * j + 3] *= g.w;
            }
        }
    }
    lo = make_uint4(bl_pack2_bf16(v[0], v[1]), bl_pack2_bf16(v[2], v[3]), bl_pack2_bf16(v[4], v[5]),
                    bl_pack2_bf16(v[6], v[7]));
    hi = make_uint4(bl_pack2_bf16(v[8], v[9]), bl_pack2_bf16(v[10], v[11]), bl_pack2_bf16(v[12], v[13]),
                    bl_pack2_bf16(v[14], v[15]));
}

/* Normalising production of token m by a 256-thread workgroup, in the fixed order of the
 * public header (thread j is leaf j).  The thread's first two groups (u = tid, tid + 256) are
 * produced once, kept in registers across the reduction and returned as normalised bf16 words
 * in xv[0..3]; groups beyond those (K > 8192) only enter the sum and are produced again by the
 * caller with the returned factor.  store_aux as in bl_produce16_f32.  s4: four doubles of LDS,
 * free to reuse after the caller's next barrier.  Contains one barrier. */
__device__ __forceinline__ float bl_norm_produce2(const bl_prod_dev& pd, int m, int K, bool store_aux, double* s4,
                                                  uint4 xv[4]) {
    const int tid = threadIdx.x, groups = K / 16;
    float tv[2][16];
    double part = 0.0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int u = tid + j * 256;
        if (u < groups) {
            bl_produce16_f32(pd, m, u, K, store_aux, tv[j]);
#pragma unroll
            for (int e = 0; e < 16; ++e) part += (double)tv[j][e] * (double)tv[j][e];
        }
    }
    for (int u = tid + 512; u < groups; u += 256) {
        float v[16];
        bl_produce16_f32(pd, m, u, K, false, v);
#pragma unroll
        for (int e = 0; e < 16; ++e) part += (double)v[e] * (double)v[e];
    }
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) part += __shfl_xor(part, s);
    if ((tid & 63) == 0) s4[tid >> 6] = part;
    __syncthreads();
    const double ss = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    const float rn = (float)(1.0 / sqrt(ss / (double)K + (double)pd.eps));
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int u = tid + j * 256;
        if (u < groups) {
            float* v = tv[j];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = v[e] * rn;
            if (pd.gain) {
                const bl_v4f BL_G* g4 = bl_gc<bl_v4f>(pd.gain + (int64_t)u * 16);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bl_v4f g = g4[q];
                    v[4 * q] *= g.x; v[4 * q + 1] *= g.y; v[4 * q + 2] *= g.z; v[4 * q + 3] *= g.w;
                }
            }
            xv[2 * j] = make_uint4(bl_pack2_bf16(v[0], v[1]), bl_pack2_bf16(v[2], v[3]), bl_pack2_bf16(v[4], v[5]),
                                   bl_pack2_bf16(v[6], v[7]));
            xv[2 * j + 1] = make_uint4(bl_pack2_bf16(v[8], v[9]), bl_pack2_bf16(v[10], v[11]),
                                       bl_pack2_bf16(v[12], v[13]), bl_pack2_bf16(v[14], v[15]));
        }
    }
    return rn;
}

/* Four int8 in one dword: q = rint(f * inv), ties to even.  Adding 1.5 * 2^23 leaves the rounded
 * integer in the low bits of the sum (its unit in the last place is 1 there), so a value costs a
 * multiply, an add and three quarters of a byte permute.  With |f| <= gamma, fl(f * fl(127 / gamma)) never
 * rounds beyond 127, so what is clamped is a choice: BL_Q_ROW where f may be NaN (it becomes -127 and no other
 * value of the row changes), BL_Q_ANY for an inv that does not come from the absmax of these values,
 * BL_Q_FINITE where the row is known to be finite. */
enum { BL_Q_FINITE, BL_Q_ROW, BL_Q_ANY };
template <int MODE>
struct bl_mode {
    static constexpr int value = MODE;
};
template <int MODE>
__device__ __forceinline__ uint32_t bl_quant4(float f0, float f1, float f2, float f3, float inv) {
    float v[4] = {f0 * inv, f1 * inv, f2 * inv, f3 * inv};
    uint32_t r[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (MODE != BL_Q_FINITE) v[e] = fmaxf(v[e], -127.0f);
        if (MODE == BL_Q_ANY) v[e] = fminf(v[e], 127.0f);
        r[e] = __float_as_uint(v[e] + 12582912.0f);
    }
    return __builtin_amdgcn_perm(r[1], r[0], 0x0C0C0400u) | __builtin_amdgcn_perm(r[3], r[2], 0x04000C0Cu);
}

/* Quantise 8 bf16 (one uint4) to two dwords of int8. */
template <int MODE = BL_Q_FINITE>
__device__ __forceinline__ void bl_quant8_words(const uint4 v, float inv, uint32_t& lo, uint32_t& hi) {
    auto l = [](uint32_t w) { return __uint_as_float(w << 16); };
    auto h = [](uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); };
    lo = bl_quant4<MODE>(l(v.x), h(v.x), l(v.y), h(v.y), inv);
    hi = bl_quant4<MODE>(l(v.z), h(v.z), l(v.w), h(v.w), inv);
}

/* Largest magnitude of 8 bf16: without its sign a bf16 orders like its bit pattern, so the maxima are
 * taken two at a time on 16-bit integers.  SKIP: NaN are passed over; with 0x7F added infinity is 0x7FFF
 * and a NaN, whose pattern lies above infinity's, negative.  Otherwise a NaN is the largest. */
typedef short bl_v2s __attribute__((ext_vector_type(2)));
typedef unsigned short bl_v2us __attribute__((ext_vector_type(2)));
template <bool SKIP>
struct bl_mag2 {
    static constexpr uint32_t BIAS = SKIP ? 0x007F007Fu : 0u;
    uint32_t m = BIAS;
    __device__ __forceinline__ void take(uint32_t w) {
        w = (w & 0x7FFF7FFFu) + BIAS;
        if (SKIP) m = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(bl_v2s, m), __builtin_bit_cast(bl_v2s, w)));
        else m = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(bl_v2us, m), __builtin_bit_cast(bl_v2us, w)));
    }
    __device__ __forceinline__ float get() const {
        const uint32_t u = m - BIAS;
        return bl_max_pos(__uint_as_float(u << 16), __uint_as_float(u & 0xFFFF0000u));
    }
};
template <bool SKIP = false>
__device__ __forceinline__ float bl_absmax8_bf16(const uint4 v) {
    bl_mag2<SKIP> m;
    m.take(v.x);
    m.take(v.y);
    m.take(v.z);
    m.take(v.w);
    return m.get();
}

/* A row whose maximum, taken with NaN as the largest, is not finite: its maximum and its int8 values once more,
 * with NaN passed over.  Every other row is spared the look: in every row it cost a product of 16 tokens
 * 2560 x 2560 5.8 % (apart: 1.6), chains of two to eight tokens 1.9 - 3.2 % (0.3 - 2.0), a short stream 2 - 3 % (0 - 0.5).  get(u, lo, hi):
 * the sixteen bf16 of group u; row_max: the maximum over the threads of the row, which all come here; put(u, a0 .. a3):
 * overwrites what the same thread put before.  Returns g. */
template <typename Get, typename RowMax, typename Put>
__device__ __forceinline__ float bl_quant_row_again(int groups, int u0, int stride, Get get, RowMax row_max, Put put) {
    float mx = 0.0f;
    uint4 lo, hi;
#pragma unroll 1
    for (int u = u0; u < groups; u += stride) {
        get(u, lo, hi);
        mx = bl_max_pos(mx, bl_max_pos(bl_absmax8_bf16<true>(lo), bl_absmax8_bf16<true>(hi)));
    }
    const float g = fmaxf(row_max(mx), 1e-5f), inv = bl_div_rn(127.0f, g);
#pragma unroll 1
    for (int u = u0; u < groups; u += stride) {
        uint32_t a0, a1, a2, a3;
        get(u, lo, hi);
        bl_quant8_words<BL_Q_ROW>(lo, inv, a0, a1);
        bl_quant8_words<BL_Q_ROW>(hi, inv, a2, a3);
        put(u, a0, a1, a2, a3);
    }
    return g;
}
__device__ __forceinline__ bool bl_not_finite(float gamma) { return __builtin_expect(!(gamma < __builtin_inff()), 0); }

__device__ __forceinline__ int bl_sum16(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3) {
    int part = __builtin_amdgcn_sdot4((int)a0, 0x01010101, 0, false);
    part = __builtin_amdgcn_sdot4((int)a1, 0x01010101, part, false);
    part = __builtin_amdgcn_sdot4((int)a2, 0x01010101, part, false);
    return __builtin_amdgcn_sdot4((int)a3, 0x01010101, part, false);
}

/* Host side: public descriptor -> device form.  Returns false on a bad descriptor. */
static inline bool bl_make_prod(const bl_producer& p, const uint16_t* x_default, int64_t K, bl_prod_dev* out) {
    bl_prod_dev d = {};
    d.kind = p.kind;
    d.in0 = p.in0 ? p.in0 : (const void*)x_default;
    d.in1 = p.in1;
    d.aux_out = p.aux_out;
    d.norm = p.norm ? 1 : 0;
    d.gain = p.norm ? p.gain : nullptr;
    d.eps = p.eps;
    if (!d.in0) return false;
    if (p.norm && !(p.eps >= 0.0f)) return false;
    if (p.kind < BL_PROD_BF16 || p.kind > BL_PROD_RELU2_GATE) return false;
    if (p.kind == BL_PROD_RESIDUAL && !p.in1) return false;
    if (p.kind == BL_PROD_ATTN_V) {
        if (p.n_q <= 0 || p.n_kv <= 0 || p.head_dim <= 0 || p.n_q % p.n_kv || p.head_dim % 16 ||
            (int64_t)p.n_q * p.head_dim != K)
            return false;
        d.voff = (p.n_q + p.n_kv) * p.head_dim;
        d.group = p.n_q / p.n_kv;
        d.hd = p.head_dim;
        d.in_stride = (p.n_q + 2 * p.n_kv) * p.head_dim;
    }
    if (((uintptr_t)d.in0 | (uintptr_t)d.in1 | (uintptr_t)d.aux_out | (uintptr_t)d.gain) & 15) return false;
    *out = d;
    return true;
}
