/* Per-token absmax int8 activation quantisation (Section 2, "Activation
 * Quantization", of the BitNet b1.58 2B4T report).  HBM-bound at prefill sizes,
 * latency-bound at decode sizes. */
#include <type_traits>

#include "bl_device.h"
#include "bl_host.h"
#include "bl_producer.h"

#define QUANT_THREADS 256

/* Unit u (eight elements) of a bf16 row: zeros behind K (RAGGED: inside the unit too). */
template <bool RAGGED>
__device__ __forceinline__ uint4 bl_row_unit(const uint16_t* x, int u, int K) {
    const int full = K >> 3;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (u < full) {
        if (RAGGED) __builtin_memcpy(&v, x + u * 8, 16);
        else v = *(const uint4*)(x + u * 8);
    } else if (RAGGED && u == full) {
        uint32_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = u * 8 + j < K ? x[u * 8 + j] : 0u;
        v = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
    }
    return v;
}
template <int MODE>
__device__ __forceinline__ int bl_quant_unit(const uint4 v, float inv, int8_t* q, int sum) {
    uint2 o;
    bl_quant8_words<MODE>(v, inv, o.x, o.y);
    *(uint2*)q = o;
    sum = __builtin_amdgcn_sdot4((int)o.x, 0x01010101, sum, false);
    return __builtin_amdgcn_sdot4((int)o.y, 0x01010101, sum, false);
}

/* The quantiser of rows that exist as bf16.  TPR threads (64 or 256) share a row and hold all of it
 * in registers between the absmax and the rounding: NV units of eight elements each (K <= 8 * TPR *
 * NV), so the row is read once.  TPR = 64: a row is one wave's work, no LDS and no barrier.
 * RAGGED: K is not a multiple of 64; the row's start need not be 16-byte aligned (the 16-byte loads
 * are then unaligned ones), its last partial unit is read element by element, and the output row of
 * Kp = ceil(K/64)*64 bytes has zeros behind K.  KNOWN: the row maximum is given in absmax[m] (bits of
 * max |x|), read by every thread of the row and then cleared, so that the next product's epilogue
 * can fold its maxima into it again.
 * Bound by HBM at prefill sizes, else by the launch and the chain load -> maximum -> round -> store.
 * A row whose maximum is infinite or NaN (without looking, a NaN is the largest) is read again with NaN passed
 * over: looking in every row cost up to a tenth (2048 x 2560 3.8 -> 4.2 us).
 * Against one workgroup per row that read the row twice (and a ragged row in 2-byte loads): quantiser +
 * product at 777 x 2999 -> 5003 42.8 -> 38.4 us, the four of a layer at 2048 tokens 177.5 -> 174.2 us. */
template <int TPR, int NV, bool RAGGED, bool KNOWN>
__global__ __launch_bounds__(QUANT_THREADS) void bl_quant_rows(const uint16_t* __restrict__ X, int M, int K, int Kp,
                                                                int* __restrict__ absmax, int8_t* __restrict__ q,
                                                                float* __restrict__ scale, int32_t* __restrict__ rowsum) {
    constexpr int ROWS = QUANT_THREADS / TPR, WPR = TPR / BL_WAVE;   /* rows per workgroup, waves per row */
    __shared__ float smax[WPR];
    __shared__ int ssum[WPR];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int t = TPR == 64 ? lane : (int)threadIdx.x;               /* thread of the row */
    const int m = (int)blockIdx.x * ROWS + (TPR == 64 ? w : 0);
    if (m >= M) return;                                              /* (whole waves, and no barrier when ROWS > 1) */
    const uint16_t* x = X + (int64_t)m * K;
    int8_t* qo = q + (int64_t)m * Kp;
    const int units = Kp >> 3;
    uint4 v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = bl_row_unit<RAGGED>(x, t + i * TPR, K);
    auto row_max = [&](float mx) {                                   /* one barrier where several waves share the row */
        mx = bl_wave_max(mx);
        if (WPR > 1) {
            if (lane == 0) smax[w] = mx;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < WPR; ++i) mx = bl_max_pos(mx, smax[i]);
        }
        return mx;
    };
    float gamma;
    if (KNOWN) {
        gamma = __int_as_float(absmax[m]);
    } else {
        float mx = 0.0f;
#pragma unroll
        for (int i = 0; i < NV; ++i) mx = bl_max_pos(mx, bl_absmax8_bf16<false>(v[i]));
        gamma = row_max(mx);
    }
    float g, inv;
    int sum = 0;
    if (__builtin_expect(KNOWN || gamma < __builtin_inff(), 1)) {    /* (the same in every thread of the row) */
        g = fmaxf(gamma, 1e-5f);
        inv = bl_div_rn(127.0f, g);
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (t + i * TPR < units) sum = bl_quant_unit<KNOWN ? BL_Q_ANY : BL_Q_FINITE>(v[i], inv, qo + (t + i * TPR) * 8, sum);
    } else {
        float mx = 0.0f;
#pragma unroll 1
        for (int u = t; u < units; u += TPR) mx = bl_max_pos(mx, bl_absmax8_bf16<true>(bl_row_unit<RAGGED>(x, u, K)));
        if (WPR > 1) __syncthreads();                                /* smax has been read */
        g = fmaxf(row_max(mx), 1e-5f);
        inv = bl_div_rn(127.0f, g);
#pragma unroll 1
        for (int u = t; u < units; u += TPR) sum = bl_quant_unit<BL_Q_ROW>(bl_row_unit<RAGGED>(x, u, K), inv, qo + u * 8, sum);
    }
    sum = bl_wave_sum(sum);
    if (WPR > 1) {
        if (lane == 0) ssum[w] = sum;
        __syncthreads();                      /* (KNOWN: every thread has read absmax[m]) */
        sum = 0;
#pragma unroll
        for (int i = 0; i < WPR; ++i) sum += ssum[i];
    }
    if (t == 0) {
        if (KNOWN) absmax[m] = 0;
        scale[m] = bl_div_rn(g, 127.0f);
        if (rowsum) rowsum[m] = sum;
    }
}

/* Rows too long for the registers (K > 8192): one workgroup per row, read twice. */
template <bool RAGGED, bool KNOWN>
__global__ __launch_bounds__(QUANT_THREADS) void bl_quant_long(const uint16_t* __restrict__ X, int K, int Kp,
                                                                int* __restrict__ absmax, int8_t* __restrict__ q,
                                                                float* __restrict__ scale, int32_t* __restrict__ rowsum) {
    __shared__ float smax[QUANT_THREADS / BL_WAVE];
    __shared__ int ssum[QUANT_THREADS / BL_WAVE];
    const int64_t m = blockIdx.x;
    const uint16_t* x = X + m * K;
    int8_t* qo = q + m * Kp;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, units = Kp >> 3;
    auto row_absmax = [&](auto skip_nan) {
        float mx = 0.0f;
        for (int u = threadIdx.x; u < units; u += QUANT_THREADS)
            mx = bl_max_pos(mx, bl_absmax8_bf16<decltype(skip_nan)::value>(bl_row_unit<RAGGED>(x, u, K)));
        mx = bl_wave_max(mx);
        if (lane == 0) smax[w] = mx;
        __syncthreads();
        return bl_max_pos(bl_max_pos(smax[0], smax[1]), bl_max_pos(smax[2], smax[3]));
    };
    float g, inv;
    int sum = 0;
    auto quantise = [&](float gamma, auto mode) {
        g = fmaxf(gamma, 1e-5f);
        inv = bl_div_rn(127.0f, g);
        for (int u = threadIdx.x; u < units; u += QUANT_THREADS)
            sum = bl_quant_unit<decltype(mode)::value>(bl_row_unit<RAGGED>(x, u, K), inv, qo + u * 8, sum);
    };
    if (KNOWN) {
        quantise(__int_as_float(absmax[m]), bl_mode<BL_Q_ANY>{});
    } else {
        const float gamma = row_absmax(std::false_type{});
        if (__builtin_expect(gamma < __builtin_inff(), 1)) {
            quantise(gamma, bl_mode<BL_Q_FINITE>{});
        } else {
            __syncthreads();                  /* smax has been read */
            quantise(row_absmax(std::true_type{}), bl_mode<BL_Q_ROW>{});
        }
    }
    sum = bl_wave_sum(sum);
    if (lane == 0) ssum[w] = sum;
    __syncthreads();                          /* (KNOWN: every thread has read absmax[m]) */
    if (threadIdx.x == 0) {
        if (KNOWN) absmax[m] = 0;
        scale[m] = bl_div_rn(g, 127.0f);
        if (rowsum) rowsum[m] = (ssum[0] + ssum[1]) + (ssum[2] + ssum[3]);
    }
}

template <bool RAGGED, bool KNOWN>
static bl_status launch_quant(const uint16_t* X, int64_t M64, int64_t K64, int* absmax, int8_t* q, float* scale,
                              int32_t* rowsum, hipStream_t st) {
    const int M = (int)M64, K = (int)K64, Kp = (int)bl_kpad(K64);
    /* A row is one wave's work when the rows alone fill the chip, else four waves share it: with few rows, or
     * long ones, a wave's own chain of instructions is what takes the time.  One wave against four, 18 heights: K <= 1024
     * from 1024 rows on 0.51 - 0.97, K = 2048 0.85 - 1.0; K = 2560 .. 4096 below 2048 rows 0.95 - 1.25, from 2048 on
     * 0.86 - 1.06; K = 4160 .. 8192 0.94 - 1.46: never. */
    const bool wave_rows = Kp <= 2048 ? M >= 1024 : Kp <= 4096 && M >= 2048;
    const unsigned b4 = (unsigned)((M + 3) / 4), b1 = (unsigned)M;
    if (Kp > 8192)
        bl_quant_long<RAGGED, KNOWN><<<b1, QUANT_THREADS, 0, st>>>(X, K, Kp, absmax, q, scale, rowsum);
    else if (!wave_rows && Kp <= 4096)
        bl_quant_rows<256, 2, RAGGED, KNOWN><<<b1, QUANT_THREADS, 0, st>>>(X, M, K, Kp, absmax, q, scale, rowsum);
    else if (!wave_rows)
        bl_quant_rows<256, 4, RAGGED, KNOWN><<<b1, QUANT_THREADS, 0, st>>>(X, M, K, Kp, absmax, q, scale, rowsum);
    else if (Kp <= 2048)
        bl_quant_rows<64, 4, RAGGED, KNOWN><<<b4, QUANT_THREADS, 0, st>>>(X, M, K, Kp, absmax, q, scale, rowsum);
    else
        bl_quant_rows<64, 8, RAGGED, KNOWN><<<b4, QUANT_THREADS, 0, st>>>(X, M, K, Kp, absmax, q, scale, rowsum);
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}

/* Producer + quantiser: the bf16 row is produced on the fly (bl_produce16) and
 * kept in registers between the absmax pass and the quantise pass (two
 * 16-element groups per thread cover K <= 8192; longer rows are produced twice). */
template <bool NORM>
__global__ __launch_bounds__(QUANT_THREADS) void bl_quant_rows_ex(const bl_prod_dev pd, int K,
                                                                   int8_t* __restrict__ q, float* __restrict__ scale,
                                                                   int32_t* __restrict__ rowsum) {
    __shared__ float smax[QUANT_THREADS / BL_WAVE];
    __shared__ int ssum[QUANT_THREADS / BL_WAVE];
    __shared__ double snorm[4];
    static_assert(QUANT_THREADS == 256, "the normalisation tree has 256 leaves");
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int groups = K / 16;
    uint4 xv[4];
    float rn = 1.0f;
    if (NORM) rn = bl_norm_produce2(pd, m, K, true, snorm, xv);
    auto row_max = [&](float mx) {
        mx = bl_wave_max(mx);
        if (lane == 0) smax[w] = mx;
        __syncthreads();
        return bl_max_pos(bl_max_pos(smax[0], smax[1]), bl_max_pos(smax[2], smax[3]));
    };
    int8_t* qo = q + (int64_t)m * K;
    float g, inv;
    int sum = 0;
    auto put = [&](int u, const uint4 lo, const uint4 hi) {
        uint32_t a0, a1, a2, a3;
        bl_quant8_words(lo, inv, a0, a1);
        bl_quant8_words(hi, inv, a2, a3);
        sum += bl_sum16(a0, a1, a2, a3);
        *(uint4*)(qo + u * 16) = make_uint4(a0, a1, a2, a3);
    };
    float mx = 0.0f;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int u = tid + j * QUANT_THREADS;
        if (u < groups) {
            if (!NORM) bl_produce16<NORM>(pd, m, u, K, true, rn, xv[2 * j], xv[2 * j + 1]);
            mx = bl_max_pos(mx, bl_max_pos(bl_absmax8_bf16<false>(xv[2 * j]), bl_absmax8_bf16<false>(xv[2 * j + 1])));
        }
    }
    uint4 lo, hi;
    for (int u = tid + 2 * QUANT_THREADS; u < groups; u += QUANT_THREADS) {
        bl_produce16<NORM>(pd, m, u, K, true, rn, lo, hi);
        mx = bl_max_pos(mx, bl_max_pos(bl_absmax8_bf16<false>(lo), bl_absmax8_bf16<false>(hi)));
    }
    const float gamma = row_max(mx);
    if (!bl_not_finite(gamma)) {
        g = fmaxf(gamma, 1e-5f);
        inv = bl_div_rn(127.0f, g);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int u = tid + j * QUANT_THREADS;
            if (u < groups) put(u, xv[2 * j], xv[2 * j + 1]);
        }
        for (int u = tid + 2 * QUANT_THREADS; u < groups; u += QUANT_THREADS) {
            bl_produce16<NORM>(pd, m, u, K, false, rn, lo, hi);
            put(u, lo, hi);
        }
    } else {
        g = bl_quant_row_again(
            groups, tid, QUANT_THREADS, [&](int u, uint4& l, uint4& h) { bl_produce16<NORM>(pd, m, u, K, false, rn, l, h); },
            [&](float v) {
                __syncthreads();              /* smax has been read */
                return row_max(v);
            },
            [&](int u, uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3) {
                sum += bl_sum16(a0, a1, a2, a3);
                *(uint4*)(qo + u * 16) = make_uint4(a0, a1, a2, a3);
            });
    }
    sum = bl_wave_sum(sum);
    if (lane == 0) ssum[w] = sum;
    __syncthreads();
    if (tid == 0) {
        scale[m] = bl_div_rn(g, 127.0f);
        if (rowsum) {
            int t = 0;
#pragma unroll
            for (int i = 0; i < QUANT_THREADS / BL_WAVE; ++i) t += ssum[i];
            rowsum[m] = t;
        }
    }
}

extern "C" bl_status bl_quant_act_ex(const bl_producer* prod, int64_t M, int64_t K, int8_t* q, float* scale,
                                     int32_t* rowsum, bl_stream s) {
    if (!prod || !q || !scale) return BL_ERR_NULL;
    if (M < 1 || M > BL_MAX_DIM || K < 64 || K % 64 != 0 || K > BL_MAX_DIM) return BL_ERR_SHAPE;
    if (!bl_aligned(q, 16) || !bl_aligned(scale, 4) || !bl_aligned(rowsum, 4)) return BL_ERR_ALIGN;
    bl_prod_dev pd;
    if (!prod->in0) return BL_ERR_NULL;
    if (!bl_make_prod(*prod, nullptr, K, &pd)) return BL_ERR_VALUE;
    if (pd.norm) bl_quant_rows_ex<true><<<(unsigned)M, QUANT_THREADS, 0, (hipStream_t)s>>>(pd, (int)K, q, scale, rowsum);
    else bl_quant_rows_ex<false><<<(unsigned)M, QUANT_THREADS, 0, (hipStream_t)s>>>(pd, (int)K, q, scale, rowsum);
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}

/* Quantiser behind a fused producer epilogue: the bf16 row and its absmax already exist. */
extern "C" bl_status bl_quant_from_absmax(const uint16_t* X, float* absmax, int64_t M, int64_t K, int8_t* q,
                                          float* scale, int32_t* rowsum, bl_stream s) {
    if (!X || !absmax || !q || !scale) return BL_ERR_NULL;
    if (M < 1 || M > BL_MAX_DIM || K < 64 || K % 64 != 0 || K > BL_MAX_DIM) return BL_ERR_SHAPE;
    if (!bl_aligned(X, 16) || !bl_aligned(q, 16) || !bl_aligned(scale, 4) || !bl_aligned(rowsum, 4) ||
        !bl_aligned(absmax, 4))
        return BL_ERR_ALIGN;
    return launch_quant<false, true>(X, M, K, (int*)absmax, q, scale, rowsum, (hipStream_t)s);
}

extern "C" bl_status bl_quant_act_int8(const uint16_t* X, int64_t M, int64_t K, int8_t* q, float* scale,
                                       int32_t* rowsum, bl_stream s) {
    if (!X || !q || !scale) return BL_ERR_NULL;
    if (M < 1 || M > BL_MAX_DIM || K < 1 || K > BL_MAX_DIM) return BL_ERR_SHAPE;
    if (K % 64 != 0) {
        if (!bl_aligned(X, 2) || !bl_aligned(q, 16) || !bl_aligned(scale, 4) || !bl_aligned(rowsum, 4))
            return BL_ERR_ALIGN;
        return launch_quant<true, false>(X, M, K, nullptr, q, scale, rowsum, (hipStream_t)s);
    }
    if (!bl_aligned(X, 16) || !bl_aligned(q, 16) || !bl_aligned(scale, 4) || !bl_aligned(rowsum, 4))
        return BL_ERR_ALIGN;
    return launch_quant<false, false>(X, M, K, nullptr, q, scale, rowsum, (hipStream_t)s);
}
