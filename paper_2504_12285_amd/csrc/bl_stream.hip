/* Persistent streaming decode (Section 5.1 of the BitNet b1.58 2B4T report: the decode
 * kernel exists to minimise memory-bandwidth use, so the packed weights of a whole stack of
 * BitLinear products are streamed from HBM in ONE launch whose loads never stop).
 *
 * A table of products lives in device memory.  The grid is as many workgroups as stay
 * resident; each owns one contiguous slice of the table's weight bytes, cut at row-group
 * boundaries, so a workgroup meets one or two products and quantises / stages the activation
 * row of a product once, into LDS.  Inside a product the 128-bit weight loads are double-buffered:
 * the next loads are issued before the products of the ones that have landed.
 */
#include <string.h>

#include <atomic>
#include <type_traits>

#include <algorithm>
#include <queue>
#include <vector>

#include "bl_device.h"
#include "bl_gemm_choice.h"
#include "bl_gemv_common.h"
#include "bl_host.h"
#include "bl_producer.h"
#include "bl_stream_cut.h"
#include "bl_stream_index.h"

/* ---- device side -------------------------------------------------------------------------- */

/* (pointers read from the product table are cast to the global address space: BL_G) */
typedef bl_v4i BL_G bl_gv4i;

/* What the streaming kernel needs to know about one product (device memory). */
struct bl_stream_item {
    const bl_v4i* packed;
    const int8_t* q;          /* [K] int8: the caller's, or the preparation kernel's output */
    const float* scale;       /* [1] token part of the rescale factor (NULL: y is not wanted) */
    const int32_t* rowsum;    /* [1] sum_k q */
    const float* beta;
    const float* residual;    /* [N] or NULL */
    int32_t* acc;             /* [N] or NULL */
    float* y;                 /* [N] or NULL */
    const uint16_t* xbf16;    /* [K] bf16, or NULL: quantised by every workgroup that meets the product */
    int8_t* q_out;            /* xbf16 only: the caller's optional copies of q and absmax/127 */
    float* scale_out;
    float fixed_scale;        /* xbf16 only: > 0 replaces absmax/127 in the rescale */
    int N, nchunks, lp, layout, units;
    int lgG;                  /* one token, bl_stream_dot: log2 of the lanes per row */
    int lq, mod, lead;        /* one token: row groups to a block (log2), what their shifts come from (bl_group_shift), the largest shift */
    int parts;                /* one token: the row is read in this many parts of wave-wide loads (128 bytes of a row each) */
    int qgroups;              /* 16-byte groups of the quantised row (its padded length / 16) */
    int m;                    /* tokens of the entry (batched form; 1 otherwise) */
    int row_chunks, c0;       /* batched form: 16-byte chunks of a whole packed row; first chunk of the entry's k part */
    int ldq;                  /* batched form: bytes of a token row of q */
    /* k-major form only: partial sums of all workgroups, and what the finishing kernel reads */
    int32_t* acc_ws;          /* [N] int32, zero between runs */
    const int32_t* rowsum_fin;
    const float* scale_fin;
    int32_t* rowsum_pub;      /* bf16 input: where the owner workgroup publishes sum_k q and the scale */
    float* scale_pub;
};

/* What the preparation kernel needs: the fused producer + quantiser of one product. */
struct bl_stream_prep_item {
    bl_prod_dev prod;
    int fused;                /* 1: produce + quantise; 0: only the row sum of a given q is missing */
    const int8_t* q_in;       /* fused == 0 */
    int8_t* q_ws;             /* [K] quantised row (fused) */
    float* scale_ws;          /* [1] rescale factor's token part (fused) */
    int32_t* rowsum_ws;       /* [1] */
    int8_t* q_out;            /* caller's optional copies */
    float* scale_out;
    float fixed_scale;
    int K;
};

/* Preparation: one workgroup per table entry that needs it.  Fused entries: producer, RMS
 * normalisation (NORM), per-token absmax, int8 quantisation (Section 2) into the workspace,
 * with the caller's optional copies; int8 entries without a row sum: the row sum. */
template <bool NORM>
__global__ __launch_bounds__(256) void bl_stream_prep(const bl_stream_prep_item* __restrict__ items) {
    __shared__ float fs[4];
    __shared__ int ssum[4];
    __shared__ double s4[4];
    const bl_stream_prep_item& it = items[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int K = it.K, groups = K / 16;
    int part = 0;
    if (it.fused) {
        const bl_prod_dev pd = it.prod;
        uint4 xv[4];
        float rn = 1.0f;
        bool have_xv = false;
        if (NORM && pd.norm) {
            rn = bl_norm_produce2(pd, 0, K, true, s4, xv);
            have_xv = true;
        }
        float mx = 0.0f;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int u = tid + j * 256;
            if (u < groups) {
                if (!have_xv) bl_produce16<NORM>(pd, 0, u, K, true, rn, xv[2 * j], xv[2 * j + 1]);
                mx = bl_max_pos(mx, bl_max_pos(bl_absmax8_bf16(xv[2 * j]), bl_absmax8_bf16(xv[2 * j + 1])));
            }
        }
        for (int u = tid + 512; u < groups; u += 256) {
            uint4 lo, hi;
            bl_produce16<NORM>(pd, 0, u, K, false, rn, lo, hi);
            mx = bl_max_pos(mx, bl_max_pos(bl_absmax8_bf16(lo), bl_absmax8_bf16(hi)));
        }
        mx = bl_wave_max(mx);
        if (lane == 0) fs[w] = mx;
        __syncthreads();
        const float gamma = bl_max_pos(bl_max_pos(fs[0], fs[1]), bl_max_pos(fs[2], fs[3]));   /* (NaN is the largest) */
        float gg = fmaxf(gamma, 1e-5f);
        const float inv = bl_div_rn(127.0f, gg);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int u = tid + j * 256;
            if (u < groups) {
                uint32_t a0, a1, a2, a3;
                bl_quant8_words(xv[2 * j], inv, a0, a1);
                bl_quant8_words(xv[2 * j + 1], inv, a2, a3);
                part += bl_sum16(a0, a1, a2, a3);
                if (it.q_out) *(bl_v4i BL_G*)(it.q_out + u * 16) = bl_v4i{(int)a0, (int)a1, (int)a2, (int)a3};
                *(bl_v4i BL_G*)(it.q_ws + u * 16) = bl_v4i{(int)a0, (int)a1, (int)a2, (int)a3};
            }
        }
        for (int u = tid + 512; u < groups; u += 256) {
            uint32_t a0, a1, a2, a3;
            uint4 lo, hi;
            bl_produce16<NORM>(pd, 0, u, K, true, rn, lo, hi);
            bl_quant8_words(lo, inv, a0, a1);
            bl_quant8_words(hi, inv, a2, a3);
            part += bl_sum16(a0, a1, a2, a3);
            if (it.q_out) *(bl_v4i BL_G*)(it.q_out + u * 16) = bl_v4i{(int)a0, (int)a1, (int)a2, (int)a3};
            *(bl_v4i BL_G*)(it.q_ws + u * 16) = bl_v4i{(int)a0, (int)a1, (int)a2, (int)a3};
        }
        if (bl_not_finite(gamma)) {
            part = 0;
            gg = bl_quant_row_again(
                groups, tid, 256, [&](int u, uint4& lo, uint4& hi) { bl_produce16<NORM>(pd, 0, u, K, false, rn, lo, hi); },
                [&](float v) {
                    v = bl_wave_max(v);
                    __syncthreads();                       /* fs has been read */
                    if (lane == 0) fs[w] = v;
                    __syncthreads();
                    return bl_max_pos(bl_max_pos(fs[0], fs[1]), bl_max_pos(fs[2], fs[3]));
                },
                [&](int u, uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3) {
                    part += bl_sum16(a0, a1, a2, a3);
                    if (it.q_out) *(bl_v4i BL_G*)(it.q_out + u * 16) = bl_v4i{(int)a0, (int)a1, (int)a2, (int)a3};
                    *(bl_v4i BL_G*)(it.q_ws + u * 16) = bl_v4i{(int)a0, (int)a1, (int)a2, (int)a3};
                });
        }
        if (tid == 0) {
            const float sc = bl_div_rn(gg, 127.0f);
            *it.scale_ws = it.fixed_scale > 0.0f ? it.fixed_scale : sc;
            if (it.scale_out) *it.scale_out = sc;
        }
    } else {
        for (int u = tid; u < groups; u += 256) {
            const uint4 v = *(const uint4*)(it.q_in + (int64_t)u * 16);
            part += bl_sum16(v.x, v.y, v.z, v.w);
        }
    }
    part = bl_wave_sum(part);
    if (lane == 0) ssum[w] = part;
    __syncthreads();
    if (tid == 0) *it.rowsum_ws = (ssum[0] + ssum[1]) + (ssum[2] + ssum[3]);
}

/* ---- the stream kernel ----------------------------------------------------------------------
 * One token, so a weight meets one activation; the products run on the matrix cores all the same,
 * because the vector unit was what a wave waited for (~60 vector instructions per 16-byte load and
 * lane: masks and four-wide dot products; five weights per byte: ~100).
 *
 * v_mfma_f32_32x32x64_f8f6f4 with a 4-bit B operand takes 32 weights of a lane as they lie: a
 * packed word masked with 0x33333333 is eight nibbles 00cc, the e2m1 number c / 2, so a word costs
 * two masks and a shift.  The activation q = 16 a + b, -8 <= a <= 7, 0 <= b <= 15, is two 6-bit numbers:
 * e2m3 holds +-n / 8 exactly for n <= 16, with the code n itself.  Both pieces ride in one
 * instruction as two rows of A.  Every product is a multiple of 1/16 and every sum below 2^24 of
 * them (K <= 20480), so the fp32 accumulators hold the exact integers whatever the order.
 *
 * Loads keep the pattern that streams: eight consecutive lanes fetch 128 consecutive bytes of a
 * row, a wave-wide load covers eight rows (read alone 6.6 TB/s; 16 rows x 64 bytes, the order the
 * matrix core would like, 5.6, and 32 x 32 bytes 3.0).  Lane 8 r + u, which holds 16-byte chunk u
 * of the r-th row, is column 8 (r % 4) + u of B in k group r / 4.  Different columns need different
 * activations (chunk u's) and the two k groups hold different rows, so A has a row for each u
 * (8), k group (2) and piece (2), 32 together, zero in the other k group; of the 32 x 32 results
 * the one with the column's own u counts, and a row's eight chunks are added at the end.  The matrix
 * core computes 32 times what is wanted and is busy 15 % of the time (five per byte: 19 %).
 * Thirty layers of 2560 / 6912 in one launch: 88.9 -> 85.4 us in the 2-bit form (six tenths of it the order of the
 * loads, below), 107.4 -> 89.4 in the form of five per byte; sixty of 640 / 1280 20.7 -> 15.4 and 39.0 -> 17.5.
 * (Small tables and long rows stay on the vector unit: bl_stream_dot.h.)
 *
 * A product's quantised activation row lives in LDS for the workgroup (staged once per product
 * and workgroup: quantised from bf16 right there, or taken from the int8 row), as the 6-bit pieces
 * in operand order, and is read right before use.
 * Every workgroup that meets a bf16 product quantises the row for itself: nothing crosses
 * workgroups inside the launch.  (A hand-over through ready flags was measured and dropped:
 * fresh data needs either an L2 write-back + invalidate per wave, +40 us per launch, or
 * uncached loads of the row by every wave, +26 us; a separate preparation launch costs 5.5 us.)
 * LDS image: per 16-byte chunk of a weight row and per piece the A operands of the instructions that
 * multiply it, 24 bytes (32 codes) each: 96 bytes a chunk (2-bit form: even and odd bit pairs of the
 * four words) or 160 (five per byte: digits 0/1, 2/3, 4; 16 unused).  Both strides put the eight
 * chunks that a wave reads together on different banks.  Zeros from the row's end to the end of the
 * last part, and one zero chunk behind for the lanes of the other k group. */
#define BL_FORM_BIT2 0
#define BL_FORM_TRIT5 1
#define BL_B2_CHUNK 96
#define BL_T5_CHUNK 160
#define BL_T5_SET 24          /* bytes between the operands of a chunk and piece */

typedef int bl_v2i __attribute__((ext_vector_type(2)));
typedef int bl_v8i __attribute__((ext_vector_type(8)));
typedef float bl_v16f __attribute__((ext_vector_type(16)));

typedef uint32_t bl_u32a2 __attribute__((aligned(2)));
/* Eight activations (two dwords, in nibble order) -> 6 bytes of the operand at dst (low piece, q % 16) and
 * dst + piece_bytes (high piece, q >> 4).  A code is sign and magnitude in six bits: the low piece is its own
 * code, the high piece -8 .. 7 is h or, where negative, 32 | (16 - h).  Two codes are joined by a dot product
 * with 1 and 64.  NEG: of -q. */
template <bool NEG = false>
__device__ __forceinline__ void bl_lds_put8(uint8_t* dst, int piece_bytes, uint32_t x, uint32_t y) {
    auto put = [](uint8_t* p, uint32_t c0, uint32_t c1) {
        if (NEG) {
            c0 ^= 0x20202020u;
            c1 ^= 0x20202020u;
        }
        auto two = [](uint32_t c, uint32_t w, uint32_t add) { return __builtin_amdgcn_udot4(c, w, add, false); };
        const uint32_t z0 = two(c0, 0x00004001u, two(c0, 0x40010000u, 0u) << 12);
        const uint32_t z1 = two(c1, 0x00004001u, two(c1, 0x40010000u, 0u) << 12);
        *(bl_u32a2*)p = z0 | (z1 << 24);
        *(uint16_t*)(p + 4) = (uint16_t)(z1 >> 8);
    };
    auto high = [](uint32_t q) {
        const uint32_t s = (q >> 7) & 0x01010101u;
        const uint32_t h = ((q >> 4) & 0x0F0F0F0Fu) ^ ((s << 4) - s);
        return h + ((s << 5) + s);
    };
    put(dst, x & 0x0F0F0F0Fu, y & 0x0F0F0F0Fu);
    put(dst + piece_bytes, high(x), high(y));
}
/* 2-bit form: the sixteen activations k = 16 c16 .. + 15 (word c16 % 4 of chunk c16 / 4).  Nibble j of
 * the word masked at bit pair parity f is bit pair 2 j + f: weight 2 j + f in layout 0, weight
 * 4 (pair % 4) + pair / 4 in layout 1. */
__device__ __forceinline__ void bl_lds_put16(uint8_t* Qs, int c16, int layout, uint32_t a0, uint32_t a1, uint32_t a2,
                                             uint32_t a3) {
    uint8_t* const dst = Qs + (c16 >> 2) * BL_B2_CHUNK + (c16 & 3) * 6;
    if (layout == 0) {
        bl_lds_put8(dst, 48, __builtin_amdgcn_perm(a1, a0, 0x06040200u), __builtin_amdgcn_perm(a3, a2, 0x06040200u));
        bl_lds_put8(dst + 24, 48, __builtin_amdgcn_perm(a1, a0, 0x07050301u), __builtin_amdgcn_perm(a3, a2, 0x07050301u));
    } else {
        bl_lds_put8(dst, 48, __builtin_amdgcn_perm(a2, a0, 0x05010400u), __builtin_amdgcn_perm(a2, a0, 0x07030602u));
        bl_lds_put8(dst + 24, 48, __builtin_amdgcn_perm(a3, a1, 0x05010400u), __builtin_amdgcn_perm(a3, a1, 0x07030602u));
    }
}
/* Five per byte: the twenty activations of word wd, x[i] = those that meet digit i of its four bytes
 * (k = 20 wd + 4 i + 0..3).  A byte's two nibbles hold digits 0 and 1, or 2 and 3, or 4 and nothing; digit 4
 * comes with the other sign (bl_t5_digits). */
__device__ __forceinline__ void bl_lds_put20(uint8_t* Qs, int wd, const uint32_t* x) {
    constexpr int PIECE = BL_T5_CHUNK / 2;
    uint8_t* const dst = Qs + (wd >> 2) * BL_T5_CHUNK + (wd & 3) * 6;
    bl_lds_put8(dst, PIECE, __builtin_amdgcn_perm(x[1], x[0], 0x05010400u), __builtin_amdgcn_perm(x[1], x[0], 0x07030602u));
    bl_lds_put8(dst + BL_T5_SET, PIECE, __builtin_amdgcn_perm(x[3], x[2], 0x05010400u),
                __builtin_amdgcn_perm(x[3], x[2], 0x07030602u));
    bl_lds_put8<true>(dst + 2 * BL_T5_SET, PIECE, __builtin_amdgcn_perm(0u, x[4], 0x05010400u),
                      __builtin_amdgcn_perm(0u, x[4], 0x07030602u));
}

/* A barrier behind which the LDS writes in front of it are seen; loads stay in flight (__syncthreads waits for them). */
__device__ __forceinline__ void bl_lds_barrier() {
    asm volatile("" ::: "memory");
    BL_WAIT_LGKM0();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

/* The activations that meet one packed word, as they were loaded (nothing waits for them here): UD pairs of bf16
 * words, or, of an int8 row, UD dwords in x[.][0] (five per byte) or in the first sixteen bytes.  A row may end
 * inside a word of five or in front of one: the values behind `valid` dwords (which may be negative) are zeros. */
template <int FORM>
struct bl_unit {
    static constexpr int UD = FORM == BL_FORM_TRIT5 ? 5 : 4;
    bl_v2i x[UD];
    int valid;
    __device__ __forceinline__ void load(const uint16_t* xbf16, int wd, int dwords) {
        valid = bl_word_valid<UD>(wd, dwords);
        if constexpr (FORM == BL_FORM_TRIT5) {
            const bl_v2i BL_G* p = bl_gc<bl_v2i>(xbf16) + bl_word_first<UD>(wd, dwords);
#pragma unroll
            for (int i = 0; i < UD; ++i) x[i] = p[bl_word_dword(i, valid)];
        } else {
            const bl_gv4i* p = (const bl_gv4i*)xbf16 + wd * 2;
            const bl_v4i a = p[0], b = p[1];
            x[0] = bl_v2i{a[0], a[1]};
            x[1] = bl_v2i{a[2], a[3]};
            x[2] = bl_v2i{b[0], b[1]};
            x[3] = bl_v2i{b[2], b[3]};
        }
    }
    __device__ __forceinline__ void load_q(const int8_t* q, int wd, int dwords) {
        valid = bl_word_valid<UD>(wd, dwords);
        if constexpr (FORM == BL_FORM_TRIT5) {
            const int BL_G* p = bl_gc<int>(q) + bl_word_first<UD>(wd, dwords);
#pragma unroll
            for (int i = 0; i < UD; ++i) x[i] = bl_v2i{p[bl_word_dword(i, valid)], 0};
        } else {
            const bl_v4i a = ((const bl_gv4i*)q)[wd];
            x[0] = bl_v2i{a[0], a[1]};
            x[1] = bl_v2i{a[2], a[3]};
            x[2] = x[3] = bl_v2i{0, 0};
        }
    }
    __device__ __forceinline__ uint32_t get(int i, int e) const {
        return FORM == BL_FORM_BIT2 || i < valid ? (uint32_t)x[i][e] : 0u;
    }
    __device__ __forceinline__ uint32_t get_q(int i) const {
        return FORM == BL_FORM_BIT2 ? (uint32_t)x[i >> 1][i & 1] : get(i, 0);
    }
    template <bool SKIP>
    __device__ __forceinline__ float absmax() const {
        bl_mag2<SKIP> m;
#pragma unroll
        for (int i = 0; i < UD; ++i) {
            m.take(get(i, 0));
            m.take(get(i, 1));
        }
        return m.get();
    }
    template <int MODE>
    __device__ __forceinline__ void quant(float inv, uint32_t* a) const {
        auto l = [](uint32_t w) { return __uint_as_float(w << 16); };
        auto h = [](uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); };
#pragma unroll
        for (int i = 0; i < UD; ++i)
            a[i] = bl_quant4<MODE>(l(get(i, 0)), h(get(i, 0)), l(get(i, 1)), h(get(i, 1)), inv);
    }
};

/* What a workgroup reads of a product besides its weights, requested in front of the first of them: loads arrive in
 * order, and the weights take longer. */
template <int FORM>
struct bl_row {
    bl_unit<FORM> x[2];       /* this thread's first two words' activations (all of them up to K = 8192) */
    int rowsum;
    float scale, beta;
};

/* Stages the activation row of P: Qs = the image above, misc[0] = what the sum of a row's products is
 * taken from (2-bit form: sum_k q, subtracted; five per byte: sum_k q with digit 4's terms negative, the
 * products are subtracted), misc[1] = token part of the rescale factor (float bits).  The waves meet at barriers that
 * wait for LDS alone: the first weights stay in flight.  Ends with a barrier. */
template <int FORM, int LP>
__device__ __forceinline__ void bl_stream_stage(const bl_stream_item& P, const bl_row<FORM>& row,
                                                    uint8_t* __restrict__ Qs, int* __restrict__ misc, bool owner) {
    constexpr int CHUNK = FORM == BL_FORM_TRIT5 ? BL_T5_CHUNK : BL_B2_CHUNK, UD = bl_unit<FORM>::UD;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));          /* nothing of this is worth a register outside (the compiler would hoist it and spill) */
    const int lane = tid & 63, w = tid >> 6;
    const int words = P.nchunks * 4, dwords = P.qgroups * 4;
    float* fs = (float*)(misc + 2);
    int* ssum = misc + 6;
    /* zeros in front of and behind the row, see bl_stream_slice */
    {
        const int lead = P.lead * CHUNK / 16, tail = (P.lead + P.nchunks) * CHUNK / 16,
                  all = (P.lead + P.parts * LP * 8 + 1) * CHUNK / 16;
#pragma unroll 1
        for (int i = tid; i < lead + all - tail; i += 256)
            ((bl_v4i*)Qs)[i < lead ? i : i - lead + tail] = bl_v4i{0, 0, 0, 0};
    }
    uint8_t* const img = Qs + P.lead * CHUNK;
    int part = 0;
    auto place = [&](int wd, const uint32_t* a) __attribute__((always_inline)) {
        if constexpr (FORM == BL_FORM_TRIT5) bl_lds_put20(img, wd, a);
        else bl_lds_put16(img, wd, P.layout, a[0], a[1], a[2], a[3]);
    };
    if (P.xbf16) {
        auto all_max = [&](float v) {
            v = bl_wave_max(v);
            if (lane == 0) fs[w] = v;
            bl_lds_barrier();
            return bl_max_pos(bl_max_pos(fs[0], fs[1]), bl_max_pos(fs[2], fs[3]));
        };
        float inv = 0.0f;
        auto put = [&](const bl_unit<FORM>& x, int wd, auto mode) __attribute__((always_inline)) {
            uint32_t a[UD];
            x.template quant<decltype(mode)::value>(inv, a);
#pragma unroll
            for (int i = 0; i < UD; ++i) part = __builtin_amdgcn_sdot4((int)a[i], i < 4 ? 0x01010101 : -1, part, false);
            if (owner && P.q_out) {
                if constexpr (FORM == BL_FORM_TRIT5) {
#pragma unroll
                    for (int i = 0; i < UD; ++i)
                        if (wd * UD + i < dwords) bl_g((uint32_t*)P.q_out)[wd * UD + i] = a[i];
                } else {
                    ((bl_gv4i*)P.q_out)[wd] = bl_v4i{(int)a[0], (int)a[1], (int)a[2], (int)a[3]};
                }
            }
            place(wd, a);
        };
        float mx = bl_max_pos(row.x[0].template absmax<false>(), row.x[1].template absmax<false>());
#pragma unroll 1
        for (int wd = tid + 512; wd < words; wd += 256) {
            bl_unit<FORM> y;
            y.load(P.xbf16, wd, dwords);
            mx = bl_max_pos(mx, y.template absmax<false>());
        }
        const float gamma = all_max(mx);                       /* (NaN is the largest) */
        float gg = fmaxf(gamma, 1e-5f);
        if (!bl_not_finite(gamma)) {
            inv = bl_div_rn(127.0f, gg);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (tid + j * 256 < words) put(row.x[j], tid + j * 256, bl_mode<BL_Q_FINITE>{});
#pragma unroll 1
            for (int wd = tid + 512; wd < words; wd += 256) {
                bl_unit<FORM> y;
                y.load(P.xbf16, wd, dwords);
                put(y, wd, bl_mode<BL_Q_FINITE>{});
            }
        } else {                                               /* once more, with NaN passed over */
            mx = 0.0f;
#pragma unroll 1
            for (int wd = tid; wd < words; wd += 256) {
                bl_unit<FORM> y;
                y.load(P.xbf16, wd, dwords);
                mx = bl_max_pos(mx, y.template absmax<true>());
            }
            bl_lds_barrier();                                   /* fs has been read */
            gg = fmaxf(all_max(mx), 1e-5f);
            inv = bl_div_rn(127.0f, gg);
#pragma unroll 1
            for (int wd = tid; wd < words; wd += 256) {
                bl_unit<FORM> y;
                y.load(P.xbf16, wd, dwords);
                put(y, wd, bl_mode<BL_Q_ROW>{});
            }
        }
        if (tid == 0) {
            const float sc = bl_div_rn(gg, 127.0f);
            misc[1] = __float_as_int(P.fixed_scale > 0.0f ? P.fixed_scale : sc);
            if (owner && P.scale_out) *(float BL_G*)P.scale_out = sc;
        }
        part = bl_wave_sum(part);
        if (lane == 0) ssum[w] = part;
        bl_lds_barrier();
        if (tid == 0) misc[0] = (ssum[0] + ssum[1]) + (ssum[2] + ssum[3]);
    } else {
        auto take = [&](const bl_unit<FORM>& y, int wd) __attribute__((always_inline)) {
            uint32_t a[UD];
#pragma unroll
            for (int i = 0; i < UD; ++i) a[i] = y.get_q(i);
            if constexpr (FORM == BL_FORM_TRIT5) part = __builtin_amdgcn_sdot4((int)a[4], 0x01010101, part, false);
            place(wd, a);
        };
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (tid + j * 256 < words) take(row.x[j], tid + j * 256);
#pragma unroll 1
        for (int wd = tid + 512; wd < words; wd += 256) {
            bl_unit<FORM> y;
            y.load_q(P.q, wd, dwords);
            take(y, wd);
        }
        if constexpr (FORM == BL_FORM_TRIT5) {
            part = bl_wave_sum(part);
            if (lane == 0) ssum[w] = part;
            bl_lds_barrier();
        }
        if (tid == 0) {
            misc[0] = FORM == BL_FORM_TRIT5 ? row.rowsum - 2 * ((ssum[0] + ssum[1]) + (ssum[2] + ssum[3])) : row.rowsum;
            misc[1] = __float_as_int(row.scale);
        }
    }
    bl_lds_barrier();
}

/* ---- five weights per byte (BL_LAYOUT_TRIT5) ---------------------------------------------------
 * A byte b = ceil(v * 256 / 243) holds v = sum_i c_i * 3^(4-i), five offset codes c_i in {0,1,2}.
 * Multiplying by 9 moves the two leading base-3 digits, as one number 0..8, into bits 8..11 and leaves
 * the rest in the low byte.  The four bytes of a word are handled as two pairs in 16-bit lanes (a byte
 * times 9 fits 12 bits); a byte permute gathers the four numbers, and another uses them as selectors
 * into an eight-byte table of both digits as two 4-bit numbers: the B operand.  Selector 8 replicates
 * the sign of table byte 1; the table holds 2 - c, so that entry 8 is zero and no sign is set.  The
 * last digit c is an operand as it is, against -q: sum_k W q = sum q (its own digit positions negative) -
 * sum (2 - c) q + sum c q.  17 vector instructions per 20 weights, each four clocks of a wave; they are what the
 * kernel waits for (without them the 30-layer table takes 74 us). */
__device__ __forceinline__ void bl_t5_digits(const uint32_t w, int& d01, int& d23, int& d4) {
    uint32_t mask = 0x00FF00FFu, nine = 9, three = 3;
    asm("" : "+s"(mask), "+s"(nine), "+s"(three));          /* (in scalar registers; or the multiplications become shift-and-add) */
    uint32_t e = w & mask, o = __builtin_amdgcn_perm(0u, w, 0x0C030C01u);
    auto two = [&]() {
        e = __umul24(e, nine);
        o = __umul24(o, nine);
        const uint32_t t = __builtin_amdgcn_perm(o, e, 0x07030501u);        /* bits 8..15 of the four lanes */
        e &= mask;
        o &= mask;
        return (int)__builtin_amdgcn_perm(0x10200111u, 0x21021222u, t);     /* (2 - t / 3) | (2 - t % 3) << 4 */
    };
    d01 = two();
    d23 = two();
    e = __umul24(e, three);
    o = __umul24(o, three);
    d4 = (int)__builtin_amdgcn_perm(o, e, 0x07030501u);
}

/* One product slice [ub, ue) of row groups of eight weight rows (eight consecutive ones, or CLASSES).  A row group is read in P.parts
 * parts of LP wave-wide loads; each of the four waves of the workgroup takes a contiguous quarter of the
 * row groups (round-robin, the workgroups read in step at one stride, which may be that of few
 * memory channels: sixty products of 13824 x 2560 100 us against 86) and
 * keeps one part in flight while another is multiplied.  Every load of the steady loop
 * is unconditional (out-of-range lanes read a clamped, valid address and meet zero activations,
 * or are never stored), so the hardware counter waits are exact and the loads of the next part
 * stay in flight during the products of this one.  The residual value of a row travels
 * with the row's weights: a load issued later, in the epilogue, could only be waited for
 * together with every weight load issued before it (with no residual every lane reads beta
 * instead, a valid address, and the value is not used). */
template <int FORM, int LP, bool CLASSES>
__device__ __forceinline__ void bl_stream_slice(const bl_stream_item& P, const int ub, const int ue,
                                                    uint8_t* __restrict__ Qs, int* __restrict__ misc,
                                                    const bool restage) {
    constexpr int CHUNK = FORM == BL_FORM_TRIT5 ? BL_T5_CHUNK : BL_B2_CHUNK;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = P.N, parts = P.parts;
    /* Lanes 0..31 take the rows of the even class of a row group, 32..63 those of the odd one.  The loads of a class that does not
     * start with a 128-byte line, and its k group of A, are bl_group_shift chunks back, so that every load of a row is one line
     * (P.lead zero chunks in front of the image): at K = 6912 odd rows by 4; with lq > 0 classes that differ from row group to
     * row group.  Where mod is 0 and rows still lie across lines they are read as they lie. */
    const int u = lane & 7, h = lane >> 5, lq = CLASSES ? P.lq : 0, mod = P.mod;
    const int r = bl_group_row((lane >> 3) & 3, h, lq);
    const int row_bytes = P.nchunks * 16;
    const char BL_G* const wbase = (const char BL_G*)P.packed;
    int32_t BL_G* const acc_g = (int32_t BL_G*)P.acc;
    float BL_G* const y_g = (float BL_G*)P.y;
    const float BL_G* const res_g = (const float BL_G*)P.residual;
    const int each = (ue - ub) >> 2, extra = (ue - ub) & 3;
    const int mine = each + (w < extra ? 1 : 0);         /* row groups of this wave (may be 0) */
    const int first = ub + w * each + (w < extra ? w : extra);
    int irg = first, ipart = 0;                          /* issue cursor */
    /* Lanes behind their row's end read its last chunk again, which meets zero activations (the next row's chunks would
     * do as well, but are fetched twice then: 60 layers of 640 / 1280 16.4 us against 15.4); a
     * shifted load in front of a row reads the end of the row before.  Rows behind N are held inside the matrix
     * and not stored.  Behind the wave's last row group every lane reads the first bytes of that row group once more: one
     * line, and the loop needs no second copy of itself without loads. */
    const int bias = P.lead * 16, row_end = r * row_bytes + row_bytes - 16 + bias;
    int rows = N - bl_group_base(first, lq);             /* rows from this row group's first one on */
    const char BL_G* rg_at = wbase + (int64_t)(N - rows) * row_bytes - bias;
    const float BL_G* rv_at = res_g ? res_g + (N - rows) : (const float BL_G*)P.beta;
    int ishift = bl_group_shift(first, h, lq, mod);
    int lane_off[LP];
#pragma unroll
    for (int i = 0; i < LP; ++i) lane_off[i] = r * row_bytes + (u - ishift) * 16 + bias + i * 128;
    auto issue = [&](bl_v4i* p, float& rv) {
        const bool over = irg == first + mine;
        const int part_at = ipart * (LP * 128);
        const int end = row_end - part_at;
        int limit = over ? 0 : bl_part_limit(rows, row_bytes, part_at, bias, lq);
        asm("" : "+s"(limit));                           /* (one scalar, not a select per lane and load) */
        const int back = bl_group_next(irg - 1, lq);     /* rows back to the row group in front */
        const char BL_G* const base = rg_at + (over ? bias - back * row_bytes : part_at);
#pragma unroll
        for (int i = 0; i < LP; ++i)
            p[i] = __builtin_nontemporal_load(
                (const bl_gv4i*)(base + (uint32_t)min(min(lane_off[i], end), limit)));
        const int rlim = res_g ? (over ? -back : rows - 1) : 0;
        rv = rv_at[min(r, rlim)];
        const bool next = !over && ++ipart == parts;
        const int skip = next ? bl_group_next(irg, lq) : 0;
        ipart = next ? 0 : ipart;
        irg += next ? 1 : 0;
        rows -= skip;
        rg_at += (int64_t)skip * row_bytes;
        rv_at += res_g ? skip : 0;
        const int was = ishift;
        ishift = bl_group_shift(irg, h, lq, mod);
#pragma unroll
        for (int i = 0; i < LP; ++i) lane_off[i] += (was - ishift) * 16;
    };
    bl_v4i pa[LP], pb[LP];
    float ra = 0.0f, rb = 0.0f;
    bl_row<FORM> row;
    row.rowsum = 0;
    row.scale = 0.0f;
    auto word = [&](int j) {                             /* (word 0 again does not change the maximum) */
        const int wd = (int)threadIdx.x + j * 256;
        return wd < P.nchunks * 4 ? wd : 0;
    };
    if (P.xbf16) {
        row.x[0].load(P.xbf16, word(0), P.qgroups * 4);
        row.x[1].load(P.xbf16, word(1), P.qgroups * 4);
    } else {
        row.x[0].load_q(P.q, word(0), P.qgroups * 4);
        row.x[1].load_q(P.q, word(1), P.qgroups * 4);
        row.rowsum = *bl_gc<int32_t>(P.rowsum);
        row.scale = *bl_gc<float>(P.scale ? P.scale : P.beta);
    }
    row.beta = *bl_gc<float>(P.beta);
    asm volatile("" ::: "memory");
    issue(pa, ra);                                       /* in flight during the staging */
    if (restage) bl_lds_barrier();                       /* every wave is done with the previous image */
    bl_stream_stage<FORM, LP>(P, row, Qs, misc, ub == 0);
    if (mine == 0) return;
    const int rs = misc[0];
    float cf = 0.0f;
    if (y_g) cf = row.beta * __int_as_float(misc[1]);

    /* this lane of A: chunk u, k group (lane / 8) % 2, piece (lane / 16) % 2; zeros in the other k group */
    const bool live = ((lane >> 3) & 1) == h;
    const int a_chunk = live ? CHUNK : 0, a_step = live ? 8 * CHUNK : 0;
    const int a_first = live ? (u + P.lead) * CHUNK + ((lane >> 4) & 1) * (CHUNK / 2) : (P.lead + parts * LP * 8) * CHUNK;
    const int live_loads = (P.nchunks + P.lead + 7) / 8 - (parts - 1) * LP;
    int ppart = 0, prg = first, prow = bl_group_base(first, lq);   /* process cursor */
    int at = a_first - bl_group_shift(prg, h, lq, mod) * a_chunk;
    const int store_row = u == 0 ? r : 1 << 30;          /* one lane of eight stores */
    bl_v16f D = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    auto step = [&](const bl_v4i* p, const float rv) {
        /* The image does not change inside the loop, so the compiler could hoist these reads
         * out of it and hold them in registers: the address is hidden from it. */
        asm volatile("" : "+v"(at));
#pragma unroll
        for (int i = 0; i < LP; ++i) {
            if (i > 0 && i >= live_loads && ppart == parts - 1) break;   /* idle slots of the last part */
            /* (one load's operands at a time: with all of them in flight the loop spills) */
            __builtin_amdgcn_sched_barrier(0);
            const uint8_t* const q = Qs + at;
            at += a_step;
            auto operand = [&](int o) {                      /* 24 bytes, at a multiple of 16 or 8 behind one */
                asm volatile("" ::: "memory");               /* (eight bytes of two operands in one read cost four moves) */
                const bool first8 = o % 16 != 0;
                const bl_v4i x = *(const bl_v4i*)(q + o + (first8 ? 8 : 0));
                const bl_v2i y = *(const bl_v2i*)(q + o + (first8 ? 0 : 16));
                return first8 ? bl_v8i{y[0], y[1], x[0], x[1], x[2], x[3], 0, 0} : bl_v8i{x[0], x[1], x[2], x[3], y[0], y[1], 0, 0};
            };
            /* (the first product of a row group starts from zero) */
            auto first_mul = [&](const bl_v8i& a, const bl_v8i& b) {
                if (i == 0 && ppart == 0) {
                    bl_v16f z = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                    D = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, z, 2, 4, 0, 0, 0, 0);
                } else {
                    D = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, D, 2, 4, 0, 0, 0, 0);
                }
            };
            if constexpr (FORM == BL_FORM_BIT2) {
                bl_v8i b0 = {0, 0, 0, 0, 0, 0, 0, 0}, b1 = b0;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const uint32_t wd = (uint32_t)p[i][d];
                    b0[d] = (int)(wd & 0x33333333u);
                    b1[d] = (int)((wd >> 2) & 0x33333333u);
                }
                first_mul(operand(0), b0);
                D = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand(24), b1, D, 2, 4, 0, 0, 0, 0);
            } else {
                bl_v8i b0 = {0, 0, 0, 0, 0, 0, 0, 0}, b1 = b0, b2 = b0;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    int d01, d23, d4;
                    bl_t5_digits((uint32_t)p[i][d], d01, d23, d4);
                    b0[d] = d01;
                    b1[d] = d23;
                    b2[d] = d4;
                }
                first_mul(operand(0), b0);
                D = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand(BL_T5_SET), b1, D, 2, 4, 0, 0, 0, 0);
                D = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand(2 * BL_T5_SET), b2, D, 2, 4, 0, 0, 0, 0);
            }
        }
        /* (pinned: otherwise the last product goes to other registers than the accumulators that the next one starts from) */
        asm volatile("" : "+v"(D));
        if (++ppart < parts) return;
        /* element v of lane l: A row (v % 4) + 8 (v / 4) + 4 (l / 32), i.e. chunk u = v % 4 + 4 (l / 32),
         * k group v / 4 % 2, piece v / 8, against column l % 32.  A lane's own chunk is element u % 4 where
         * u / 4 is its half. */
        bl_mfma_fence();
        float S[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            float e[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) e[j] = __builtin_fmaf(D[8 + 4 * g + j], 16.0f, D[4 * g + j]);
            S[g] = (u & 2) ? ((u & 1) ? e[3] : e[2]) : ((u & 1) ? e[1] : e[0]);
        }
        /* lower lanes: the even rows of the group, upper lanes: the odd ones */
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(S[0]), __float_as_uint(S[1]), false, false);
        float t = __uint_as_float(u < 4 ? sw[0] : sw[1]);
        t += bl_dppf<BL_DPP_QUAD_XOR1>(t);
        t += bl_dppf<BL_DPP_QUAD_XOR2>(t);
        t += bl_dppf<BL_DPP_ROW_HALF_MIRROR>(t);
        const int v = (int)(t * 16.0f);
        if (store_row < N - prow) {
            const int val = FORM == BL_FORM_TRIT5 ? rs - v : v - rs;
            if (acc_g) acc_g[(int64_t)prow + (uint32_t)store_row] = val;
            if (y_g) {
                const float o = (float)val * cf;
                y_g[(int64_t)prow + (uint32_t)store_row] = res_g ? rv + o : o;
            }
        }
        ppart = 0;
        prow += bl_group_next(prg, lq);
        ++prg;
        at = a_first - bl_group_shift(prg, h, lq, mod) * a_chunk;
    };
    for (int left = mine * parts;;) {
        issue(pb, rb);
        step(pa, ra);
        if (--left == 0) break;
        issue(pa, ra);
        step(pb, rb);
        if (--left == 0) break;
    }
}

/* Persistent grid: workgroup b walks the table slice wgstart[b] .. wgstart[b+1], each entry
 * (product, row group).  One part length per table: the host takes the one that leaves the fewest
 * load slots idle (a row whose loads do not divide by it re-reads its last chunk, a cache hit).
 * Four waves per SIMD, no scratch memory: a version that spilled lost a third of the stream rate. */
template <int FORM, int LP, bool CLASSES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
void bl_stream_m1(const bl_stream_item* __restrict__ items, const int2* __restrict__ wgstart, const int q_ints) {
    extern __shared__ __attribute__((aligned(16))) int lds[];   /* q_ints ints of image + 16 */
    uint8_t* Qs = (uint8_t*)lds;
    int* misc = lds + q_ints;
    const int2 s0 = wgstart[blockIdx.x], s1 = wgstart[blockIdx.x + 1];
    const int p_first = __builtin_amdgcn_readfirstlane(s0.x), u_first = __builtin_amdgcn_readfirstlane(s0.y);
    const int p_last = __builtin_amdgcn_readfirstlane(s1.x), u_last = __builtin_amdgcn_readfirstlane(s1.y);
    bool staged = false;
    for (int pi = p_first; pi <= p_last; ++pi) {
        if (pi == p_last && u_last == 0) break;
        const bl_stream_item P = items[pi];
        const int ub = pi == p_first ? u_first : 0;
        const int ue = pi == p_last ? u_last : P.units;
        if (ub >= ue) continue;
        bl_stream_slice<FORM, LP, CLASSES>(P, ub, ue, Qs, misc, staged);
        staged = true;
    }
}

#include "bl_stream_dot.h"

/* ---- k-major form (BL_LAYOUT_KMAJOR): skipping the weights of zero activations -----------------
 * Section 2 of the report takes squared ReLU in the feed-forward block for the sparsity it gives
 * the activations of the down projection.  Stored k-major (one row of N codes per input feature k),
 * the weights of a zero activation are simply not read.  A wave takes 64 consecutive k, finds the
 * non-zero activations with one ballot and walks them four at a time: lane l loads its dword
 * (16 output features) from each of the four rows, a byte permute puts the same byte of the four
 * rows side by side, and the mask-only level trick of the other kernels turns that into operands
 * of v_dot4_i32_i8 against the four activations (uniform, so they sit in a scalar register).
 * Every workgroup holds partial sums over its own k range: they meet in LDS, then in an int32
 * array in device memory (integer atomics: exact, order-free), and a small finishing kernel
 * subtracts the row sum, rescales, adds the residual and clears the array for the next run. */
template <int CB>
__device__ __forceinline__ void bl_km_slice(const bl_stream_item& P, const int ub, const int ue,
                                                int* __restrict__ Qs, int* __restrict__ misc,
                                                int* __restrict__ red, const bool restage) {
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ncols = P.nchunks, N = P.N;
    const uint32_t BL_G* const wbase = (const uint32_t BL_G*)P.packed;
    int col[CB];
    bool ok[CB];
#pragma unroll
    for (int j = 0; j < CB; ++j) {
        const int c = 64 * j + lane;
        ok[j] = c < ncols;
        col[j] = ok[j] ? c : ncols - 1;
    }
    if (restage) __syncthreads();
    /* the int8 row in its natural order, zeros up to the end of the last 64-wide k block */
    {
        const int groups = P.qgroups, lw = tid >> 6;
        float* fs = (float*)(misc + 2);
        int* ssum = misc + 6;
        bl_v4i* Q4 = (bl_v4i*)Qs;
        for (int u = groups + tid; u < P.units * 4; u += 256) Q4[u] = bl_v4i{0, 0, 0, 0};
        for (int n = tid; n < ncols * 16; n += 256) red[n] = 0;
        if (P.xbf16) {
            const bl_gv4i* x = (const bl_gv4i*)P.xbf16;
            auto ld = [&](int i) {
                const bl_v4i v = x[i];
                return make_uint4((uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3]);
            };
            float mx = 0.0f;
            for (int u = tid; u < groups; u += 256)
                mx = bl_max_pos(mx, bl_max_pos(bl_absmax8_bf16(ld(2 * u)), bl_absmax8_bf16(ld(2 * u + 1))));
            mx = bl_wave_max(mx);
            if (lane == 0) fs[lw] = mx;
            __syncthreads();
            const float gamma = bl_max_pos(bl_max_pos(fs[0], fs[1]), bl_max_pos(fs[2], fs[3]));   /* (NaN is the largest) */
            float gg = fmaxf(gamma, 1e-5f);
            const float inv = bl_div_rn(127.0f, gg);
            int part = 0;
            for (int u = tid; u < groups; u += 256) {
                uint32_t a0, a1, a2, a3;
                bl_quant8_words(ld(2 * u), inv, a0, a1);
                bl_quant8_words(ld(2 * u + 1), inv, a2, a3);
                part += bl_sum16(a0, a1, a2, a3);
                const bl_v4i qv = {(int)a0, (int)a1, (int)a2, (int)a3};
                if (ub == 0 && P.q_out) *(bl_gv4i*)(P.q_out + u * 16) = qv;
                Q4[u] = qv;
            }
            if (bl_not_finite(gamma)) {
                part = 0;
                gg = bl_quant_row_again(
                    groups, tid, 256, [&](int u, uint4& lo, uint4& hi) {
                        lo = ld(2 * u);
                        hi = ld(2 * u + 1);
                    },
                    [&](float v) {
                        v = bl_wave_max(v);
                        __syncthreads();                       /* fs has been read */
                        if (lane == 0) fs[lw] = v;
                        __syncthreads();
                        return bl_max_pos(bl_max_pos(fs[0], fs[1]), bl_max_pos(fs[2], fs[3]));
                    },
                    [&](int u, uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3) {
                        part += bl_sum16(a0, a1, a2, a3);
                        const bl_v4i qv = {(int)a0, (int)a1, (int)a2, (int)a3};
                        if (ub == 0 && P.q_out) *(bl_gv4i*)(P.q_out + u * 16) = qv;
                        Q4[u] = qv;
                    });
            }
            part = bl_wave_sum(part);
            if (lane == 0) ssum[lw] = part;
            __syncthreads();
            if (tid == 0 && ub == 0) {
                const float sc = bl_div_rn(gg, 127.0f);
                *(int32_t BL_G*)P.rowsum_pub = (ssum[0] + ssum[1]) + (ssum[2] + ssum[3]);
                *(float BL_G*)P.scale_pub = P.fixed_scale > 0.0f ? P.fixed_scale : sc;
                if (P.scale_out) *(float BL_G*)P.scale_out = sc;
            }
        } else {
            const bl_gv4i* qg = (const bl_gv4i*)P.q;
            for (int u = tid; u < groups; u += 256) Q4[u] = qg[u];
        }
        __syncthreads();
    }
    int A[CB][4][4];
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int t = 0; t < 4; ++t) A[j][b][t] = 0;

    /* the stream of (four non-zero activations, their weight dwords): one step ahead of the arithmetic */
    int u = ub + w, k0 = 0, qv = 0;
    uint64_t mask = 0;
    auto fetch = [&](uint32_t (*wv)[4], int& q4) -> bool {
        while (mask == 0 && u < ue) {
            k0 = u * 64;
            qv = (int)((const int8_t*)Qs)[k0 + lane];
            mask = __ballot(qv != 0);
            u += 4;
        }
        if (mask == 0) return false;
        int kk[4];
        uint32_t q = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (mask) {
                const int idx = __builtin_amdgcn_readfirstlane(__builtin_ctzll(mask));
                mask &= mask - 1;
                kk[i] = idx;
                q |= ((uint32_t)__builtin_amdgcn_readlane(qv, idx) & 0xFFu) << (8 * i);
            } else {
                kk[i] = kk[0];                    /* a valid row; its activation byte stays 0 */
            }
        }
        q4 = (int)q;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t BL_G* row = wbase + (int64_t)(k0 + kk[i]) * ncols;
#pragma unroll
            for (int j = 0; j < CB; ++j) wv[j][i] = __builtin_nontemporal_load(row + col[j]);
        }
        return true;
    };
    auto compute = [&](const uint32_t (*wv)[4], const int q4) {
#pragma unroll
        for (int j = 0; j < CB; ++j)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                /* byte b of the four rows side by side: byte i of R = codes of (k_i, n = 16c + 4b + 0..3) */
                const uint32_t sel = 0x0C0C0400u + 0x0101u * (uint32_t)b;         /* [s1.b, s0.b, 0, 0] */
                const uint32_t lo = __builtin_amdgcn_perm(wv[j][1], wv[j][0], sel);
                const uint32_t hi = __builtin_amdgcn_perm(wv[j][3], wv[j][2], sel);
                const uint32_t R = lo | (hi << 16);
                A[j][b][0] = __builtin_amdgcn_sdot4((int)(R & 0x03030303u), q4, A[j][b][0], false);
                A[j][b][1] = __builtin_amdgcn_sdot4((int)(R & 0x0C0C0C0Cu), q4, A[j][b][1], false);
                A[j][b][2] = __builtin_amdgcn_sdot4((int)(R & 0x30303030u), q4, A[j][b][2], false);
                A[j][b][3] = __builtin_amdgcn_sdot4((int)((R >> 2) & 0x30303030u), q4, A[j][b][3], false);
            }
    };
    uint32_t wa[CB][4], wb[CB][4];
    int qa = 0, qb = 0;
    bool have = fetch(wa, qa);
    while (have) {
        const bool have2 = fetch(wb, qb);
        compute(wa, qa);
        if (!have2) break;
        have = fetch(wa, qa);
        compute(wb, qb);
    }
    /* partial sums of the four waves meet in LDS, then go to the product's int32 array */
#pragma unroll
    for (int j = 0; j < CB; ++j)
        if (ok[j]) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int n0 = 16 * (64 * j + lane) + 4 * b;
                const int v0 = A[j][b][0], v1 = A[j][b][1] >> 2, v2 = A[j][b][2] >> 4, v3 = A[j][b][3] >> 4;
                if (v0) atomicAdd(red + n0, v0);
                if (v1) atomicAdd(red + n0 + 1, v1);
                if (v2) atomicAdd(red + n0 + 2, v2);
                if (v3) atomicAdd(red + n0 + 3, v3);
            }
        }
    __syncthreads();
    for (int n = tid; n < N; n += 256) {
        const int v = red[n];
        if (v) atomicAdd((int32_t*)P.acc_ws + n, v);
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
void bl_stream_m1_km(const bl_stream_item* __restrict__ items, const int2* __restrict__ wgstart, const int q_ints,
                     const int red_ints) {
    extern __shared__ __attribute__((aligned(16))) int lds[];
    int* Qs = lds;
    int* red = lds + q_ints;
    int* misc = red + red_ints;
    const int2 s0 = wgstart[blockIdx.x], s1 = wgstart[blockIdx.x + 1];
    const int p_first = __builtin_amdgcn_readfirstlane(s0.x), u_first = __builtin_amdgcn_readfirstlane(s0.y);
    const int p_last = __builtin_amdgcn_readfirstlane(s1.x), u_last = __builtin_amdgcn_readfirstlane(s1.y);
    bool staged = false;
    for (int pi = p_first; pi <= p_last; ++pi) {
        if (pi == p_last && u_last == 0) break;
        const bl_stream_item P = items[pi];
        const int ub = pi == p_first ? u_first : 0;
        const int ue = pi == p_last ? u_last : P.units;
        if (ub >= ue) continue;
        switch (P.lp) {
            case 1: bl_km_slice<1>(P, ub, ue, Qs, misc, red, staged); break;
            case 2: bl_km_slice<2>(P, ub, ue, Qs, misc, red, staged); break;
            default: bl_km_slice<3>(P, ub, ue, Qs, misc, red, staged); break;
        }
        staged = true;
    }
}

/* Finishing kernel of the k-major form: grid (ceil(max N / 256), products). */
__global__ __launch_bounds__(256) void bl_km_finish(const bl_stream_item* __restrict__ items) {
    const bl_stream_item& P = items[blockIdx.y];
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= P.N) return;
    const int val = P.acc_ws[n] - *P.rowsum_fin;
    P.acc_ws[n] = 0;
    if (P.acc) P.acc[n] = val;
    if (P.y) {
        const float cf = *P.beta * *P.scale_fin;
        const float t = (float)val * cf;
        P.y[n] = P.residual ? P.residual[n] + t : t;
    }
}


/* ---- batched form: 2..64 tokens per table entry on the matrix cores --------------------------
 * The same persistent walk for a few tokens per product (batched decode: the packed weights are
 * still read once, Section 5.1).  Workgroups of eight waves.  The int8 activations of all m
 * tokens of the product live in LDS for the workgroup (m rows of Kp + 16 bytes: the 16 spread
 * the rows over the banks), staged once per product and workgroup, so between two products no
 * wave waits for another: a wave takes row groups of 32 weight rows round-robin and streams
 * their packed bytes global -> registers in batches of 32 rows x 512 k (4 KiB: four wave-wide
 * loads in which eight consecutive lanes fetch 128 consecutive bytes of one row, the access
 * pattern of the one-token kernel), two batches in flight while a third is multiplied.
 * The matrix core wants another lane order (lane r + 32h supplies sixteen consecutive k of row
 * r), so a landed batch takes one trip through a 4 KiB tile of LDS that belongs to the wave
 * alone (ds_write_b128 as loaded, ds_read_b128 as needed; 16-byte items XOR-swizzled against
 * the row so that both directions are free of bank conflicts; a wave's LDS operations execute
 * in order, so no barrier is involved).  Each 16-byte item is four packed words; a word is
 * opened into sixteen int8 codes by shift and mask and is the B operand of one
 * v_mfma_i32_32x32x32_i8 (two for more than 32 tokens) whose A operand is the same sixteen k of
 * token r (and 32 + r) read from the image
 * (any k order serves as long as both operands agree).  Lanes whose chunk lies behind the row's
 * end re-read its last chunk and meet sixteen zero bytes kept behind the image; tokens behind
 * m re-read token m-1 and are never stored.  Offset codes: sum_k q of the token is subtracted
 * once per output. */
#define BL_MB_THREADS 512
#define BL_MB_WAVES 8
#define BL_MB_MISC 576        /* bytes behind the image: 64 zero bytes, 64 row sums, 64 factors */
#define BL_MB_TILE 4096       /* bytes of a wave's private tile */

template <int TB, bool RES>
__device__ __forceinline__ void bl_stream_slice_mb(const bl_stream_item& P, const int ub, const int ue,
                                                   uint8_t* __restrict__ img, uint8_t* __restrict__ tiles,
                                                   const bool restage) {
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5, r8 = lane >> 3, c8 = lane & 7;
    const int N = P.N, nchunks = P.nchunks, m = P.m, rowc = P.row_chunks, c0 = P.c0;
    const int stride = nchunks * 64 + 16;                               /* image row: the entry's k part + 16 */
    const int nb = (nchunks + 7) / 8;                                   /* batches of 512 k per row */
    int32_t BL_G* const ws_g = (int32_t BL_G*)P.acc_ws;                 /* k parts of a split product meet here */
    const bl_gv4i* const wbase = (const bl_gv4i*)P.packed;
    int32_t BL_G* const acc_g = (int32_t BL_G*)P.acc;
    float BL_G* const y_g = (float BL_G*)P.y;
    const float BL_G* const res_g = (const float BL_G*)P.residual;
    uint8_t* const zero = img + m * stride;                             /* 64 zero bytes */
    int* const rs_s = (int*)(zero + 64);
    float* const cf_s = (float*)(rs_s + 64);
    bl_v4i* const tile = (bl_v4i*)(tiles + w * BL_MB_TILE);

    /* batch b of row group rg: load i covers rows 8i .. 8i+7, lane (r8, c8) chunk 8b + c8 of row 8i + r8 */
    auto issue = [&](bl_v4i* p, int rg, int b) {
        const int chunk = b * 8 + c8;
        const int cc = chunk < nchunks ? chunk : nchunks - 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int n = rg * 32 + i * 8 + r8;
            n = n < N ? n : N - 1;
            p[i] = __builtin_nontemporal_load(wbase + (int64_t)n * rowc + c0 + cc);
        }
    };
    int arow[TB];                                                        /* token l32 of tile tt (clamped) */
#pragma unroll
    for (int tt = 0; tt < TB; ++tt) arow[tt] = (tt * 32 + l32 < m ? tt * 32 + l32 : m - 1) * stride;
    const int zoff = m * stride;
    auto process = [&](const bl_v4i* p, int b, bl_v16i* C) {
        /* registers -> tile: row 8i + r8, item c8 ^ ((row / 2) % 8) */
#pragma unroll
        for (int i = 0; i < 4; ++i) tile[(i * 8 + r8) * 8 + (c8 ^ (((i * 8 + r8) >> 1) & 7))] = p[i];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bl_v4i w4 = tile[l32 * 8 + ((2 * j + h) ^ ((l32 >> 1) & 7))];
            const int chunk = b * 8 + 2 * j + h;
            const bool valid = chunk < nchunks;
            int ao[TB];
#pragma unroll
            for (int tt = 0; tt < TB; ++tt) {
                ao[tt] = valid ? arow[tt] + chunk * 64 : zoff;
                asm volatile("" : "+v"(ao[tt]));                        /* read at the point of use, not hoisted */
            }
            const int step = valid ? 16 : 0;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const uint32_t wd = (uint32_t)w4[t];
                const uint32_t l0 = wd & 0x03030303u, l1 = (wd >> 2) & 0x03030303u, l2 = (wd >> 4) & 0x03030303u,
                               l3 = (wd >> 6) & 0x03030303u;
                const bl_v4i bop = {(int)l0, (int)l1, (int)l2, (int)l3};
#pragma unroll
                for (int tt = 0; tt < TB; ++tt) {
                    const bl_v4i a = *(const bl_v4i*)(img + ao[tt] + t * step);
                    C[tt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, bop, C[tt], 0, 0, 0);
                }
            }
        }
    };
    /* lane (n = l32, h) holds, in element v of tile tt, token 32tt + (v/4)*8 + 4h + v%4 of output feature n */
    auto epilogue = [&](bl_v16i& C, int rg, int tt) {
        bl_mfma_fence();
        /* (the row length and the lane half are hidden from the compiler here: it would otherwise
         * keep the sixteen 64-bit row offsets of a lane's tokens in registers across the k loop) */
        int Nl = N, hl = h;
        asm volatile("" : "+s"(Nl));
        asm volatile("" : "+v"(hl));
        const int n = rg * 32 + l32;
        const bool nok = n < N;
        float rv[16];
        if (RES) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = tt * 32 + (v >> 2) * 8 + hl * 4 + (v & 3);
                rv[v] = (nok && t < m) ? res_g[(int64_t)t * Nl + n] : 0.0f;
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int t = tt * 32 + (v >> 2) * 8 + hl * 4 + (v & 3);
            if (nok && t < m) {
                if (ws_g) {                                             /* one k part: integer atomics, exact and order-free */
                    atomicAdd((int*)(ws_g + (int64_t)t * Nl + n), C[v]);
                    continue;
                }
                const int val = C[v] - rs_s[t];
                if (acc_g) acc_g[(int64_t)t * Nl + n] = val;
                if (y_g) {
                    const float o = (float)val * cf_s[t];
                    y_g[(int64_t)t * Nl + n] = RES ? rv[v] + o : o;
                }
            }
        }
    };

    bl_v4i pa[4], pb[4], pc[4];
    const int rg0 = ub + w;
    const bool work = rg0 < ue;
    /* issue cursor (two batches ahead of the process cursor); behind the wave's last row group it
     * stays on that row group: valid addresses, data never used */
    int irg = rg0, ib = 0;
    auto advance = [&]() {
        if (++ib == nb) {
            ib = 0;
            if (irg + BL_MB_WAVES < ue) irg += BL_MB_WAVES;
        }
    };
    if (work) {                                                          /* in flight during the staging */
        issue(pa, irg, ib);
        advance();
        issue(pb, irg, ib);
        advance();
    }
    if (restage) __syncthreads();                                       /* every wave is done with the previous image */
    {
        /* stage the m token rows (16 bytes per thread and step), the zero bytes and the token terms */
        const int upr = nchunks * 4, ldu = P.ldq / 16;
        const bl_gv4i* qg = (const bl_gv4i*)P.q + c0 * 4;
        for (int u = tid; u < m * upr; u += BL_MB_THREADS) {
            const int row = u / upr, c = u - row * upr;
            *(bl_v4i*)(img + row * stride + c * 16) = qg[row * ldu + c];
        }
        if (tid < 16) ((int*)zero)[tid] = 0;
        if (tid < 64) {
            const int t = tid < m ? tid : m - 1;
            rs_s[tid] = ((const int32_t BL_G*)P.rowsum)[t];
            cf_s[tid] = P.y ? *(const float BL_G*)P.beta * ((const float BL_G*)P.scale)[t] : 0.0f;
        }
    }
    __syncthreads();
    if (!work) return;

    int prg = rg0, pbt = 0;                                             /* process cursor */
    bl_v16i C[TB];
#pragma unroll
    for (int tt = 0; tt < TB; ++tt)
#pragma unroll
        for (int v = 0; v < 16; ++v) C[tt][v] = 0;
    /* one batch out of `buf`; true when the wave's last row group is finished */
    auto step = [&](const bl_v4i* buf) {
        process(buf, pbt, C);
        if (++pbt < nb) return false;
#pragma unroll
        for (int tt = 0; tt < TB; ++tt) {
            epilogue(C[tt], prg, tt);
#pragma unroll
            for (int v = 0; v < 16; ++v) C[tt][v] = 0;
        }
        pbt = 0;
        prg += BL_MB_WAVES;
        return prg >= ue;
    };
    while (true) {
        issue(pc, irg, ib);
        advance();
        if (step(pa)) break;
        issue(pa, irg, ib);
        advance();
        if (step(pb)) break;
        issue(pb, irg, ib);
        advance();
        if (step(pc)) break;
    }
}

/* TB = token tiles of 32 an entry may hold: 1 for tables of at most 32 tokens (fewer registers:
 * two workgroups per compute unit when the images are small), 2 beyond. */
template <int TB>
__global__ __launch_bounds__(BL_MB_THREADS)
void bl_stream_mb(const bl_stream_item* __restrict__ items, const int2* __restrict__ wgstart) {
    extern __shared__ __attribute__((aligned(16))) uint8_t img[];   /* tiles of the eight waves, then the image */
    uint8_t* const tiles = img;
    uint8_t* const image = img + BL_MB_WAVES * BL_MB_TILE;
    const int2 s0 = wgstart[blockIdx.x], s1 = wgstart[blockIdx.x + 1];
    const int p_first = __builtin_amdgcn_readfirstlane(s0.x), u_first = __builtin_amdgcn_readfirstlane(s0.y);
    const int p_last = __builtin_amdgcn_readfirstlane(s1.x), u_last = __builtin_amdgcn_readfirstlane(s1.y);
    bool staged = false;
    for (int pi = p_first; pi <= p_last; ++pi) {
        if (pi == p_last && u_last == 0) break;
        const bl_stream_item P = items[pi];
        const int ub = pi == p_first ? u_first : 0;
        const int ue = pi == p_last ? u_last : P.units;
        if (ub >= ue) continue;
        if (TB == 2 && P.m > 32) {
            if (P.residual) bl_stream_slice_mb<TB, true>(P, ub, ue, image, tiles, staged);
            else bl_stream_slice_mb<TB, false>(P, ub, ue, image, tiles, staged);
        } else {
            if (P.residual) bl_stream_slice_mb<1, true>(P, ub, ue, image, tiles, staged);
            else bl_stream_slice_mb<1, false>(P, ub, ue, image, tiles, staged);
        }
        staged = true;
    }
}

/* Finishing kernel of the batched form for products that were split along k: subtracts the
 * row sum, rescales, adds the residual, stores, and clears the partial sums for the next run.
 * grid (ceil(max M*N / 1024), split products). */
struct bl_mb_fin_item {
    int32_t* ws;              /* [M][N] partial sums */
    const int32_t* rowsum;
    const float* scale;
    const float* beta;
    const float* residual;
    int32_t* acc;
    float* y;
    int M, N;
};
__global__ __launch_bounds__(256) void bl_mb_finish(const bl_mb_fin_item* __restrict__ items) {
    const bl_mb_fin_item F = items[blockIdx.y];
    const int64_t total = (int64_t)F.M * F.N;
    const int64_t base = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    if (base >= total) return;
    const float bt = F.y ? *bl_gc<float>(F.beta) : 0.0f;
    /* four elements per thread, every load of a step issued before the first use */
    int part[4], rs[4];
    float cf[4], res[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t e = base + j * 256;
        const bool ok = e < total;
        const int t = ok ? (int)(e / F.N) : 0;
        part[j] = ok ? bl_g(F.ws)[e] : 0;
        rs[j] = bl_gc<int32_t>(F.rowsum)[t];
        cf[j] = F.y ? bl_gc<float>(F.scale)[t] : 0.0f;
        res[j] = (ok && F.residual) ? bl_gc<float>(F.residual)[e] : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t e = base + j * 256;
        if (e < total) {
            const int val = part[j] - rs[j];
            bl_g(F.ws)[e] = 0;
            if (F.acc) bl_g(F.acc)[e] = val;
            if (F.y) {
                const float o = (float)val * (bt * cf[j]);
                bl_g(F.y)[e] = F.residual ? res[j] + o : o;
            }
        }
    }
}

/* ---- host side ---------------------------------------------------------------------------- */

#define BL_STREAM_LMIN 3
#define BL_STREAM_LMAX 5
#define BL_STREAM_MAX_BLOCKS 4096
#define BL_STREAM_LDS_BYTES                                                                          \
    (layout == BL_LAYOUT_KMAJOR ? max_units * 64 + max_cols * 64 + 64                                \
                                : (max_slots + 1) * (dot ? (layout == BL_LAYOUT_TRIT5 ? bl_dot_stride<BL_FORM_TRIT5>() : bl_dot_stride<BL_FORM_BIT2>()) * 4 \
                                                        : layout == BL_LAYOUT_TRIT5 ? BL_T5_CHUNK : BL_B2_CHUNK) + 64)
static_assert(sizeof(bl_cut_pos) == sizeof(int2), "read as int2 by the kernels");
#define BL_KM_MAX_N 3072      /* k-major form: at most three dword columns of 64 lanes per weight row (48 sums per lane) */

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

/* Device buffer layout: [items][slice table][preparation items][rowsum_ws][scale_ws][q_ws][acc_ws]. */
struct bl_stream_layout {
    size_t wg_off, prep_off, rowsum_off, scale_off, q_off, acc_off, total;
};
static bl_stream_layout stream_layout(int count, size_t q_bytes, size_t acc_bytes = 0) {
    bl_stream_layout L;
    L.wg_off = align_up((size_t)count * sizeof(bl_stream_item), 256);
    L.prep_off = L.wg_off + align_up((size_t)(BL_STREAM_MAX_BLOCKS + 1) * sizeof(int2), 256);
    L.rowsum_off = L.prep_off + align_up((size_t)count * sizeof(bl_stream_prep_item), 256);
    L.scale_off = L.rowsum_off + align_up((size_t)count * 4, 256);
    L.q_off = L.scale_off + align_up((size_t)count * 4, 256);
    L.acc_off = L.q_off + align_up(q_bytes, 256);
    L.total = L.acc_off + align_up(acc_bytes, 256);
    return L;
}

static bool desc_is_fused(const bl_decode_desc& d) { return d.X || d.prod.in0; }

static bl_status check_stack_desc(const bl_decode_desc& d, int layout) {
    if (!d.packed || !d.beta) return BL_ERR_NULL;
    const bool fused = desc_is_fused(d);
    if (!fused && !d.q) return BL_ERR_NULL;
    if (!d.acc && !d.y) return BL_ERR_NULL;
    if (!fused && d.y && !d.scale) return BL_ERR_NULL;
    if (!bl_shape_ok(d.N, d.K) || d.K > 64 * 64 * BL_STREAM_LMAX || d.N > (1 << 28)) return BL_ERR_SHAPE;
    if (fused && d.K % 64 != 0) return BL_ERR_SHAPE;     /* bf16 / producer rows are read 16 elements at a time */
    if (layout == BL_LAYOUT_KMAJOR && d.N > BL_KM_MAX_N) return BL_ERR_SHAPE;
    if (layout < BL_LAYOUT_ROWMAJOR || layout > BL_LAYOUT_KMAJOR) return BL_ERR_LAYOUT;
    if (!bl_aligned(d.packed, 16) || !bl_aligned(d.X, 16) || !bl_aligned(d.q, 16) || !bl_aligned(d.q_out, 16) ||
        !bl_aligned(d.acc, 4) || !bl_aligned(d.y, 4) || !bl_aligned(d.scale, 4) || !bl_aligned(d.beta, 4) ||
        !bl_aligned(d.rowsum, 4) || !bl_aligned(d.scale_out, 4) || !bl_aligned(d.residual, 4))
        return BL_ERR_ALIGN;
    return BL_OK;
}

/* ---- batched form (2 .. BL_STACK_MAX_TOKENS tokens per product) ------------------------------ */

#define BL_MB_LDS_MAX (160 * 1024)

/* How one product is entered in the table: token groups of at most 64 (two matrix-core tiles),
 * the M tokens split evenly over the fewest groups, and k parts of whole 512-k batches so that a
 * group's rows of one part fit LDS beside each other.  A product with more than one k part
 * collects its partial sums in `ws` and is finished by bl_mb_finish. */
struct mb_split {
    int groups, per_group;    /* token groups, tokens per group (the last may hold fewer) */
    int parts, part_chunks;   /* k parts, 16-byte chunks per part (the last may hold fewer) */
};
static bool mb_split_product(int64_t M, int64_t Kp, mb_split* sp) {
    const int64_t budget = BL_MB_LDS_MAX - BL_MB_MISC - BL_MB_WAVES * BL_MB_TILE;
    const int64_t nchunks = Kp / 64;
    /* two matrix-core tiles of tokens per entry where their rows fit LDS whole (the weights are
     * then read once and nothing meets through atomics: measured at M = 64, 2560 <= K: two groups
     * of 32 tokens 267 us per 30 layers, one group of 64 in k parts 375 us); else one tile */
    sp->groups = (int)((M + 63) / 64);
    sp->per_group = (int)((M + sp->groups - 1) / sp->groups);
    if (sp->per_group > 32 && (int64_t)sp->per_group * (Kp + 16) > budget) {
        sp->groups = (int)((M + 31) / 32);
        sp->per_group = (int)((M + sp->groups - 1) / sp->groups);
    }
    int64_t parts = ((int64_t)sp->per_group * (Kp + 16) + budget - 1) / budget;
    int64_t pc = (nchunks + parts - 1) / parts;
    pc = (pc + 7) / 8 * 8;
    while (pc > 8 && (int64_t)sp->per_group * (pc * 64 + 16) > budget) pc -= 8;
    if ((int64_t)sp->per_group * (pc * 64 + 16) > budget) return false;
    sp->part_chunks = (int)pc;
    sp->parts = (int)((nchunks + pc - 1) / pc);
    return true;
}

/* Device buffer of the batched form: [entries][slice table][finishing items][partial sums]. */
struct mb_layout_t {
    size_t wg_off, fin_off, ws_off, total;
};
static mb_layout_t mb_layout(int64_t entries, int count, size_t ws_bytes) {
    mb_layout_t L;
    L.wg_off = align_up((size_t)entries * sizeof(bl_stream_item), 256);
    L.fin_off = L.wg_off + align_up((size_t)(BL_STREAM_MAX_BLOCKS + 1) * sizeof(int2), 256);
    L.ws_off = L.fin_off + align_up((size_t)count * sizeof(bl_mb_fin_item), 256);
    L.total = L.ws_off + align_up(ws_bytes, 256);
    return L;
}

static bl_status check_batched_desc(const bl_decode_desc& d, int layout) {
    if (!d.packed || !d.beta || !d.q || !d.rowsum) return BL_ERR_NULL;
    if (d.X || d.prod.in0) return BL_ERR_VALUE;            /* int8 inputs only: quantise with bl_quant_act_int8 */
    if (!d.acc && !d.y) return BL_ERR_NULL;
    if (d.y && !d.scale) return BL_ERR_NULL;
    if (!bl_shape_ok(d.N, d.K) || d.N > (1 << 24)) return BL_ERR_SHAPE;
    if (layout != BL_LAYOUT_K16) return BL_ERR_LAYOUT;
    if (!bl_aligned(d.packed, 16) || !bl_aligned(d.q, 16) || !bl_aligned(d.acc, 4) || !bl_aligned(d.y, 4) ||
        !bl_aligned(d.scale, 4) || !bl_aligned(d.beta, 4) || !bl_aligned(d.rowsum, 4) || !bl_aligned(d.residual, 4))
        return BL_ERR_ALIGN;
    return BL_OK;
}

static bool mb_sizes(const bl_decode_desc* descs, int count, int64_t M, int64_t* entries, size_t* ws_bytes) {
    *entries = 0;
    *ws_bytes = 0;
    for (int i = 0; i < count; ++i) {
        if (!bl_shape_ok(descs[i].N, descs[i].K) || descs[i].N > (1 << 24)) return false;
        mb_split sp;
        if (!mb_split_product(M, bl_kpad(descs[i].K), &sp)) return false;
        *entries += (int64_t)sp.groups * sp.parts;
        if (sp.parts > 1) *ws_bytes += align_up((size_t)(M * descs[i].N * 4), 256);
    }
    return *entries <= 64 * BL_STACK_MAX_COUNT;
}

static bool mb_tile_route(const bl_decode_desc* descs, int count, int64_t M);
static size_t tile_route_total(const bl_decode_desc* descs, int count);

extern "C" size_t bl_stack_table_bytes_batched(const bl_decode_desc* descs, int count, int64_t M) {
    if (!descs || count < 1 || count > BL_STACK_MAX_COUNT || M < 2 || M > BL_STACK_MAX_TOKENS) return 0;
    int64_t entries = 0;
    size_t ws_bytes = 0;
    if (!mb_sizes(descs, count, M, &entries, &ws_bytes)) return 0;
    size_t total = mb_layout(entries, count, ws_bytes).total;
    if (mb_tile_route(descs, count, M)) {
        const size_t tt = tile_route_total(descs, count);
        if (tt > total) total = tt;
    }
    return total;
}

/* More than 32 tokens per product: the token rows of most products no longer fit LDS whole and go in two groups, which read the
 * weights twice; the work is a dense contraction, and the table is walked by the prefill tile kernel instead (tiles of 64 x 256,
 * both operands streamed through LDS per k step, weights read once).  Needs rows padded to 128; up to 48 tokens where it pays
 * (bl_table_in_tiles).  At 32 tokens, one group, it is the form with the tokens in LDS: thirty layers of 2560 / 6912 150 us, tiles 164,
 * three 23 / 34 (though twenty of 1024 / 2816 take 27.7 there and 25.2 in tiles, twelve of 4096 / 11008 186 and 158). */
#define BL_MB_TILE_ROUTE_MIN 33
static bool mb_tile_route(const bl_decode_desc* descs, int count, int64_t M) {
    if (M < BL_MB_TILE_ROUTE_MIN) return false;
    int64_t tiles = 0, entries = 0, steps = 0, chain = 0;
    for (int i = 0; i < count; ++i) {
        const int64_t Kp = bl_kpad(descs[i].K), blocks = (descs[i].N + BL_TILE_ROWS - 1) / BL_TILE_ROWS;
        if (Kp % 128 != 0) return false;
        tiles += (descs[i].N + 127) / 128;
        entries += blocks;
        steps += blocks * (Kp / 128);
        chain = std::max(chain, Kp / 128);
    }
    if (M <= 48 && !bl_table_in_tiles(entries, steps, chain)) return false;
    return tiles <= ((int64_t)1 << 22);       /* beyond ~4 M tiles (a 16 MB tile list) the table stays on bl_stream_mb */
}

/* Device buffer of the tile route: [products][first list position of each workgroup][tile list]. */
struct tile_layout_t {
    size_t wg_off, list_off, total;
};
static tile_layout_t tile_layout(int count, int64_t tiles) {
    tile_layout_t L;
    L.wg_off = align_up((size_t)count * sizeof(bl_tile_item), 256);
    L.list_off = L.wg_off + align_up((size_t)(BL_STREAM_MAX_BLOCKS + 1) * sizeof(int), 256);
    L.total = L.list_off + align_up((size_t)tiles * sizeof(int), 256);
    return L;
}
static int64_t tile_route_tiles(const bl_decode_desc* descs, int count) {
    int64_t tiles = 0;
    for (int i = 0; i < count; ++i) tiles += (descs[i].N + 127) / 128;
    return tiles;
}

static size_t tile_route_total(const bl_decode_desc* descs, int count) {
    return tile_layout(count, tile_route_tiles(descs, count)).total;
}

static bl_status stack_build_tiles(const bl_decode_desc* descs, int count, int layout, int M, void* table,
                                   bl_stack_plan* plan, hipStream_t st) {
    const int resident = bl_gemm_table_blocks();
    if (resident < 1) return BL_ERR_HIP;
    const int64_t tiles = tile_route_tiles(descs, count);
    const tile_layout_t L = tile_layout(count, tiles);
    int64_t entries = 0;                                  /* of the list: blocks of BL_TILE_ROWS rows, no more than `tiles` */
    for (int i = 0; i < count; ++i) entries += (descs[i].N + BL_TILE_ROWS - 1) / BL_TILE_ROWS;
    int blocks = (int)(entries < resident ? entries : resident);
    if (blocks > BL_STREAM_MAX_BLOCKS) blocks = BL_STREAM_MAX_BLOCKS;
    std::vector<uint8_t> blob(L.total, 0);
    bl_tile_item* items = (bl_tile_item*)blob.data();
    int* wg_start = (int*)(blob.data() + L.wg_off);
    int* tile_list = (int*)(blob.data() + L.list_off);
    int64_t packed_bytes = 0;
    /* (cost, first tile, tiles) of each product; cost of a tile = its k steps + a fixed part for
     * set-up and stores */
    std::vector<std::pair<int, int>> by_cost;             /* (-cost, product) */
    for (int i = 0; i < count; ++i) {
        const bl_decode_desc& d = descs[i];
        const int64_t Kp = bl_kpad(d.K);
        items[i] = bl_tile_item{d.packed, d.q, d.rowsum, d.beta, d.y ? d.scale : nullptr, d.residual, d.acc, d.y,
                                (int)d.N, (int)Kp};
        packed_bytes += d.N * (Kp / 4);
        by_cost.push_back({-(int)(Kp / 128 + 4), i});
    }
    /* longest tiles first, each to the workgroup with the least work so far */
    std::sort(by_cost.begin(), by_cost.end());
    std::vector<std::vector<int>> lists((size_t)blocks);
    std::priority_queue<std::pair<int64_t, int>, std::vector<std::pair<int64_t, int>>, std::greater<std::pair<int64_t, int>>> load;
    for (int b = 0; b < blocks; ++b) load.push({0, b});
    for (const auto& pc : by_cost) {
        const int i = pc.second, n_tiles = (int)((descs[i].N + BL_TILE_ROWS - 1) / BL_TILE_ROWS);
        for (int j = 0; j < n_tiles; ++j) {
            auto top = load.top();
            load.pop();
            lists[(size_t)top.second].push_back(i << BL_TILE_BITS | j);
            top.first += -pc.first;
            load.push(top);
        }
    }
    int pos = 0;
    for (int b = 0; b < blocks; ++b) {
        wg_start[b] = pos;
        for (int v : lists[(size_t)b]) tile_list[pos++] = v;
    }
    wg_start[blocks] = pos;
    if (hipMemcpyAsync(table, blob.data(), blob.size(), hipMemcpyHostToDevice, st) != hipSuccess) return BL_ERR_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) return BL_ERR_HIP;   /* the host copy of the table dies here */
    memset(plan, 0, sizeof(*plan));
    plan->count = count;
    plan->blocks = blocks;
    plan->layout = layout;
    plan->wg_offset = (int64_t)L.wg_off;
    plan->prep_offset = (int64_t)L.list_off;
    plan->packed_bytes = packed_bytes;
    plan->table_bytes = (int64_t)bl_stack_table_bytes_batched(descs, count, M);
    plan->tokens = M;
    plan->entries = count;
    plan->red_ints = (int32_t)tiles;                      /* blocks of 128 rows of the whole table: room for the list */
    plan->norm = 3;                                       /* the tile route */
    return BL_OK;
}

static std::atomic<bool> g_mb_attr_set;

static bl_status stack_build_batched(const bl_decode_desc* descs, int count, int layout, int M, void* table,
                                     bl_stack_plan* plan, hipStream_t st) {
    for (int i = 0; i < count; ++i) {
        const bl_status rc = check_batched_desc(descs[i], layout);
        if (rc != BL_OK) return rc;
    }
    int64_t entries64 = 0;
    size_t ws_bytes = 0;
    if (!mb_sizes(descs, count, M, &entries64, &ws_bytes)) return BL_ERR_SHAPE;
    if (mb_tile_route(descs, count, M)) return stack_build_tiles(descs, count, layout, M, table, plan, st);
    const int entries = (int)entries64;
    const mb_layout_t L = mb_layout(entries, count, ws_bytes);
    uint8_t* const dev_base = (uint8_t*)table;
    std::vector<bl_stream_item> items;
    std::vector<bl_mb_fin_item> fins;                    /* one per product that is split along k */
    std::vector<int> units_v;
    std::vector<int64_t> ucost_v, ecost_v;
    int64_t packed_bytes = 0, total_units = 0, max_elems = 0;
    int lds = 0, split_products = 0;
    size_t ws_used = 0;
    for (int i = 0; i < count; ++i) {
        const bl_decode_desc& d = descs[i];
        const int64_t Kp = bl_kpad(d.K);
        mb_split sp;
        mb_split_product(M, Kp, &sp);
        packed_bytes += d.N * (Kp / 4);
        int32_t* ws = nullptr;
        if (sp.parts > 1) {
            ws = (int32_t*)(dev_base + L.ws_off + ws_used);
            ws_used += align_up((size_t)((int64_t)M * d.N * 4), 256);
            ++split_products;
            if ((int64_t)M * d.N > max_elems) max_elems = (int64_t)M * d.N;
        }
        if (ws) fins.push_back(bl_mb_fin_item{ws, d.rowsum, d.scale, d.beta, d.residual, d.acc, d.y, M, (int)d.N});
        for (int g = 0; g < sp.groups; ++g) {
            const int m0 = g * sp.per_group, m = M - m0 < sp.per_group ? M - m0 : sp.per_group;
            for (int pt = 0; pt < sp.parts; ++pt) {
                const int c0 = pt * sp.part_chunks;
                const int nch = (int)(Kp / 64) - c0 < sp.part_chunks ? (int)(Kp / 64) - c0 : sp.part_chunks;
                bl_stream_item it;
                memset(&it, 0, sizeof(it));
                it.packed = (const bl_v4i*)d.packed;
                it.beta = d.beta;
                it.q = d.q + (int64_t)m0 * Kp;
                it.scale = d.scale ? d.scale + m0 : nullptr;
                it.rowsum = d.rowsum + m0;
                it.residual = d.residual ? d.residual + (int64_t)m0 * d.N : nullptr;
                it.acc = d.acc ? d.acc + (int64_t)m0 * d.N : nullptr;
                it.y = d.y ? d.y + (int64_t)m0 * d.N : nullptr;
                it.acc_ws = ws ? ws + (int64_t)m0 * d.N : nullptr;
                it.N = (int)d.N;
                it.nchunks = nch;
                it.row_chunks = (int)(Kp / 64);
                it.c0 = c0;
                it.ldq = (int)Kp;
                it.qgroups = (int)(Kp / 16);
                it.layout = layout;
                it.m = m;
                it.units = (int)((d.N + 31) / 32);
                const int need = (int)(m * (nch * 64 + 16) + BL_MB_MISC + BL_MB_WAVES * BL_MB_TILE);
                if (need > lds) lds = need;
                items.push_back(it);
                units_v.push_back(it.units);
                ucost_v.push_back((int64_t)32 * nch * 16);
                ecost_v.push_back((int64_t)2 * m * nch * 64);   /* staging the token rows */
                total_units += it.units;
            }
        }
    }
    lds = (lds + 255) / 256 * 256;
    bool two_tiles = false;
    for (int i = 0; i < count; ++i) {
        mb_split sp;
        mb_split_product(M, bl_kpad(descs[i].K), &sp);
        two_tiles = two_tiles || sp.per_group > 32;
    }
    const void* kern = two_tiles ? (const void*)bl_stream_mb<2> : (const void*)bl_stream_mb<1>;
    if (!g_mb_attr_set.load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute((const void*)bl_stream_mb<1>, hipFuncAttributeMaxDynamicSharedMemorySize, BL_MB_LDS_MAX) !=
                hipSuccess ||
            hipFuncSetAttribute((const void*)bl_stream_mb<2>, hipFuncAttributeMaxDynamicSharedMemorySize, BL_MB_LDS_MAX) !=
                hipSuccess)
            return BL_ERR_HIP;
        g_mb_attr_set.store(true, std::memory_order_release);
    }
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, BL_MB_THREADS, (size_t)lds) !=
            hipSuccess ||
        cus < 1 || per_cu < 1)
        return BL_ERR_HIP;
    int64_t blocks64 = (int64_t)cus * per_cu;
    if (blocks64 > (total_units + BL_MB_WAVES - 1) / BL_MB_WAVES) blocks64 = (total_units + BL_MB_WAVES - 1) / BL_MB_WAVES;
    if (blocks64 > BL_STREAM_MAX_BLOCKS) blocks64 = BL_STREAM_MAX_BLOCKS;
    if (blocks64 < 1) blocks64 = 1;
    const int blocks = (int)blocks64;
    const std::vector<bl_cut_pos> wg = bl_cut_slices(units_v, ucost_v, ecost_v, blocks, BL_MB_WAVES);
    std::vector<uint8_t> blob(L.ws_off, 0);
    memcpy(blob.data(), items.data(), items.size() * sizeof(bl_stream_item));
    memcpy(blob.data() + L.wg_off, wg.data(), wg.size() * sizeof(bl_cut_pos));
    if (!fins.empty()) memcpy(blob.data() + L.fin_off, fins.data(), fins.size() * sizeof(bl_mb_fin_item));
    /* the partial sums start at zero; every run leaves them at zero again */
    if (ws_bytes && hipMemsetAsync(dev_base + L.ws_off, 0, ws_bytes, st) != hipSuccess) return BL_ERR_HIP;
    if (hipMemcpyAsync(table, blob.data(), blob.size(), hipMemcpyHostToDevice, st) != hipSuccess) return BL_ERR_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) return BL_ERR_HIP;   /* the host copy of the table dies here */
    memset(plan, 0, sizeof(*plan));
    plan->count = count;
    plan->blocks = blocks;
    plan->lds_bytes = lds;
    plan->layout = layout;
    plan->wg_offset = (int64_t)L.wg_off;
    plan->prep_offset = (int64_t)L.fin_off;
    plan->packed_bytes = packed_bytes;
    plan->table_bytes = (int64_t)L.total;
    plan->tokens = M;
    plan->entries = entries;
    plan->prep_count = split_products;                  /* > 0: the finishing kernel runs */
    plan->red_ints = (int32_t)((max_elems + 1023) / 1024);   /* its grid in x */
    plan->norm = two_tiles ? 2 : 1;                       /* token tiles of the kernel variant */
    return BL_OK;
}

extern "C" size_t bl_stack_table_bytes(const bl_decode_desc* descs, int count) {
    if (!descs || count < 1 || count > BL_STACK_MAX_COUNT) return 0;
    size_t q_bytes = 0, acc_bytes = 0;
    for (int i = 0; i < count; ++i) {
        if (descs[i].K < 1 || descs[i].K > 64 * 64 * BL_STREAM_LMAX || descs[i].N < 1 || descs[i].N > (1 << 28)) return 0;
        if (desc_is_fused(descs[i])) q_bytes += align_up((size_t)descs[i].K, 256);
        acc_bytes += align_up((size_t)descs[i].N * 4, 256);     /* partial sums of the k-major form */
    }
    return stream_layout(count, q_bytes, acc_bytes).total;
}

/* 16-byte chunks of a packed weight row (not the k-major form). */
static int64_t row_chunks(int64_t K, int layout) {
    return layout == BL_LAYOUT_TRIT5 ? bl_kpad5(K) / 80 : bl_kpad(K) / 64;
}
/* Rows that are no multiple of 64 bytes: read from the starts of their lines too, by row groups of two classes of rows
 * (bl_stream_index.h), where they are longer than 2560 weights, in the 2-bit form.  A load whose eight pieces each lie across
 * two lines asks for sixteen: 250 MB of K = 3200 53.6 -> 46.8 us, 8768 57.8 -> 48.8, 19904 64 -> 57; up to 2560 the loop does not wait for
 * it (K = 2240 48.6 / 47.6, 1472 48.8 / 50.0; five per byte K = 4000 64 / 64, and 3440 62 / 71 for the extra load of some rows).
 * A table takes the kernel for it where such products are an eighth of its bytes (8 layers of 4096 / 9408, where they are 24 %, 68.0
 * us without it, 55.9 with it; the other products lose up to 1 %) and 6 MiB: 10240 x 3200 5.16 / 4.93, 6144 x 3200 4.67 / 4.90, 1024 x 3200
 * 4.54 / 4.76 (more zeros to stage). */
static bool wants_classes(int64_t K, int layout) {
    const int64_t chunks = row_chunks(K, layout);
    return (layout == BL_LAYOUT_ROWMAJOR || layout == BL_LAYOUT_K16) && chunks > 40 && chunks % 4 != 0;
}
static bool table_classes(const bl_decode_desc* descs, int count, int layout) {
    int64_t all = 0, such = 0;
    for (int i = 0; i < count; ++i) {
        const int64_t bytes = descs[i].N * row_chunks(descs[i].K, layout) * 16;
        all += bytes;
        if (wants_classes(descs[i].K, layout)) such += bytes;
    }
    return such >= (int64_t)6 << 20 && such >= all / 8;
}
/* How the rows of a product are read: lq, mod and lead of its bl_stream_item, and the wave-wide loads of a row group. */
struct row_plan {
    int lq, mod, lead, loads;
};
static row_plan plan_rows(int64_t K, int layout, bool classes) {
    const int chunks = (int)row_chunks(K, layout);
    row_plan r;
    r.lq = classes && wants_classes(K, layout) ? bl_row_classes(chunks) : 0;
    r.mod = r.lq || chunks % 4 == 0 ? chunks % 8 : 0;
    r.lead = bl_row_lead(r.mod);
    r.loads = (chunks + r.lead + 7) / 8;
    return r;
}
/* Lanes of a row in bl_stream_dot (log2): at most BL_STREAM_LMAX loads of a lane. */
static int dot_lanes(int64_t chunks) {
    int lgG = 3;
    while (((chunks + (1 << lgG) - 1) >> lgG) > BL_STREAM_LMAX) ++lgG;   /* (K is bounded: at most 6) */
    return lgG;
}
/* Tables for bl_stream_dot, by the row groups of eight of the whole table and the loads of one.  With few of them a workgroup stages
 * its row and multiplies one or two row groups, and a long row is one wave's serial chain on the matrix cores.  Measured over
 * 2150 tables (one product of 64 .. 50000 rows x 64 .. 20480, 1 .. 70 layers, mixed sizes), dot / matrix cores:
 * 2-bit: rows of 6 loads (K > 2560) and more under 600 row groups .53 - .98 (1024 x 14336 5.6 / 9.2 us, 256 x 4096 3.9 / 4.5), 600 - 900
 * 1.05 - 1.1; of 30 loads up to 1400 .89 - 1.03; shorter rows 1.02 - 1.15.
 * Five per byte, tables of one width: rows of 3 - 5 loads under 3500 row groups .92 - 1.0, above 1.0 - 1.2; of 6 and more, under 600 or 75 per load
 * .43 - .98 (2048 x 20480 6.5 / 13.1), above 1.05 - 1.2; shorter rows under 200 .95 - 1.01, larger tables up to 2.3.  Of several widths under 5000
 * .81 - 1.03 (one layer of 2560 / 6912 9.7 / 10.3, of 4096 / 11008 15.5 / 17.9), above 1.0 - 1.35.  K > 19200: an image of which four
 * fit no compute unit (32768 x 20480 34 / 40, 32768 x 19840 33 / 38, twenty of 2560 x 19840 55 / 61). */
static bool table_dot(const bl_decode_desc* descs, int count, int layout) {
    int64_t groups = 0, loads = 0, longest = 0;
    for (int i = 0; i < count; ++i) {
        const int64_t g = (descs[i].N + 7) / 8, l = plan_rows(descs[i].K, layout, false).loads;
        groups += g;
        loads += g * l;
        longest = std::max(longest, l);
    }
    if (layout != BL_LAYOUT_TRIT5) return loads >= 6 * groups && (groups < 600 || (loads >= 30 * groups && groups < 1400));
    if (longest > 30) return true;
    if (loads < 3 * groups) return groups < 200;
    if (2 * longest * groups >= 3 * loads) return groups < 5000;
    return loads < 6 * groups ? groups < 3500 : groups < 600 || groups * groups < 75 * loads;
}
/* Wave-wide loads of a part (3, 4 or 5) for a table of one-token products: the least cost over the table,
 * in quarters of a load that is multiplied; an idle slot of a row's last part is loaded (a cache hit) but not
 * multiplied, and a part costs about half a load besides. */
static int part_loads(const bl_decode_desc* descs, int count, int layout, bool classes) {
    int best = BL_STREAM_LMAX;
    int64_t least = INT64_MAX;
    for (int lp = BL_STREAM_LMAX; lp >= BL_STREAM_LMIN; --lp) {
        int64_t cost = 0;
        for (int i = 0; i < count; ++i) {
            const int64_t loads = plan_rows(descs[i].K, layout, classes).loads, parts = (loads + lp - 1) / lp;
            cost += (descs[i].N + 7) / 8 * (3 * loads + parts * lp + 2 * parts);
        }
        if (cost < least) {
            least = cost;
            best = lp;
        }
    }
    return best;
}
/* The kernel of a table: `form` = 0 bl_stream_dot; otherwise loads of a part, + BL_STREAM_CLASSES where row groups of classes occur. */
#define BL_STREAM_CLASSES 8
template <int FORM, bool CLASSES>
static const void* stream_kernel_lp(int lp) {
    return lp == 5 ? (const void*)bl_stream_m1<FORM, 5, CLASSES>
         : lp == 4 ? (const void*)bl_stream_m1<FORM, 4, CLASSES> : (const void*)bl_stream_m1<FORM, 3, CLASSES>;
}
static const void* stream_kernel(int layout, int form) {
    if (layout == BL_LAYOUT_KMAJOR) return (const void*)bl_stream_m1_km;
    if (form == 0) return layout == BL_LAYOUT_TRIT5 ? (const void*)bl_stream_dot<BL_FORM_TRIT5> : (const void*)bl_stream_dot<BL_FORM_BIT2>;
    if (layout == BL_LAYOUT_TRIT5) return stream_kernel_lp<BL_FORM_TRIT5, false>(form);
    return form & BL_STREAM_CLASSES ? stream_kernel_lp<BL_FORM_BIT2, true>(form & ~BL_STREAM_CLASSES) : stream_kernel_lp<BL_FORM_BIT2, false>(form);
}

extern "C" bl_status bl_stack_build(const bl_decode_desc* descs, int count, int layout, int64_t M, void* table,
                                    bl_stack_plan* plan, bl_stream s) {
    if (!descs || !table || !plan) return BL_ERR_NULL;
    if (count < 1 || count > BL_STACK_MAX_COUNT || M < 1 || M > BL_STACK_MAX_TOKENS) return BL_ERR_SHAPE;
    if (!bl_aligned(table, 256)) return BL_ERR_ALIGN;
    if (M > 1) return stack_build_batched(descs, count, layout, (int)M, table, plan, (hipStream_t)s);
    size_t q_bytes = 0, acc_bytes = 0;
    for (int i = 0; i < count; ++i) {
        const bl_status st = check_stack_desc(descs[i], layout);
        if (st != BL_OK) return st;
        if (desc_is_fused(descs[i])) q_bytes += align_up((size_t)descs[i].K, 256);
        acc_bytes += align_up((size_t)descs[i].N * 4, 256);
    }
    const bl_stream_layout L = stream_layout(count, q_bytes, acc_bytes);
    uint8_t* const dev_base = (uint8_t*)table;
    const bool dot = layout != BL_LAYOUT_KMAJOR && table_dot(descs, count, layout);
    const bool classes = layout != BL_LAYOUT_KMAJOR && !dot && table_classes(descs, count, layout);
    const int lp = layout == BL_LAYOUT_KMAJOR || dot ? 0 : part_loads(descs, count, layout, classes);
    std::vector<bl_stream_item> items((size_t)count);
    std::vector<bl_stream_prep_item> preps;
    int inline_count = 0, max_slots = 0, max_units = 0, max_cols = 0;
    size_t acc_used = 0;
    std::vector<int64_t> unit_bytes((size_t)count);
    bool any_norm = false;
    int64_t total = 0, packed_bytes = 0, total_units = 0;
    size_t q_used = 0;
    for (int i = 0; i < count; ++i) {
        const bl_decode_desc& d = descs[i];
        const bool fused = desc_is_fused(d);
        const int64_t Kp = bl_kpad(d.K);                 /* row length of the packed weights and of q */
        bl_stream_item it;
        memset(&it, 0, sizeof(it));
        it.packed = (const bl_v4i*)d.packed;
        it.beta = d.beta;
        it.residual = d.residual;
        it.acc = d.acc;
        it.y = d.y;
        it.N = (int)d.N;
        /* 16-byte loads per weight row: 64 weights each, or 80 in the five-per-byte form */
        const int64_t row_bytes = (layout == BL_LAYOUT_KMAJOR ? (d.N + 63) / 64 : row_chunks(d.K, layout)) * 16;
        it.nchunks = (int)(row_bytes / 16);
        it.qgroups = (int)(Kp / 16);
        it.layout = layout;
        int R = 8;                                           /* weight rows of a unit */
        if (dot) {
            it.lgG = dot_lanes(it.nchunks);
            it.lp = (it.nchunks + (1 << it.lgG) - 1) >> it.lgG;
            R = 64 >> it.lgG;
            it.units = (it.N + R - 1) / R;
            if (it.nchunks > max_slots) max_slots = it.nchunks;
        } else if (layout != BL_LAYOUT_KMAJOR) {
            const row_plan rp = plan_rows(d.K, layout, classes);
            it.lq = rp.lq;
            it.mod = rp.mod;
            it.lead = rp.lead;
            it.parts = (rp.loads + lp - 1) / lp;
            it.units = bl_groups(it.N, it.lq);
            if (it.parts * lp * 8 + it.lead > max_slots) max_slots = it.parts * lp * 8 + it.lead;
        }
        if (layout == BL_LAYOUT_KMAJOR) {
            /* one row per k: dword columns of 16 output features; a unit is 64 consecutive k */
            const int ncols = (int)((d.N + 63) / 64 * 4);
            it.nchunks = ncols;
            it.lp = (ncols + 63) / 64;
            it.units = (int)(Kp / 64);
            it.acc_ws = (int32_t*)(dev_base + L.acc_off + acc_used);
            acc_used += align_up((size_t)d.N * 4, 256);
            if (it.units > max_units) max_units = it.units;
            if (ncols > max_cols) max_cols = ncols;
            R = 64;                                          /* weight rows of a unit */
        }
        if (fused && d.prod.in0 == nullptr) {
            /* a plain bf16 row: quantised inside the stream launch by each workgroup that meets it */
            it.xbf16 = d.X;
            it.q_out = d.q_out;
            it.scale_out = d.scale_out;
            it.fixed_scale = d.fixed_scale;
            it.rowsum_pub = (int32_t*)(dev_base + L.rowsum_off) + i;
            it.scale_pub = (float*)(dev_base + L.scale_off) + i;
            if (layout == BL_LAYOUT_KMAJOR) {                /* read back by the finishing kernel */
                it.rowsum = it.rowsum_pub;
                it.scale = it.scale_pub;
            }
            ++inline_count;
        } else if (fused || !d.rowsum) {
            bl_stream_prep_item pp;
            memset(&pp, 0, sizeof(pp));
            pp.K = (int)Kp;
            pp.rowsum_ws = (int32_t*)(dev_base + L.rowsum_off) + i;
            it.rowsum = pp.rowsum_ws;
            if (fused) {
                pp.fused = 1;
                if (!bl_make_prod(d.prod, d.X, d.K, &pp.prod)) return BL_ERR_VALUE;
                any_norm = any_norm || pp.prod.norm;
                pp.q_ws = (int8_t*)(dev_base + L.q_off + q_used);
                q_used += align_up((size_t)d.K, 256);
                pp.scale_ws = (float*)(dev_base + L.scale_off) + i;
                pp.q_out = d.q_out;
                pp.scale_out = d.scale_out;
                pp.fixed_scale = d.fixed_scale;
                it.q = pp.q_ws;
                it.scale = pp.scale_ws;
            } else {
                pp.q_in = d.q;
                it.q = d.q;
                it.scale = d.scale;
            }
            preps.push_back(pp);
        } else {
            it.q = d.q;
            it.scale = d.scale;
            it.rowsum = d.rowsum;
        }
        it.rowsum_fin = it.rowsum;
        it.scale_fin = it.scale ? it.scale : it.beta;        /* unused without y; a valid address */
        unit_bytes[(size_t)i] = (int64_t)R * row_bytes;
        total += (int64_t)it.units * unit_bytes[(size_t)i];
        total_units += it.units;
        packed_bytes += (layout == BL_LAYOUT_KMAJOR ? d.K : d.N) * row_bytes;
        items[(size_t)i] = it;
    }
    /* persistent grid: the workgroups that are resident at once, but no more than one per four
     * row groups' worth of work (a workgroup has four waves) */
    const int form = classes ? lp | BL_STREAM_CLASSES : lp;
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu, stream_kernel(layout, form), 256, (size_t)BL_STREAM_LDS_BYTES) != hipSuccess ||
        cus < 1 || per_cu < 1)
        return BL_ERR_HIP;
    /* (four workgroups per compute unit also where a fifth would fit: 72 products of 13824 x 2048 84 us against 88) */
    if (layout != BL_LAYOUT_KMAJOR && !dot && per_cu > 4) per_cu = 4;
    int64_t blocks64 = (int64_t)cus * per_cu;
    if (blocks64 > (total_units + 3) / 4) blocks64 = (total_units + 3) / 4;
    if (blocks64 > BL_STREAM_MAX_BLOCKS) blocks64 = BL_STREAM_MAX_BLOCKS;
    if (blocks64 < 1) blocks64 = 1;
    const int blocks = (int)blocks64;

    /* Slice boundaries: a workgroup's time is its bytes, plus a fixed cost each time it enters a
     * product (activation row, pipeline refill; larger when it quantises the row itself), expressed
     * in bytes at a workgroup's share of the stream rate.  A row group of short rows takes a wave about as long as 2 KiB
     * (0.65 us, a load's latency over two in flight): with their bytes alone one workgroup was given thousands of them (twelve products of
     * 64 .. 11776 columns, 45 MB: 43.1 us, 12.3 like this; 1024 and 3072 instead of 2048: 14.7 and 11.3, but tables of 640 - 1024 columns
     * 0 - 10 % and up to 20 % slower with 3072). */
    std::vector<int> units_v((size_t)count);
    std::vector<int64_t> ucost_v((size_t)count), ecost_v((size_t)count);
    for (int i = 0; i < count; ++i) {
        units_v[(size_t)i] = items[(size_t)i].units;
        ucost_v[(size_t)i] = layout == BL_LAYOUT_KMAJOR ? unit_bytes[(size_t)i] : std::max<int64_t>(unit_bytes[(size_t)i], 2048);
        if (dot && items[(size_t)i].lp != 5) ucost_v[(size_t)i] = ucost_v[(size_t)i] * 26 / 25;   /* (four slots of a lane stream 4 % slower than five) */
        ecost_v[(size_t)i] = items[(size_t)i].xbf16 ? (int64_t)36 << 10 : (int64_t)12 << 10;
    }
    const std::vector<bl_cut_pos> wg = bl_cut_slices(units_v, ucost_v, ecost_v, blocks, 4);
    std::vector<uint8_t> blob(L.rowsum_off, 0);
    memcpy(blob.data(), items.data(), items.size() * sizeof(bl_stream_item));
    memcpy(blob.data() + L.wg_off, wg.data(), wg.size() * sizeof(bl_cut_pos));
    if (!preps.empty()) memcpy(blob.data() + L.prep_off, preps.data(), preps.size() * sizeof(bl_stream_prep_item));
    hipStream_t st = (hipStream_t)s;
    /* the k-major form's partial sums start at zero; every run leaves them at zero again */
    if (layout == BL_LAYOUT_KMAJOR && hipMemsetAsync(dev_base + L.acc_off, 0, acc_bytes, st) != hipSuccess)
        return BL_ERR_HIP;
    if (hipMemcpyAsync(table, blob.data(), blob.size(), hipMemcpyHostToDevice, st) != hipSuccess) return BL_ERR_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) return BL_ERR_HIP;   /* the host copy of the table dies here */

    memset(plan, 0, sizeof(*plan));
    plan->count = count;
    plan->blocks = blocks;
    plan->prep_count = (int32_t)preps.size();
    plan->inline_count = inline_count;
    plan->norm = any_norm ? 1 : 0;
    plan->lds_bytes = BL_STREAM_LDS_BYTES;
    plan->layout = layout;
    plan->red_ints = layout == BL_LAYOUT_KMAJOR ? max_cols * 16 : form;
    plan->wg_offset = (int64_t)L.wg_off;
    plan->prep_offset = (int64_t)L.prep_off;
    plan->packed_bytes = packed_bytes;
    plan->table_bytes = (int64_t)L.total;
    plan->tokens = 1;
    plan->entries = count;
    return BL_OK;
}

static bool stream_form_ok(int layout, int form) {
    const int lp = form & ~BL_STREAM_CLASSES;
    return form == 0 || (lp >= BL_STREAM_LMIN && lp <= BL_STREAM_LMAX && (lp == form || layout != BL_LAYOUT_TRIT5));
}

extern "C" bl_status bl_stack_run(void* table, const bl_stack_plan* plan, bl_stream s) {
    if (!table || !plan) return BL_ERR_NULL;
    if (plan->tokens > 1 && plan->norm == 3) {               /* the tile route of the batched form */
        if (plan->tokens < BL_MB_TILE_ROUTE_MIN || plan->tokens > BL_STACK_MAX_TOKENS || plan->count < 1 ||
            plan->count > BL_STACK_MAX_COUNT || plan->entries != plan->count || plan->red_ints < plan->count ||
            plan->blocks < 1 || plan->blocks > plan->red_ints || plan->blocks > BL_STREAM_MAX_BLOCKS ||
            plan->layout != BL_LAYOUT_K16 || plan->prep_count != 0)
            return BL_ERR_VALUE;
        const tile_layout_t Lt = tile_layout(plan->count, plan->red_ints);
        if (plan->wg_offset != (int64_t)Lt.wg_off || plan->prep_offset != (int64_t)Lt.list_off) return BL_ERR_VALUE;
        if (!bl_aligned(table, 256)) return BL_ERR_ALIGN;
        const uint8_t* tb = (const uint8_t*)table;
        return bl_gemm_table_launch((const bl_tile_item*)tb, plan->tokens, plan->blocks, (const int*)(tb + Lt.wg_off),
                                    (const int*)(tb + Lt.list_off), s);
    }
    if (plan->tokens > 1) {
        if (plan->tokens > BL_STACK_MAX_TOKENS || plan->count < 1 || plan->count > BL_STACK_MAX_COUNT ||
            plan->entries < plan->count || plan->entries > 64 * BL_STACK_MAX_COUNT || plan->blocks < 1 ||
            plan->blocks > BL_STREAM_MAX_BLOCKS || plan->lds_bytes < BL_MB_MISC + BL_MB_WAVES * BL_MB_TILE || plan->lds_bytes > BL_MB_LDS_MAX ||
            plan->lds_bytes % 256 || plan->layout != BL_LAYOUT_K16)
            return BL_ERR_VALUE;
        const mb_layout_t Lb = mb_layout(plan->entries, plan->count, 0);
        if (plan->wg_offset != (int64_t)Lb.wg_off || plan->prep_offset != (int64_t)Lb.fin_off || plan->prep_count < 0 ||
            plan->prep_count > plan->count || plan->red_ints < 0 || (plan->prep_count > 0 && plan->red_ints < 1) ||
            plan->norm < 1 || plan->norm > 2)
            return BL_ERR_VALUE;
        if (!bl_aligned(table, 256)) return BL_ERR_ALIGN;
        if (!g_mb_attr_set.load(std::memory_order_acquire)) return BL_ERR_VALUE;   /* no table was built in this process */
        const uint8_t* tb = (const uint8_t*)table;
        if (plan->norm == 2)
            bl_stream_mb<2><<<plan->blocks, BL_MB_THREADS, (size_t)plan->lds_bytes, (hipStream_t)s>>>(
                (const bl_stream_item*)tb, (const int2*)(tb + Lb.wg_off));
        else
            bl_stream_mb<1><<<plan->blocks, BL_MB_THREADS, (size_t)plan->lds_bytes, (hipStream_t)s>>>(
                (const bl_stream_item*)tb, (const int2*)(tb + Lb.wg_off));
        if (hipGetLastError() != hipSuccess) return BL_ERR_HIP;
        if (plan->prep_count > 0)
            bl_mb_finish<<<dim3((unsigned)plan->red_ints, (unsigned)plan->prep_count), 256, 0, (hipStream_t)s>>>(
                (const bl_mb_fin_item*)(tb + Lb.fin_off));
        return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
    }
    if (plan->count < 1 || plan->count > BL_STACK_MAX_COUNT || plan->blocks < 1 ||
        plan->blocks > BL_STREAM_MAX_BLOCKS || plan->prep_count < 0 || plan->inline_count < 0 ||
        plan->prep_count + plan->inline_count > plan->count || plan->lds_bytes < 64 ||
        plan->lds_bytes > 64 * 1024 || plan->lds_bytes % 16 ||
        plan->layout < 0 || plan->layout > BL_LAYOUT_KMAJOR || plan->red_ints < 0 || plan->red_ints > BL_KM_MAX_N ||
        (plan->layout == BL_LAYOUT_KMAJOR ? plan->red_ints < 64 || plan->lds_bytes < 64 + 64 + plan->red_ints * 4
                                          : !stream_form_ok(plan->layout, plan->red_ints)))
        return BL_ERR_VALUE;
    const bl_stream_layout L = stream_layout(plan->count, 0);
    if (plan->wg_offset != (int64_t)L.wg_off || plan->prep_offset != (int64_t)L.prep_off) return BL_ERR_VALUE;
    if (!bl_aligned(table, 256)) return BL_ERR_ALIGN;
    uint8_t* base = (uint8_t*)table;
    hipStream_t st = (hipStream_t)s;
    if (plan->prep_count > 0) {
        const bl_stream_prep_item* pp = (const bl_stream_prep_item*)(base + L.prep_off);
        if (plan->norm) bl_stream_prep<true><<<plan->prep_count, 256, 0, st>>>(pp);
        else bl_stream_prep<false><<<plan->prep_count, 256, 0, st>>>(pp);
        if (hipGetLastError() != hipSuccess) return BL_ERR_HIP;
    }
    if (plan->layout == BL_LAYOUT_KMAJOR) {
        bl_stream_m1_km<<<plan->blocks, 256, (size_t)plan->lds_bytes, st>>>(
            (const bl_stream_item*)base, (const int2*)(base + L.wg_off), (plan->lds_bytes - 64) / 4 - plan->red_ints,
            plan->red_ints);
        if (hipGetLastError() != hipSuccess) return BL_ERR_HIP;
        bl_km_finish<<<dim3((unsigned)((plan->red_ints + 255) / 256), (unsigned)plan->count), 256, 0, st>>>(
            (const bl_stream_item*)base);
    } else {
        const bl_stream_item* items = (const bl_stream_item*)base;
        const int2* wg = (const int2*)(base + L.wg_off);
        int q_ints = (plan->lds_bytes - 64) / 4;
        void* args[] = {&items, &wg, &q_ints};
        if (hipLaunchKernel(stream_kernel(plan->layout, plan->red_ints), dim3((unsigned)plan->blocks), dim3(256), args,
                            (size_t)plan->lds_bytes, st) != hipSuccess)
            return BL_ERR_HIP;
    }
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}
