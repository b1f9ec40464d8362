/* Weight quantisation (absmean -> ternary, Section 2 of the BitNet b1.58 2B4T
 * report) and 2-bit packing (Section 5.1), plus the inverse for round trips.
 * Offline step: bandwidth-trivial, but every bit must match the definition in
 * bitlinear.h. */
#include "bl_device.h"
#include "bl_host.h"

#define PACK_THREADS 256

/* Partial sums of |W| in fp64: block b sums a contiguous span of float4s in a fixed order
 * (thread-strided, then a fixed LDS tree); the last block also takes the one to three values
 * behind the last float4.  Reads the matrix at the streaming rate (141 MB: 21.7 us, 6.5 TB/s). */
__global__ __launch_bounds__(PACK_THREADS) void bl_abs_sum_partial(const float* __restrict__ W, int64_t count,
                                                                    double* __restrict__ partial) {
    __shared__ double red[PACK_THREADS];
    const bl_v4f* W4 = (const bl_v4f*)W;
    const int64_t n4 = count >> 2, per = (n4 + gridDim.x - 1) / gridDim.x;
    const int64_t lo = per * blockIdx.x;
    const int64_t hi = lo + per < n4 ? lo + per : n4;
    double s = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += PACK_THREADS) {
        const bl_v4f v = W4[i];
        s += (double)fabsf(v[0]);
        s += (double)fabsf(v[1]);
        s += (double)fabsf(v[2]);
        s += (double)fabsf(v[3]);
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x < (count & 3)) s += (double)fabsf(W[n4 * 4 + threadIdx.x]);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = PACK_THREADS / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

/* What turns W into codes: the caller's partial sums, and where beta goes.  Every workgroup of a
 * packing kernel adds the partial sums up for itself, in one fixed order (mean in fp64, one
 * rounding to fp32), so the sum takes no launch of its own; the first one stores beta. */
struct bl_pack_scale {
    const double* partial;
    int np;
    double count;
    float* beta;
};

/* The threshold of the ternariser: rint(W / d) is non-zero exactly where |W| > T.  The fp32 quotient
 * rounds above 0.5 (ties to even: 0.5 itself gives 0) exactly where the real quotient is greater than
 * 0.5 + 2^-25, the midpoint between 0.5 and its successor, i.e. where |W| > d * (0.5 + 2^-25); that
 * product is exact in fp64, and T is the largest fp32 not above it.  A quotient that is NaN clamps to -1,
 * code 0: every weight where beta is NaN, the infinite ones where it is infinite (`above` is then 0).  Every
 * thread of the workgroup calls bl_pack_threshold; red: PACK_THREADS doubles of LDS. */
struct bl_ternary {
    float T;
    uint32_t above;           /* code of w > T */
};
__device__ __forceinline__ bl_ternary bl_ternary_of(float beta) {
    const double td = (double)(beta + 1e-5f) * (0.5 + 0x1p-25);
    float T = (float)td;
    if ((double)T > td) T = __uint_as_float(__float_as_uint(T) - 1);
    const bool inf = T == __builtin_inff();
    return {inf ? 0x1.fffffep127f : T, inf ? 0u : 2u};
}
__device__ __forceinline__ bl_ternary bl_pack_threshold(const bl_pack_scale& sc, double* red) {
    double s = 0.0;
    for (int i = threadIdx.x; i < sc.np; i += PACK_THREADS) s += sc.partial[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = PACK_THREADS / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    const float beta = (float)(red[0] / sc.count);
    if (blockIdx.x == 0 && threadIdx.x == 0) *sc.beta = beta;
    return bl_ternary_of(beta);
}
__device__ __forceinline__ uint32_t bl_code(float w, bl_ternary t) {
    const uint32_t c = w > t.T ? t.above : 1u;
    return w >= -t.T ? c : 0u;
}
__device__ __forceinline__ uint32_t bl_code_i8(int b) { return (uint32_t)((b < -1 ? -1 : (b > 1 ? 1 : b)) + 1); }

/* The codes of four consecutive weights, one per byte; nv < 4: the row ends behind nv of them, the
 * others are weight 0 (code 1).  The address need not be aligned beyond the element. */
template <int IN>
__device__ __forceinline__ uint32_t bl_codes4(const void* __restrict__ Wv, int64_t at, int nv, bl_ternary T) {
    if (IN == 0) {
        const float* p = (const float*)Wv + at;
        bl_v4f f = {0, 0, 0, 0};
        if (nv >= 4) {
            __builtin_memcpy(&f, p, 16);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < nv) f[e] = p[e];
        }
        uint32_t c = bl_code(f[0], T) | bl_code(f[1], T) << 8 | bl_code(f[2], T) << 16 | bl_code(f[3], T) << 24;
        if (nv < 4) c = (c & ~(~0u << (8 * nv))) | (0x01010101u & (~0u << (8 * nv)));
        return c;
    }
    const int8_t* p = (const int8_t*)Wv + at;
    uint32_t w = 0;
    if (nv >= 4) {
        __builtin_memcpy(&w, p, 4);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < nv) w |= (uint32_t)(uint8_t)p[e] << (8 * e);
    }
    return bl_code_i8((int8_t)w) | bl_code_i8((int8_t)(w >> 8)) << 8 | bl_code_i8((int8_t)(w >> 16)) << 16 |
           bl_code_i8((int8_t)(w >> 24)) << 24;
}

/* Bit position of weight i (0..15) inside its 32-bit word. */
template <int LAYOUT>
__device__ __forceinline__ int bl_bitpos(int i) {
    return LAYOUT == 0 ? 2 * i : 8 * (i & 3) + 2 * (i >> 2);
}

/* Layouts 0 and 1.  A wave takes 1024 weights at a time, four chunks of 256: lane l reads the four
 * consecutive weights 4l .. 4l+3 of a chunk (a wave-wide load is 1 KB without gaps), puts their codes
 * where they lie in the packed word, the four lanes of a quad merge theirs (two DPP steps), and lane l
 * keeps the word of chunk l % 4, so that every lane stores one.
 * c: the codes of chunk j, one per byte; layout 1: code e of the quad's lane s at bits 8e + 2s of the
 * word; layout 0: at bits 8s + 2e. */
template <int LAYOUT>
__device__ __forceinline__ uint32_t bl_quad_words(const uint32_t c[4]) {
    const int lane = threadIdx.x & 63, j = lane & 3;
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w[i] = LAYOUT == 1 ? c[i] << (2 * j) : ((c[i] | c[i] >> 6 | c[i] >> 12 | c[i] >> 18) & 0xFFu) << (8 * j);
        w[i] |= (uint32_t)bl_dpp<BL_DPP_QUAD_XOR1>((int)w[i]);
        w[i] |= (uint32_t)bl_dpp<BL_DPP_QUAD_XOR2>((int)w[i]);
    }
    return j == 0 ? w[0] : j == 1 ? w[1] : j == 2 ? w[2] : w[3];
}

/* The codes of four chunks of W that a wave has read, packed. */
template <int LAYOUT>
__device__ __forceinline__ uint32_t bl_pack_group(const bl_v4f f[4], bl_ternary T) {
    uint32_t c[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        c[j] = bl_code(f[j][0], T) | bl_code(f[j][1], T) << 8 | bl_code(f[j][2], T) << 16 | bl_code(f[j][3], T) << 24;
    return bl_quad_words<LAYOUT>(c);
}

/* fp32 weights of a matrix without padding (N % 4 == 0 and K % 64 == 0): one run of chunks.  Bound by the
 * read of W: the first loads go out before the threshold is known, the next ones before a group is
 * packed.  One comparison per sign where a division and a rint stood; 35 M weights: 24.0 us, and the 4.6 us
 * launch that added up the partial sums is gone (before: 21.9 - 23.3 us). */
template <int LAYOUT, class SCALE>
__device__ __forceinline__ void bl_pack_run(const bl_v4f* __restrict__ W, int64_t chunks, uint32_t* __restrict__ packed, const SCALE& scale) {
    const int lane = threadIdx.x & 63;
    const int64_t step = (int64_t)gridDim.x * PACK_THREADS / 16;         /* chunks of all waves together */
    int64_t c0 = ((int64_t)blockIdx.x * (PACK_THREADS / 64) + (threadIdx.x >> 6)) * 4;
    bl_v4f f[4];
    auto load = [&](int64_t c) {
#pragma unroll
        for (int j = 0; j < 4; ++j) f[j] = W[(c + j < chunks ? c + j : chunks - 1) * 64 + lane];
    };
    load(c0);
    const bl_ternary T = scale();
    while (c0 < chunks) {
        bl_v4f g[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) g[j] = f[j];
        const int64_t at = c0;
        c0 += step;
        load(c0);
        const uint32_t mine = bl_pack_group<LAYOUT>(g, T);
        if (at + (lane & 3) < chunks) packed[(at + (lane & 3)) * 16 + (lane >> 2)] = mine;
    }
}
template <int LAYOUT>
__global__ __launch_bounds__(PACK_THREADS) void bl_pack_flat(const bl_v4f* __restrict__ W, const bl_pack_scale sc, int64_t chunks,
                                                              uint32_t* __restrict__ packed) {
    __shared__ double red[PACK_THREADS];
    bl_pack_run<LAYOUT>(W, chunks, packed, [&] { return bl_pack_threshold(sc, red); });
}

/* The same matrix, large: one read of W instead of two.  beta, which every code needs, is known only when all of W has been
 * read; but a sample of W (2^20 weights in pieces of 16, spread evenly) puts it between two ends, and a weight whose code is
 * the same at both ends is settled.  bl_pack_guess writes those codes, writes the unused code 3 for the others (0.2 % of
 * normally distributed weights) and adds up |W| on its way; bl_pack_settle, with beta, takes up the words that hold a 3, from
 * W.  Where beta is not between the ends (also NaN, infinite) it packs the whole matrix again.  Exact for every
 * input: the sample decides the time alone.  Bound by the one read of W, beside the write of the codes: 13824 x 2560 53.9 ->
 * 38.6 us (sample 4, guess 25, settle 9 with their launches), 28672 x 8192 352 -> 215; with |W| heavy-tailed (0.1 % of it
 * fiftyfold) 54.0 -> 41.1, every weight undecided 53.7 -> 61, beta NaN 52.8 -> 59 (smaller matrices of such
 * weights up to 1.3 times: 5120 x 2560). */
typedef uint32_t bl_v4w __attribute__((ext_vector_type(4)));
#define PACK_SAMPLE_BLOCKS 256
#define PACK_SAMPLE_PIECES 65536                /* of 16 weights: a lane of every quad reads four */
#define PACK_GUESS_BLOCKS (BL_PACK_PARTIALS - PACK_SAMPLE_BLOCKS)
struct bl_pack_sample {                         /* in the place of one partial sum */
    float sum, squares;
};
__global__ __launch_bounds__(PACK_THREADS) void bl_abs_sum_sample(const bl_v4f* __restrict__ W, int64_t pieces, bl_pack_sample* __restrict__ out) {
    __shared__ bl_pack_sample red[PACK_THREADS / 64];
    bl_v4f f[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        f[j] = W[((int64_t)(j * 64 * PACK_SAMPLE_BLOCKS + blockIdx.x * 64 + (threadIdx.x >> 2)) * pieces / PACK_SAMPLE_PIECES) * 4 + (threadIdx.x & 3)];
    bl_pack_sample s = {0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s.sum += fabsf(f[j][i]);
            s.squares += f[j][i] * f[j][i];
        }
    for (int o = 32; o > 0; o >>= 1) {
        s.sum += __shfl_xor(s.sum, o);
        s.squares += __shfl_xor(s.squares, o);
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        s.sum = (red[0].sum + red[1].sum) + (red[2].sum + red[3].sum);
        s.squares = (red[0].squares + red[1].squares) + (red[2].squares + red[3].squares);
        out[blockIdx.x] = s;
    }
}

/* The ends: five standard deviations of the sample's mean to each side (normally distributed weights: 0.4 %), 2^-11 to 2^-5 of it. */
struct bl_pack_ends {
    float lo, hi;                               /* of beta */
};
__device__ __forceinline__ bl_pack_ends bl_guess_ends(const bl_pack_sample* __restrict__ sample, float* red) {
    static_assert(PACK_SAMPLE_BLOCKS == PACK_THREADS && PACK_THREADS == 256, "four waves, one sum per lane");
    bl_pack_sample s = sample[threadIdx.x];
    for (int o = 32; o > 0; o >>= 1) {
        s.sum += __shfl_xor(s.sum, o);
        s.squares += __shfl_xor(s.squares, o);
    }
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = s.sum;
        red[4 + (threadIdx.x >> 6)] = s.squares;
    }
    __syncthreads();
    const float n = 16.0f * PACK_SAMPLE_PIECES;
    const float mean = ((red[0] + red[1]) + (red[2] + red[3])) / n, square = ((red[4] + red[5]) + (red[6] + red[7])) / n;
    const float far = 5.0f * __builtin_sqrtf(square / (mean * mean) / n);
    const float d = far > 0x1p-5f ? 0x1p-5f : far > 0x1p-11f ? far : 0x1p-11f;
    return {mean * (1.0f - d), mean * (1.0f + d)};
}

/* The sum over a workgroup, by lanes, then by waves. */
__device__ __forceinline__ double bl_sum_waves(double s, double* red) {
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

template <int LAYOUT, bool NT>
__global__ __launch_bounds__(PACK_THREADS) void bl_pack_guess(const bl_v4f* __restrict__ W, const bl_pack_sample* __restrict__ sample, int64_t chunks,
                                                               uint32_t* __restrict__ packed, double* __restrict__ partial) {
    __shared__ double red[PACK_THREADS / 64];
    __shared__ float ends[8];
    const int lane = threadIdx.x & 63;
    const int64_t step = (int64_t)gridDim.x * PACK_THREADS / 16;         /* chunks of all waves together */
    int64_t c0 = ((int64_t)blockIdx.x * (PACK_THREADS / 64) + (threadIdx.x >> 6)) * 4;
    bl_v4f f[4];
    auto load = [&](int64_t c) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bl_v4f* p = W + (c + j < chunks ? c + j : chunks - 1) * 64 + lane;
            f[j] = NT ? __builtin_nontemporal_load(p) : *p;
        }
    };
    load(c0);
    const bl_pack_ends e = bl_guess_ends(sample, ends);
    const float T0 = bl_ternary_of(e.lo).T, T1 = bl_ternary_of(e.hi).T;
    double s = 0.0;
    while (c0 < chunks) {
        uint32_t c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float w = f[j][i];
                const uint32_t sure = w > T1 ? 2u : w >= -T1 ? 3u : 0u;
                c[j] |= (fabsf(w) <= T0 ? 1u : sure) << (8 * i);
            }
            if (c0 + j < chunks)
                s += ((double)fabsf(f[j][0]) + (double)fabsf(f[j][1])) + ((double)fabsf(f[j][2]) + (double)fabsf(f[j][3]));
        }
        const int64_t at = c0;
        c0 += step;
        load(c0);
        const uint32_t mine = bl_quad_words<LAYOUT>(c);
        if (at + (lane & 3) < chunks) packed[(at + (lane & 3)) * 16 + (lane >> 2)] = mine;
    }
    s = bl_sum_waves(s, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

/* The words that hold a 3 are gathered by the wave, a quad of lanes takes one each. */
template <int LAYOUT>
__global__ __launch_bounds__(PACK_THREADS) void bl_pack_settle(const bl_v4f* __restrict__ W, const bl_pack_sample* __restrict__ sample,
                                                                const bl_pack_scale sc, int64_t quads, uint32_t* __restrict__ packed) {
    __shared__ double red[PACK_THREADS / 64];
    __shared__ float ends[8];
    __shared__ uint8_t list[PACK_THREADS / 64][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t step = (int64_t)gridDim.x * PACK_THREADS;
    int64_t g0 = (int64_t)blockIdx.x * PACK_THREADS + wave * 64;
    const bl_v4w* p4 = (const bl_v4w*)packed;
    bl_v4w next = p4[g0 + lane < quads ? g0 + lane : quads - 1];
    double sum = 0.0;
    for (int i = threadIdx.x; i < sc.np; i += PACK_THREADS) sum += sc.partial[i];
    const bl_pack_ends e = bl_guess_ends(sample, ends);
    const float beta = (float)(bl_sum_waves(sum, red) / sc.count);
    if (blockIdx.x == 0 && threadIdx.x == 0) *sc.beta = beta;
    const bl_ternary T = bl_ternary_of(beta);
    if (!(beta >= e.lo && beta <= e.hi && e.hi < __builtin_inff())) {
        bl_pack_run<LAYOUT>(W, quads / 4, packed, [&] { return T; });
        return;
    }
    for (; g0 < quads; g0 += step) {
        const bl_v4w w = next;
        const int64_t gn = g0 + step + lane;
        next = p4[gn < quads ? gn : quads - 1];
        int n = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool redo = g0 + lane < quads && (w[j] & (w[j] >> 1) & 0x55555555u) != 0;
            const uint64_t m = __ballot(redo);
            if (redo) list[wave][n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0))] = (uint8_t)(lane * 4 + j);
            n += __builtin_popcountll(m);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (n > 128) {                          /* most of them: whole chunks, read without gaps */
            for (int i = 0; i < 16; i += 4) {
                const int64_t c0 = g0 / 4 + i, chunks = quads / 4;
                bl_v4f f[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) f[j] = W[(c0 + j < chunks ? c0 + j : chunks - 1) * 64 + lane];
                const uint32_t v = bl_pack_group<LAYOUT>(f, T);
                if (c0 + (lane & 3) < chunks) packed[(c0 + (lane & 3)) * 16 + (lane >> 2)] = v;
            }
            continue;
        }
        for (int i = 0; i < n; i += 32) {
            bl_v4f f[2];
            int64_t word[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int at = i + 16 * h + (lane >> 2);
                word[h] = g0 * 4 + list[wave][at < n ? at : n - 1];
                f[h] = W[word[h] * 4 + (lane & 3)];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t v = 0;
#pragma unroll
                for (int t = 0; t < 4; ++t) v |= bl_code(f[h][t], T) << (LAYOUT == 1 ? 8 * t + 2 * (lane & 3) : 8 * (lane & 3) + 2 * t);
                v |= (uint32_t)bl_dpp<BL_DPP_QUAD_XOR1>((int)v);
                v |= (uint32_t)bl_dpp<BL_DPP_QUAD_XOR2>((int)v);
                if (i + 16 * h + (lane >> 2) < n && (lane & 3) == 0) packed[word[h]] = v;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

/* Any shape: a row is wpr words, chunks do not cross rows, what lies outside the matrix is code 1.
 * 5003 x 2999: 12.6 us (before, a thread per word with element loads: 42). */
template <int LAYOUT, int IN>
__global__ __launch_bounds__(PACK_THREADS) void bl_pack_words(const void* __restrict__ Wv, const bl_pack_scale sc, int64_t N,
                                                               int64_t K, int64_t wpr, uint32_t* __restrict__ packed) {
    __shared__ double red[PACK_THREADS];
    const bl_ternary T = IN == 0 ? bl_pack_threshold(sc, red) : bl_ternary{};
    const int lane = threadIdx.x & 63;
    const int64_t cpr = (wpr + 15) / 16, chunks = (N + 3) / 4 * 4 * cpr;
    const int64_t waves = (int64_t)gridDim.x * (PACK_THREADS / 64);
    for (int64_t c0 = ((int64_t)blockIdx.x * (PACK_THREADS / 64) + (threadIdx.x >> 6)) * 4; c0 < chunks; c0 += waves * 4) {
        int64_t n = c0 / cpr, kc = c0 - n * cpr, to = -1;
        uint32_t c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t k = kc * 256 + lane * 4, word = kc * 16 + (lane >> 2);
            const int64_t left = c0 + j < chunks && n < N ? K - k : 0;
            c[j] = bl_codes4<IN>(Wv, n * K + k, left >= 4 ? 4 : left < 0 ? 0 : (int)left, T);
            if ((lane & 3) == j && c0 + j < chunks && word < wpr) to = n * wpr + word;
            if (++kc == cpr) {
                kc = 0;
                ++n;
            }
        }
        const uint32_t mine = bl_quad_words<LAYOUT>(c);
        if (to >= 0) packed[to] = mine;
    }
}

/* Weights that are ternary int8 already, without padding: 16 bytes in, one word out per thread. */
template <int LAYOUT>
__global__ __launch_bounds__(PACK_THREADS) void bl_pack_int8(const bl_v4i* __restrict__ Wt, int64_t words,
                                                              uint32_t* __restrict__ packed) {
    const int64_t g = (int64_t)blockIdx.x * PACK_THREADS + threadIdx.x;
    if (g >= words) return;
    const bl_v4i v = Wt[g];
    uint32_t w = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) w |= bl_code_i8((int8_t)((uint32_t)v[i >> 2] >> (8 * (i & 3)))) << bl_bitpos<LAYOUT>(i);
    packed[g] = w;
}

template <int LAYOUT>
__global__ __launch_bounds__(PACK_THREADS) void bl_unpack_kernel(const uint32_t* __restrict__ packed, int64_t words,
                                                                  bl_v4i* __restrict__ Wt, int32_t* __restrict__ bad) {
    const int64_t g = (int64_t)blockIdx.x * PACK_THREADS + threadIdx.x;
    if (g >= words) return;
    const uint32_t w = packed[g];
    bl_v4i out = {0, 0, 0, 0};
    int nbad = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int c = (int)((w >> bl_bitpos<LAYOUT>(i)) & 3u);
        nbad += (c == 3);
        out[i >> 2] |= (int)(((uint32_t)(c - 1) & 0xFFu) << (8 * (i & 3)));
    }
    Wt[g] = out;
    if (nbad) atomicAdd(bad, nbad);
}

/* ---- shapes with a ragged K (not a multiple of 64) or N (not a multiple of 4) ------------------ */
template <int LAYOUT>
__global__ __launch_bounds__(PACK_THREADS) void bl_unpack_any(const uint32_t* __restrict__ packed, int64_t N, int64_t K,
                                                               int64_t wpr, int64_t words, int8_t* __restrict__ Wt,
                                                               int32_t* __restrict__ bad) {
    const int64_t g = (int64_t)blockIdx.x * PACK_THREADS + threadIdx.x;
    if (g >= words) return;
    const int64_t n = g / wpr, k0 = (g % wpr) * 16;
    if (n >= N) return;
    const uint32_t w = packed[g];
    int nbad = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int c = (int)((w >> bl_bitpos<LAYOUT>(i)) & 3u);
        if (k0 + i < K) {
            nbad += (c == 3);
            Wt[n * K + k0 + i] = (int8_t)(c - 1);
        }
    }
    if (nbad) atomicAdd(bad, nbad);
}

/* ---- five weights per byte (BL_LAYOUT_TRIT5, see bitlinear.h) -----------------------------------
 * One thread = one 4-byte word = 20 consecutive k of one padded row; byte j of the word holds
 * k = 20g + 4i + j, i = 0..4, leading digit first.  The five digits of all four bytes are put
 * together at once (v = 3 v + c on four bytes: at most 242, nothing crosses a byte), then
 * b = ceil(256 v / 243) = v + ceil(13 v / 243) byte by byte.  Five 16-byte loads per thread instead of
 * twenty of four bytes: 13824 x 2560 27 us (before: 122). */
template <int IN>
__global__ __launch_bounds__(PACK_THREADS) void bl_pack_t5(const void* __restrict__ Wv, const bl_pack_scale sc, int64_t N,
                                                            int64_t K, int64_t wpr, int64_t words,
                                                            uint32_t* __restrict__ packed) {
    __shared__ double red[PACK_THREADS];
    const bl_ternary T = IN == 0 ? bl_pack_threshold(sc, red) : bl_ternary{};
    for (int64_t g = (int64_t)blockIdx.x * PACK_THREADS + threadIdx.x; g < words; g += (int64_t)gridDim.x * PACK_THREADS) {
        const int64_t n = g / wpr, k0 = (g - n * wpr) * 20;
        uint32_t c[5], v = 0;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int64_t left = n < N ? K - (k0 + 4 * i) : 0;
            c[i] = bl_codes4<IN>(Wv, n * K + k0 + 4 * i, left >= 4 ? 4 : left < 0 ? 0 : (int)left, T);
        }
#pragma unroll
        for (int i = 0; i < 5; ++i) v = v * 3 + c[i];
        uint32_t word = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t b = (v >> (8 * j)) & 0xFFu;
            word |= (b + (13 * b + 242) / 243) << (8 * j);
        }
        packed[g] = word;
    }
}

__global__ __launch_bounds__(PACK_THREADS) void bl_unpack_t5(const uint32_t* __restrict__ packed, int64_t N, int64_t K,
                                                              int64_t wpr, int64_t words, int8_t* __restrict__ Wt,
                                                              int32_t* __restrict__ bad) {
    const int64_t g = (int64_t)blockIdx.x * PACK_THREADS + threadIdx.x;
    if (g >= words) return;
    const int64_t n = g / wpr, k0 = (g % wpr) * 20;
    if (n >= N) return;
    const uint32_t w = packed[g];
    int nbad = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t b = (w >> (8 * j)) & 0xFFu;
        uint32_t r = b, v = 0;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const uint32_t t = r * 3;
            const int c = (int)(t >> 8);
            r = t & 0xFFu;
            v = v * 3 + (uint32_t)c;
            const int64_t k = k0 + 4 * i + j;
            if (k < K) Wt[n * K + k] = (int8_t)(c - 1);
        }
        nbad += ((v * 256 + 242) / 243 != b);          /* a byte that is not the code of its own digits */
    }
    if (nbad) atomicAdd(bad, nbad);
}

/* ---- k-major form (BL_LAYOUT_KMAJOR, see bitlinear.h): the transposed matrix, one row per k ------
 * A workgroup takes 64 k x 64 J n (J = 4, or 1 where that would leave compute units without work): lane = k, so that a wave reads 64 consecutive weights of a row of W
 * at a time; each thread packs J words (16 rows n each), which go through LDS so that the 16 J bytes
 * of a k leave together.  2560 x 6912: 31 us (before, a thread per word with the lanes 16 rows apart: 125). */
template <int IN, int J>
__global__ __launch_bounds__(PACK_THREADS) void bl_pack_km(const void* __restrict__ Wv, const bl_pack_scale sc, int64_t N,
                                                            int64_t K, int64_t wpr, uint32_t* __restrict__ packed) {
    __shared__ double red[PACK_THREADS];
    __shared__ uint32_t tile[64][4 * J + 1];
    const bl_ternary T = IN == 0 ? bl_pack_threshold(sc, red) : bl_ternary{};
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t kt = (K + 63) / 64, nt = (wpr + 4 * J - 1) / (4 * J);
    for (int64_t t = blockIdx.x; t < kt * nt; t += gridDim.x) {
        const int64_t tn = t / kt, k = (t - tn * kt) * 64 + lane, nw0 = (tn * 4 + w) * J;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            uint32_t word = 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int64_t n = (nw0 + j) * 16 + i;
                uint32_t c = 1;
                if (n < N && k < K) c = IN == 0 ? bl_code(((const float*)Wv)[n * K + k], T) : bl_code_i8(((const int8_t*)Wv)[n * K + k]);
                word |= c << (2 * i);
            }
            tile[lane][w * J + j] = word;
        }
        __syncthreads();
        const int64_t ko = (t - tn * kt) * 64 + (threadIdx.x >> 2);
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int64_t nw = (tn * 4 + (threadIdx.x & 3)) * J + j;
            if (ko < K && nw < wpr) packed[ko * wpr + nw] = tile[threadIdx.x >> 2][(threadIdx.x & 3) * J + j];
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(PACK_THREADS) void bl_unpack_km(const uint32_t* __restrict__ packed, int64_t N, int64_t K,
                                                              int64_t wpr, int64_t words, int8_t* __restrict__ Wt,
                                                              int32_t* __restrict__ bad) {
    const int64_t g = (int64_t)blockIdx.x * PACK_THREADS + threadIdx.x;
    if (g >= words) return;
    const int64_t k = g / wpr, n0 = (g % wpr) * 16;
    const uint32_t w = packed[g];
    int nbad = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int c = (int)((w >> (2 * i)) & 3u);
        if (n0 + i < N) {
            nbad += (c == 3);
            Wt[(n0 + i) * K + k] = (int8_t)(c - 1);
        }
    }
    if (nbad) atomicAdd(bad, nbad);
}

__global__ void bl_zero_i32(int32_t* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

/* From 12 Mi weights: the third launch costs what the shorter read saves at about 10 (1920 x 5120 17.3 us in two reads, 17.1
 * with a guess; 2560 x 2560 14.1 and 14.6; 2560 x 6912 24.7 and 22.8).  Non-temporal loads from 128 MiB of W (4096 x 11008 50.1
 * us without, 46.3 with them; 13824 x 2560 39.6, 37.9; 2560 x 6912 22.8, 23.3: the settling finds less of W in the caches). */
#define PACK_GUESS_COUNT (12 << 20)
#define PACK_NT_COUNT (32 << 20)
template <int LAYOUT>
static bl_status launch_pack_guess(const bl_v4f* W, int64_t count, uint8_t* packed, float* beta, double* partial, hipStream_t st) {
    const int64_t chunks = count / 256, quads = count / 64, blocks = (quads + PACK_THREADS - 1) / PACK_THREADS;
    bl_pack_sample* sample = (bl_pack_sample*)(partial + PACK_GUESS_BLOCKS);
    const bl_pack_scale sc = {partial, PACK_GUESS_BLOCKS, (double)count, beta};
    bl_abs_sum_sample<<<PACK_SAMPLE_BLOCKS, PACK_THREADS, 0, st>>>(W, count / 16, sample);
    if (count < PACK_NT_COUNT) bl_pack_guess<LAYOUT, false><<<PACK_GUESS_BLOCKS, PACK_THREADS, 0, st>>>(W, sample, chunks, (uint32_t*)packed, partial);
    else bl_pack_guess<LAYOUT, true><<<PACK_GUESS_BLOCKS, PACK_THREADS, 0, st>>>(W, sample, chunks, (uint32_t*)packed, partial);
    bl_pack_settle<LAYOUT><<<(unsigned)(blocks < 1024 ? blocks : 1024), PACK_THREADS, 0, st>>>(W, sample, sc, quads, (uint32_t*)packed);
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}

extern "C" bl_status bl_pack_ternary(const void* W, int in_kind, int64_t N, int64_t K, int layout,
                                     uint8_t* packed, float* beta, void* workspace, bl_stream s) {
    if (!W || !packed || !beta) return BL_ERR_NULL;
    if (!bl_shape_ok(N, K)) return BL_ERR_SHAPE;
    if (layout < BL_LAYOUT_ROWMAJOR || layout > BL_LAYOUT_KMAJOR) return BL_ERR_LAYOUT;
    if (in_kind != BL_IN_FP32_LATENT && in_kind != BL_IN_INT8_TERNARY) return BL_ERR_VALUE;
    if (!bl_aligned(W, 16) || !bl_aligned(packed, 16) || !bl_aligned(beta, 4)) return BL_ERR_ALIGN;
    hipStream_t st = (hipStream_t)s;
    const bool latent = in_kind == BL_IN_FP32_LATENT;
    bl_pack_scale sc = {};
    if (latent) {
        if (!workspace) return BL_ERR_WORKSPACE;
        if (!bl_aligned(workspace, 8)) return BL_ERR_ALIGN;
        const int64_t count = N * K, n4 = count / 4;
        if (bl_shape_unpadded(N, K) && count >= PACK_GUESS_COUNT && (layout == BL_LAYOUT_ROWMAJOR || layout == BL_LAYOUT_K16)) {
            if (layout == BL_LAYOUT_ROWMAJOR) return launch_pack_guess<0>((const bl_v4f*)W, count, packed, beta, (double*)workspace, st);
            return launch_pack_guess<1>((const bl_v4f*)W, count, packed, beta, (double*)workspace, st);
        }
        sc.partial = (double*)workspace;
        sc.np = (int)(n4 < 1 ? 1 : n4 < BL_PACK_PARTIALS ? n4 : BL_PACK_PARTIALS);
        sc.count = (double)count;
        sc.beta = beta;
        bl_abs_sum_partial<<<sc.np, PACK_THREADS, 0, st>>>((const float*)W, count, (double*)workspace);
    }
    uint32_t* out = (uint32_t*)packed;
    /* grids of what is resident at once (eight workgroups per compute unit): each adds the partial sums up once */
    const auto grid = [](int64_t blocks) { return (unsigned)(blocks < 8 * 256 ? blocks : 8 * 256); };
    if (layout == BL_LAYOUT_KMAJOR) {
        const int64_t wpr = (N + 63) / 64 * 4, kt = (K + 63) / 64, tiles = kt * ((wpr + 15) / 16), tiles1 = kt * (wpr / 4);
        /* (896 x 704 from int8: with 154 workgroups of one word per thread 5.4 us; 44 of four words made the
         * call 1.7 us longer) */
        if (tiles >= 1024) {
            if (latent) bl_pack_km<0, 4><<<grid(tiles), PACK_THREADS, 0, st>>>(W, sc, N, K, wpr, out);
            else bl_pack_km<1, 4><<<grid(tiles), PACK_THREADS, 0, st>>>(W, sc, N, K, wpr, out);
        } else {
            if (latent) bl_pack_km<0, 1><<<grid(tiles1), PACK_THREADS, 0, st>>>(W, sc, N, K, wpr, out);
            else bl_pack_km<1, 1><<<grid(tiles1), PACK_THREADS, 0, st>>>(W, sc, N, K, wpr, out);
        }
    } else if (layout == BL_LAYOUT_TRIT5) {
        const int64_t wpr = bl_kpad5(K) / 20, words = bl_npad(N) * wpr;
        const unsigned g = grid((words + PACK_THREADS - 1) / PACK_THREADS);
        if (latent) bl_pack_t5<0><<<g, PACK_THREADS, 0, st>>>(W, sc, N, K, wpr, words, out);
        else bl_pack_t5<1><<<g, PACK_THREADS, 0, st>>>(W, sc, N, K, wpr, words, out);
    } else {
        const int64_t wpr = bl_kpad(K) / 16, words = bl_npad(N) * wpr;
        if (bl_shape_unpadded(N, K)) {
            const unsigned g = grid((words + 16 * 16 - 1) / (16 * 16)), g8 = (unsigned)((words + PACK_THREADS - 1) / PACK_THREADS);
            if (latent && layout == 0) bl_pack_flat<0><<<g, PACK_THREADS, 0, st>>>((const bl_v4f*)W, sc, words / 16, out);
            else if (latent) bl_pack_flat<1><<<g, PACK_THREADS, 0, st>>>((const bl_v4f*)W, sc, words / 16, out);
            else if (layout == 0) bl_pack_int8<0><<<g8, PACK_THREADS, 0, st>>>((const bl_v4i*)W, words, out);
            else bl_pack_int8<1><<<g8, PACK_THREADS, 0, st>>>((const bl_v4i*)W, words, out);
        } else {
            const unsigned g = grid((bl_npad(N) * ((wpr + 15) / 16) + 15) / 16);
            if (layout == 0 && latent) bl_pack_words<0, 0><<<g, PACK_THREADS, 0, st>>>(W, sc, N, K, wpr, out);
            else if (layout == 0) bl_pack_words<0, 1><<<g, PACK_THREADS, 0, st>>>(W, sc, N, K, wpr, out);
            else if (latent) bl_pack_words<1, 0><<<g, PACK_THREADS, 0, st>>>(W, sc, N, K, wpr, out);
            else bl_pack_words<1, 1><<<g, PACK_THREADS, 0, st>>>(W, sc, N, K, wpr, out);
        }
    }
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}

extern "C" bl_status bl_unpack_ternary(const uint8_t* packed, int64_t N, int64_t K, int layout,
                                       int8_t* Wt, int32_t* bad, bl_stream s) {
    if (!packed || !Wt || !bad) return BL_ERR_NULL;
    if (!bl_shape_ok(N, K)) return BL_ERR_SHAPE;
    if (layout < BL_LAYOUT_ROWMAJOR || layout > BL_LAYOUT_KMAJOR) return BL_ERR_LAYOUT;
    if (!bl_aligned(packed, 16) || !bl_aligned(Wt, 16) || !bl_aligned(bad, 4)) return BL_ERR_ALIGN;
    hipStream_t st = (hipStream_t)s;
    if (layout == BL_LAYOUT_TRIT5 || layout == BL_LAYOUT_KMAJOR) {
        const bool km = layout == BL_LAYOUT_KMAJOR;
        const int64_t wpr = km ? (N + 63) / 64 * 4 : bl_kpad5(K) / 20, pwords = (km ? K : bl_npad(N)) * wpr;
        const unsigned pgrid = (unsigned)((pwords + PACK_THREADS - 1) / PACK_THREADS);
        bl_zero_i32<<<1, 64, 0, st>>>(bad, 1);
        if (km) bl_unpack_km<<<pgrid, PACK_THREADS, 0, st>>>((const uint32_t*)packed, N, K, wpr, pwords, Wt, bad);
        else bl_unpack_t5<<<pgrid, PACK_THREADS, 0, st>>>((const uint32_t*)packed, N, K, wpr, pwords, Wt, bad);
        return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
    }
    if (!bl_shape_unpadded(N, K)) {
        const int64_t wpr = bl_kpad(K) / 16, pwords = bl_npad(N) * wpr;
        const unsigned pgrid = (unsigned)((pwords + PACK_THREADS - 1) / PACK_THREADS);
        bl_zero_i32<<<1, 64, 0, st>>>(bad, 1);
        if (layout == 0) bl_unpack_any<0><<<pgrid, PACK_THREADS, 0, st>>>((const uint32_t*)packed, N, K, wpr, pwords, Wt, bad);
        else bl_unpack_any<1><<<pgrid, PACK_THREADS, 0, st>>>((const uint32_t*)packed, N, K, wpr, pwords, Wt, bad);
        return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
    }
    const int64_t words = N * K / 16;
    const unsigned grid = (unsigned)((words + PACK_THREADS - 1) / PACK_THREADS);
    bl_zero_i32<<<1, 64, 0, st>>>(bad, 1);
    if (layout == 0)
        bl_unpack_kernel<0><<<grid, PACK_THREADS, 0, st>>>((const uint32_t*)packed, words, (bl_v4i*)Wt, bad);
    else
        bl_unpack_kernel<1><<<grid, PACK_THREADS, 0, st>>>((const uint32_t*)packed, words, (bl_v4i*)Wt, bad);
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}
