/* Decode product of ONE token and ONE matrix (Section 5.1 of the BitNet b1.58 2B4T report), with
 * the producer, the normalisation and the per-token quantiser of Section 2 in front of it: the
 * kernel of a dependent chain of BitLinears, where a launch moves 1.6 - 8.8 MB of weights and its
 * length is a serial chain (arguments -> row -> sum of squares -> absmax -> quantised row -> dot
 * products -> store), not bandwidth.
 *
 * What shortens that chain here: one workgroup of four waves per compute unit (what every wave does
 * for itself is then done once per SIMD: with 8 / 16 waves the thirty-layer chain took 636 / 657 us
 * against 590); all loads of the row and the weights go out in one step, without a branch in between
 * (global, not flat, and unconditional, so that the waits count exactly: 657 against 745); 16 or 32 lanes
 * on a weight row, whose activations sit in registers, read from LDS once for all rows of the wave;
 * reductions by DPP and readlane; two barriers, with normalisation too (the row maximum is settled
 * from the sum of squares and max|t*gain|, which meet together).
 * Measured in the chain (N x K, norm on; launch boundary 1.6 us included): 3840 x 2560 3.9 us,
 * 2560 x 2560 4.0, 13824 x 2560 5.1, 2560 x 6912 6.0, against 5.8 / 5.8 / 8.0 / 8.6 on bl_gemv_rows.
 * What is left: 1.3 - 1.6 us launch boundary, about 1 us until the row has come from beyond the L2,
 * two exchanges through LDS, and the vector instructions of a whole row on every compute unit. */
#include <type_traits>

#include "bl_device.h"
#include "bl_gemv_common.h"
#include "bl_host.h"
#include "bl_producer.h"

#define BL_ONE_GAIN_MAX 0x1p40f   /* normalisation gains beyond it take the maximum of the row itself */
#define BL_ONE_WAVES 4            /* (bl_few_sum and bl_few_max join four) */
#define BL_ONE_QSTRIDE 80     /* bytes of LDS per 64-wide k chunk: 16 lanes reading 16 bytes each meet 64 banks */

template <int CTRL>
__device__ __forceinline__ double bl_dppd(double v) {
    return __hiloint2double(bl_dpp<CTRL>(__double2hiint(v)), bl_dpp<CTRL>(__double2loint(v)));
}
__device__ __forceinline__ double bl_row_sum(double v) {
    v += bl_dppd<BL_DPP_QUAD_XOR1>(v);
    v += bl_dppd<BL_DPP_QUAD_XOR2>(v);
    v += bl_dppd<BL_DPP_ROW_HALF_MIRROR>(v);
    return v + bl_dppd<BL_DPP_ROW_MIRROR>(v);
}
/* Over aligned groups of four lanes (one value per wave). */
__device__ __forceinline__ double bl_few_sum(double v) {
    v += bl_dppd<BL_DPP_QUAD_XOR1>(v);
    return v + bl_dppd<BL_DPP_QUAD_XOR2>(v);
}
__device__ __forceinline__ float bl_few_max(float v) {
    v = bl_max_pos(v, bl_dppf<BL_DPP_QUAD_XOR1>(v));
    return bl_max_pos(v, bl_dppf<BL_DPP_QUAD_XOR2>(v));
}
/* Sum over the G = 16 or 32 lanes of a weight row, in every one of them. */
template <int G>
__device__ __forceinline__ int bl_lanes_sum(int v) {
    static_assert(G == 16 || G == 32, "");
    v = bl_group_sum<16>(v);
    if (G == 32) {
        const auto t = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
        v = (int)(t[0] + t[1]);
    }
    return v;
}
__device__ __forceinline__ double bl_lane_d(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}

/* 1 / sqrt(v) in fp64: the hardware estimate and two Newton steps (relative error ~1e-15; a
 * correctly rounded square root and two divisions are a chain of ~40 dependent fp64 operations). */
__device__ __forceinline__ double bl_rsqrt64(double v) {
    double r = __builtin_amdgcn_rsq(v);
#pragma unroll
    for (int i = 0; i < 2; ++i) r = r * (1.5 - 0.5 * v * r * r);
    return r;
}

/* The factor r = fp32(1 / sqrt(ss / K + eps)) of the normalisation, the bits of those fp64 operations rounded
 * one by one.  The fast form is off by less than 2^-50 (the estimate's last step, inv_k for a division),
 * they by less than 2^-51, so it rounds like them unless it lies within 2^-47 of the midpoint of two fp32,
 * which the 29 bits that the rounding drops tell.  About one row in 2^22, and rows whose sum is zero,
 * infinite or NaN, take the operations themselves; every thread of the workgroup decides on the same sum. */
__device__ __forceinline__ float bl_norm_factor(double ss, double inv_k, int K, float eps) {
    const double e = bl_rsqrt64(ss * inv_k + (double)eps);
    float r = (float)e;
    const uint32_t off = (__double2loint(e) & 0x1FFFFFFFu) - (0x10000000u - 32u);
    if (__builtin_expect(!(off > 64u && r > 0x1p-126f && r < __builtin_inff()), 0))
        r = (float)(1.0 / sqrt(ss / (double)K + (double)eps));
    return r;
}

/* What the kernel needs to know late, fetched from the arguments in one go ... */
struct bl_one_rest {
    float* aux_out;
    const float* beta;
    const float* scale;              /* int8 input */
    int32_t* acc;
    float* y;
    int8_t* q_out;
    float* scale_out;
    double inv_k;
    int layout;
    float eps, fixed_scale;
};
/* ... and what its first loads need (bl_gemv_one). */
struct bl_one_args : bl_one_rest {
    const void* packed;
    const void* in0;                 /* bf16, fp32 or int8 row */
    const float* in1;                /* second fp32 row: the other summand, or the up half */
    const float* gain;
    const float* residual;
    int N, K, rows;                  /* rows of a workgroup */
    int kind, voff, hd;
    uint32_t mul_hd, mul_group;      /* V gather: ceil(2^32 / .): quotients by a multiply (mul_group = 0: group 1) */
};
typedef uint32_t bl_v4u __attribute__((ext_vector_type(4)));
enum { BL_ONE_BF16, BL_ONE_F32, BL_ONE_PAIR, BL_ONE_INT8, BL_ONE_V };   /* plain, residual or gate, quantised, V gather */

/* G lanes share a weight row (64 / G rows at a time, RW times); NL: 16-byte weight loads per lane and
 * row (K <= 64 * G * NL); UN: units of four elements of the activation row per thread (K <= 4 * UN *
 * threads).  SRC and NORM fix which loads there are, so that all of them go out without a wait. */
template <int SRC, int G, int RW, int NL, int UN, bool NORM>
/* What the row's and the weights' loads need comes first, 14 registers of it (`where`: weights, row; `beside`: second row or the two
 * multipliers of the V gather, gains; `size`: residual, N, K; `how`: rows of a workgroup | kind << 8 | head size << 16, offset of V):
 * the hardware has them in place when a wave starts (the build asks for that), the structure behind them is fetched while the loads
 * travel.  One token through thirty layers 545 - 558 -> 528 - 545 us (1.03), fifteen without normalisation 240 -> 231 (the same
 * fetched by the kernel: half of that); an eager call gains nothing, the host bounds it.  Four vectors and not nine scalars, which cost the host .2 us more a launch. */
__global__ __launch_bounds__(BL_ONE_WAVES * 64) void bl_gemv_one(const bl_v4u where, const bl_v4u beside, const bl_v4u size, const bl_v2u how,
                                                                 const bl_one_rest Pin) {
    constexpr int R = 64 / G, NW = BL_ONE_WAVES, nthreads = NW * 64;
    __shared__ __attribute__((aligned(16))) uint8_t Qs[SRC == BL_ONE_INT8 ? 16 : (G * NL + 1) * BL_ONE_QSTRIDE];
    __shared__ float fs[NW];
    __shared__ double sd[NW];
    __shared__ int qsum[NW];
    const auto wide = [](uint32_t lo, uint32_t hi) { return (uint64_t)hi << 32 | lo; };
    const void *const packed = (const void*)wide(where[0], where[1]), *const in0 = (const void*)wide(where[2], where[3]);
    const uint64_t second = wide(beside[0], beside[1]);
    const float *const in1 = (const float*)second, *const gain = (const float*)wide(beside[2], beside[3]);
    const float* const residual = (const float*)wide(size[0], size[1]);
    const int N = (int)size[2], K = (int)size[3], voff = (int)how[1];
    const uint32_t rows_kind = how[0];
    const int rows = rows_kind & 0xFF, kind = (rows_kind >> 8) & 0xFF;
    const int nchunks = K >> 6;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int units = K >> 2;
    const bool first_block = blockIdx.x == 0;
    const bool norm = NORM;
    const int r = lane / G, g = lane % G;
    const int n0 = (int)blockIdx.x * rows + w * RW * R;  /* first row of this wave; row j * R + r is lane (r, g)'s */
    const int nend = min(N, ((int)blockIdx.x + 1) * rows);

    /* 1. every load of the row, then every load of the weights.  All but the residual's are
     * unconditional (out of range: a valid address, and a zero chunk of activations or no store), so
     * the waits count exactly and the row is not waited for together with the weights. */
    float res = 0.0f;
    if (residual && g < RW && n0 + g * R + r < nend) res = bl_gc<float>(residual)[n0 + g * R + r];
    bl_v4i aq[NL][4];                                      /* this lane's activations: dword s of packed word d */
    bl_v2u xb[UN];
    bl_v4f ra[UN], rb[UN], rg[UN];
    const bool has_gain = NORM && gain != nullptr;
    if (SRC != BL_ONE_INT8) {
#pragma unroll
        for (int j = 0; j < UN; ++j) {
            int u = tid + j * nthreads;
            u = u < units ? u : units - 1;
            if (SRC == BL_ONE_BF16) {
                xb[j] = bl_gc<bl_v2u>(in0)[u];
            } else {
                int off = u * 4;
                if (SRC == BL_ONE_V) {
                    const int hd = rows_kind >> 16, head = (int)__umulhi((uint32_t)off, (uint32_t)second);
                    const uint32_t mul_group = (uint32_t)(second >> 32);
                    const int kv = mul_group ? (int)__umulhi((uint32_t)head, mul_group) : head;
                    off = voff + kv * hd + (off - head * hd);
                }
                ra[j] = *bl_gc<bl_v4f>((const float*)in0 + off);
                if (SRC == BL_ONE_PAIR) rb[j] = *bl_gc<bl_v4f>(in1 + off);
            }
            if (NORM && has_gain) rg[j] = *bl_gc<bl_v4f>(gain + u * 4);
        }
    } else {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int chunk = g + G * i;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                aq[i][d] = bl_v4i{0, 0, 0, 0};
                if (chunk < nchunks) aq[i][d] = bl_gc<bl_v4i>(in0)[chunk * 4 + d];
            }
        }
    }
    bl_v4i p[RW][NL];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < RW; ++j) {
        const int n = n0 + j * R + r;
        const bl_v4i BL_G* wrow = bl_gc<bl_v4i>(packed) + (int64_t)(n < nend ? n : nend - 1) * nchunks;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int chunk = g + G * i;
            p[j][i] = __builtin_nontemporal_load(wrow + (chunk < nchunks ? chunk : nchunks - 1));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    bl_one_rest P = Pin;
    /* one pin for all: the fields arrive together and stay in scalar registers */
    asm volatile("" : "+s"(P.aux_out), "+s"(P.beta), "+s"(P.scale), "+s"(P.acc), "+s"(P.y), "+s"(P.q_out), "+s"(P.scale_out),
                      "+s"(P.layout), "+s"(P.eps), "+s"(P.fixed_scale), "+s"(P.inv_k));
    const float bt = *bl_gc<float>(P.beta);
    float cf = 0.0f;
    int nq = 0;                                            /* sum_k q */
    if (SRC == BL_ONE_INT8 && P.scale) cf = *bl_gc<float>(P.scale);
    __builtin_amdgcn_sched_barrier(0);

    /* 2. produce, normalise, narrow, quantise */
    if (SRC != BL_ONE_INT8) {
        float v[UN][4];
        double part = 0.0;
        float um = 0.0f, gm = 0.0f;
        const int lw = lane & (NW - 1);
        if (SRC != BL_ONE_BF16 || norm) {
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                const int u = tid + j * nthreads;
                const bool inside = u < units;
                const float a[4] = {ra[j].x, ra[j].y, ra[j].z, ra[j].w}, b[4] = {rb[j].x, rb[j].y, rb[j].z, rb[j].w};
                if (SRC == BL_ONE_BF16) {
                    v[j][0] = __uint_as_float(xb[j].x << 16);
                    v[j][1] = __uint_as_float(xb[j].x & 0xFFFF0000u);
                    v[j][2] = __uint_as_float(xb[j].y << 16);
                    v[j][3] = __uint_as_float(xb[j].y & 0xFFFF0000u);
                } else if (SRC == BL_ONE_PAIR && kind == BL_PROD_RELU2_GATE) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float rl = fmaxf(a[e], 0.0f);
                        const float r2 = rl * rl;
                        v[j][e] = r2 * b[e];
                    }
                } else if (SRC == BL_ONE_PAIR) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[j][e] = a[e] + b[e];
                    if (inside && first_block && P.aux_out) *(bl_v4f BL_G*)(P.aux_out + u * 4) = bl_v4f{v[j][0], v[j][1], v[j][2], v[j][3]};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[j][e] = a[e];
                }
                if (norm && inside) {
                    const float gn[4] = {rg[j].x, rg[j].y, rg[j].z, rg[j].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        /* (an fp32 value squared is exact in fp64, so the fused form rounds as the separate one) */
                        part = __builtin_fma((double)v[j][e], (double)v[j][e], part);
                        um = fmaxf(um, fabsf(has_gain ? v[j][e] * gn[e] : v[j][e]));
                        if (has_gain) gm += fabsf(gn[e]);              /* (at least the maximum, and NaN if one is) */
                    }
                }
            }
        }
        auto narrow = [&](float rn) {
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                if (norm) {
                    const float gn[4] = {rg[j].x, rg[j].y, rg[j].z, rg[j].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[j][e] = v[j][e] * rn;
                        if (has_gain) v[j][e] *= gn[e];
                    }
                }
                xb[j] = bl_v2u{bl_pack2_bf16(v[j][0], v[j][1]), bl_pack2_bf16(v[j][2], v[j][3])};
            }
        };
        auto row_absmax = [&](auto skip_nan) {                 /* over the whole row; contains one barrier */
            bl_mag2<decltype(skip_nan)::value> m2;
#pragma unroll
            for (int j = 0; j < UN; ++j) {                     /* (a thread beyond the row holds its last unit again) */
                m2.take(xb[j].x);
                m2.take(xb[j].y);
            }
            const float mx = bl_wave_max(m2.get());
            if (lane == 0) fs[w] = mx;
            __syncthreads();
            return bl_few_max(fs[lw]);
        };
        /* the rows that may hold a NaN take their maximum and their quantiser with it in mind */
        bool special = false;
        float gamma = 0.0f;
        if (norm) {
            part = bl_row_sum(part);
            part = (bl_lane_d(part, 0) + bl_lane_d(part, 16)) + (bl_lane_d(part, 32) + bl_lane_d(part, 48));
            um = bl_wave_max(gm <= BL_ONE_GAIN_MAX ? um : __builtin_inff());
            if (lane == 0) {
                sd[w] = part;
                fs[w] = um;
            }
            __syncthreads();
            const double ss = bl_few_sum(sd[lw]);
            const float U = bl_few_max(fs[lw]);
            const float rn = bl_norm_factor(ss, P.inv_k, K, P.eps);
            narrow(rn);
            /* The maximum of |bf16((t*r)*gain)| without a second meeting of the waves: it lies within a
             * relative 2^-22 of r * max|t*gain| (three roundings), and narrowing is monotonic, so where both
             * ends of a slightly wider interval narrow to the same bf16, that is it.  About one row in 2^12
             * straddles a boundary (and rows where subnormal or infinite products could break the bound are
             * sent the same way, as are sums and gains that are not finite): those take the maximum itself.  Every
             * thread decides on the same values. */
            const float c = rn * U;
            const uint32_t ends = bl_pack2_bf16(c * (1.0f - 0x1p-20f), c * (1.0f + 0x1p-20f));
            if ((ends & 0xFFFFu) == (ends >> 16) && c >= 0x1p-60f && c <= 0x1p120f && rn <= 0x1p40f && U <= 0x1p120f) {
                gamma = __uint_as_float(ends & 0xFFFF0000u);
            } else {
                special = true;
            }
        } else {
            if (SRC != BL_ONE_BF16) narrow(1.0f);
            gamma = row_absmax(std::false_type{});
            special = !(gamma < __builtin_inff());
        }
        if (__builtin_expect(special, 0)) {
            __syncthreads();                                   /* every wave has read fs */
            gamma = row_absmax(std::true_type{});
        }
        const float gg = fmaxf(gamma, 1e-5f);
        const float inv = bl_div_rn(127.0f, gg);
        int part_q = 0;
        auto quantise = [&](auto mode) {
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                const int u = tid + j * nthreads;
                if (u >= units) continue;
                const uint32_t o = bl_quant4<decltype(mode)::value>(
                    __uint_as_float(xb[j].x << 16), __uint_as_float(xb[j].x & 0xFFFF0000u),
                    __uint_as_float(xb[j].y << 16), __uint_as_float(xb[j].y & 0xFFFF0000u), inv);
                *(uint32_t*)(Qs + (u >> 4) * BL_ONE_QSTRIDE + (u & 15) * 4) = o;
                part_q = __builtin_amdgcn_sdot4((int)o, 0x01010101, part_q, false);
                if (first_block && P.q_out) *(uint32_t BL_G*)(P.q_out + u * 4) = o;
            }
        };
        if (__builtin_expect(special, 0)) quantise(bl_mode<BL_Q_ROW>{});
        else quantise(bl_mode<BL_Q_FINITE>{});
        if (tid < 16) *(uint32_t*)(Qs + nchunks * BL_ONE_QSTRIDE + tid * 4) = 0;
        part_q = bl_wave_sum(part_q);
        if (lane == 0) qsum[w] = part_q;
        const float sc = bl_div_rn(gg, 127.0f);
        cf = bt * (P.fixed_scale > 0.0f ? P.fixed_scale : sc);
        if (first_block && tid == 0 && P.scale_out) *bl_g(P.scale_out) = sc;
        __syncthreads();
        if (n0 >= nend) return;                                /* no barrier from here on */
        nq = bl_group_sum<NW>(qsum[lw]);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int chunk = g + G * i;                       /* (beyond the row: the zero chunk) */
            const bl_v4i* src = (const bl_v4i*)(Qs + (chunk < nchunks ? chunk : nchunks) * BL_ONE_QSTRIDE);
#pragma unroll
            for (int d = 0; d < 4; ++d) aq[i][d] = src[d];
        }
    } else {
        if (n0 >= nend) return;
        cf = bt * cf;
#pragma unroll
        for (int i = 0; i < NL; ++i)
#pragma unroll
            for (int d = 0; d < 4; ++d) nq += bl_sum16((uint32_t)aq[i][d][0], (uint32_t)aq[i][d][1], (uint32_t)aq[i][d][2], (uint32_t)aq[i][d][3]);
        nq = bl_lanes_sum<G>(nq);
    }

    /* 3. dot products (bit-pair levels as in bl_gemv.hip) */
    if (P.layout == 0) {
#pragma unroll
        for (int i = 0; i < NL; ++i)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t a0 = (uint32_t)aq[i][d][0], a1 = (uint32_t)aq[i][d][1], a2 = (uint32_t)aq[i][d][2], a3 = (uint32_t)aq[i][d][3];
                bl_transpose4x4(a0, a1, a2, a3);
                aq[i][d] = bl_v4i{(int)a0, (int)a1, (int)a2, (int)a3};
            }
    }
    int mine = 0;
#pragma unroll
    for (int j = 0; j < RW; ++j) {
        int A[4] = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < NL; ++i)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t wd = (uint32_t)p[j][i][d];
                A[0] = __builtin_amdgcn_sdot4((int)(wd & 0x03030303u), aq[i][d][0], A[0], false);
                A[1] = __builtin_amdgcn_sdot4((int)(wd & 0x0C0C0C0Cu), aq[i][d][1], A[1], false);
                A[2] = __builtin_amdgcn_sdot4((int)(wd & 0x30303030u), aq[i][d][2], A[2], false);
                A[3] = __builtin_amdgcn_sdot4((int)((wd >> 2) & 0x30303030u), aq[i][d][3], A[3], false);
            }
        const int pv = A[0] + (A[1] >> 2) + ((A[2] + A[3]) >> 4);
        const int sv = bl_lanes_sum<G>(pv);
        mine = g == j ? sv : mine;
    }
    mine -= nq;
    const int n = n0 + g * R + r;
    if (g < RW && n < nend) {
        if (P.acc) bl_g(P.acc)[n] = mine;
        if (P.y) {
            const float t = (float)mine * cf;
            bl_g(P.y)[n] = residual ? res + t : t;
        }
    }
}

template <int G, int RW, int NL, int UN>
static void launch_one(const bl_one_args& A, int src, bool norm, hipStream_t st) {
    const int blocks = (A.N + A.rows - 1) / A.rows, threads = BL_ONE_WAVES * 64;
    const auto lo = [](uint64_t v) { return (uint32_t)v; };
    const auto hi = [](uint64_t v) { return (uint32_t)(v >> 32); };
    const uint64_t w = (uint64_t)A.packed, x = (uint64_t)A.in0, g = (uint64_t)A.gain, r = (uint64_t)A.residual;
    const uint64_t s = src == BL_ONE_V ? (uint64_t)A.mul_group << 32 | A.mul_hd : (uint64_t)A.in1;
    const bl_v4u where = {lo(w), hi(w), lo(x), hi(x)}, beside = {lo(s), hi(s), lo(g), hi(g)};
    const bl_v4u size = {lo(r), hi(r), (uint32_t)A.N, (uint32_t)A.K};
    const bl_v2u how = {(uint32_t)A.rows | (uint32_t)A.kind << 8 | (uint32_t)A.hd << 16, (uint32_t)A.voff};
    switch (src) {
        case BL_ONE_BF16:
            if (norm) bl_gemv_one<BL_ONE_BF16, G, RW, NL, UN, true><<<blocks, threads, 0, st>>>(where, beside, size, how, A);
            else bl_gemv_one<BL_ONE_BF16, G, RW, NL, UN, false><<<blocks, threads, 0, st>>>(where, beside, size, how, A);
            break;
        case BL_ONE_F32:
            if (norm) bl_gemv_one<BL_ONE_F32, G, RW, NL, UN, true><<<blocks, threads, 0, st>>>(where, beside, size, how, A);
            else bl_gemv_one<BL_ONE_F32, G, RW, NL, UN, false><<<blocks, threads, 0, st>>>(where, beside, size, how, A);
            break;
        case BL_ONE_V:
            if (norm) bl_gemv_one<BL_ONE_V, G, RW, NL, UN, true><<<blocks, threads, 0, st>>>(where, beside, size, how, A);
            else bl_gemv_one<BL_ONE_V, G, RW, NL, UN, false><<<blocks, threads, 0, st>>>(where, beside, size, how, A);
            break;
        case BL_ONE_PAIR:
            if (norm) bl_gemv_one<BL_ONE_PAIR, G, RW, NL, UN, true><<<blocks, threads, 0, st>>>(where, beside, size, how, A);
            else bl_gemv_one<BL_ONE_PAIR, G, RW, NL, UN, false><<<blocks, threads, 0, st>>>(where, beside, size, how, A);
            break;
        default: bl_gemv_one<BL_ONE_INT8, G, RW, NL, UN, false><<<blocks, threads, 0, st>>>(where, beside, size, how, A);
    }
}

/* Which single products of one token this kernel takes; the others go to bl_gemv_rows.  Ratios: time here over
 * time there, both layouts, bf16 and int8 inputs / normalised rows, 22 widths x 16 lengths.
 *   N <= 4096 (one or two row groups to a wave): 0.73 - 1.01 / 0.64 - 0.80: all.
 *   N = 4097 .. 4351 and 8193 .. 8447 (a 17th row to a workgroup, a 257th workgroup): 0.93 - 1.16 / 0.71 - 0.89.
 *   K > 4096 (32 lanes to a row), other N: 0.67 - 1.04 / 0.59 - 0.91: all.
 *   K <= 4096, N = 16385 .. 24576 (257 .. 384 workgroups of 64 rows): 0.88 - 1.45 / 0.60 - 1.09, from K = 1025 on 0.60 - 1.05.
 *   K <= 4096, other N: 0.43 - 0.92 normalised: all; bf16 and int8 up to K = 2048 0.77 - 1.44: none; K = 2049 .. 3072
 *   0.75 - 1.03 (below N = 8193 from K = 2305 on; 1.0 - 1.06 before); K = 3073 .. 4096 0.78 - 1.07 beyond N = 8192,
 *   0.94 - 1.16 below. */
static bool one_token_kernel(int N, int K, bool norm) {
    if (N <= 4096) return true;
    if (!norm && N < 8448 && N % 4096 > 0 && N % 4096 < 256) return false;
    if (K > 4096) return true;
    if (N > 16384 && N <= 24576) return norm && K > 1024;
    if (norm) return true;
    if (N <= 8192) return K > 2304 && K <= 3072;
    return K > 2048;
}

/* One token, one product, K <= 8192: one workgroup per compute unit (256) while the rows last.  Four
 * waves, one per SIMD: what every wave does for itself (reductions, the factor of the normalisation, the
 * reciprocal) is a third of the instructions, and with eight or sixteen waves the SIMDs do it two and
 * four times.  Sixteen lanes to a weight row (K <= 4096) or 32: at K = 2560 a row is 40 loads of 16 bytes, 40 of
 * 48 slots. */
bool bl_gemv_one_launch(const bl_gemv_prob& P, hipStream_t st, bl_status* status) {
    const bl_prod_dev& d = P.prod;
    if (!one_token_kernel(P.N, P.K, P.fused && d.norm)) return false;
    bl_one_args A = {};
    A.packed = P.packed; A.beta = P.beta; A.residual = P.residual; A.acc = P.acc; A.y = P.y;
    A.N = P.N; A.K = P.K; A.layout = P.layout;
    int src = BL_ONE_INT8;
    bool norm = false;
    if (P.fused) {
        A.in0 = d.in0; A.aux_out = d.kind == BL_PROD_RESIDUAL ? d.aux_out : nullptr; A.kind = d.kind;
        A.q_out = P.q_out; A.scale_out = P.scale_out; A.fixed_scale = P.fixed_scale;
        src = d.kind == BL_PROD_BF16 ? BL_ONE_BF16 : d.kind == BL_PROD_RESIDUAL || d.kind == BL_PROD_RELU2_GATE ? BL_ONE_PAIR :
              d.kind == BL_PROD_ATTN_V ? BL_ONE_V : BL_ONE_F32;
        A.in1 = d.kind == BL_PROD_RESIDUAL ? d.in1 : (const float*)d.in0 + P.K;
        if (d.kind == BL_PROD_ATTN_V) {
            A.voff = d.voff; A.hd = d.hd;
            A.mul_hd = (uint32_t)((((uint64_t)1 << 32) + d.hd - 1) / d.hd);
            A.mul_group = d.group == 1 ? 0 : (uint32_t)((((uint64_t)1 << 32) + d.group - 1) / d.group);
        }
        norm = d.norm != 0;
        A.gain = d.gain; A.eps = d.eps;
    } else {
        A.in0 = P.q; A.scale = P.scale;
    }
    A.inv_k = 1.0 / (double)P.K;
    /* rows of a workgroup: up to 16 with one (K <= 4096) or two row groups in a wave's registers, up to 64
     * (32) with four; more rows than that: more workgroups than compute units */
    int rows = P.N > 8 * 256 ? (P.N + 255) / 256 : 8;
    const int most = P.K <= 4096 ? 64 : 32;
    if (rows > most) rows = most;
    A.rows = rows;                                         /* (8 bits, like the kind; a head has at most K = 8192 values) */
    if (rows <= 16) {
        if (P.K <= 3072) launch_one<16, 1, 3, 3>(A, src, norm, st);
        else if (P.K <= 4096) launch_one<16, 1, 4, 4>(A, src, norm, st);
        else if (P.K <= 7168) launch_one<32, 2, 4, 7>(A, src, norm, st);
        else launch_one<32, 2, 4, 8>(A, src, norm, st);
    } else {
        if (P.K <= 3072) launch_one<16, 4, 3, 3>(A, src, norm, st);
        else if (P.K <= 4096) launch_one<16, 4, 4, 4>(A, src, norm, st);
        else if (P.K <= 7168) launch_one<32, 4, 4, 7>(A, src, norm, st);
        else launch_one<32, 4, 4, 8>(A, src, norm, st);
    }
    *status = hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
    return true;
}
