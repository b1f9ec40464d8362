/* The one-token stream on the vector unit: the form of bl_stream_m1 for tables that give a workgroup little to do (included by
 * bl_stream.hip, which says when).  Staging is what such a launch waits for, and here it is a copy, not a conversion to 6-bit pieces;
 * and a row of many chunks is spread over up to 64 lanes, where the matrix cores take eight rows of it one part after the other.
 *
 * Inside a product the lanes of a wave hold LP 16-byte loads per row (k chunks g, g + G, .. of the row; G = 1 << lgG lanes
 * per row, 64 / G rows per wave-wide load: a row group).  Offset codes c = Wt + 1, four-wide dot products with the int8 activations,
 * DPP sums over the G lanes, the row sum accounted for once per output.
 * 2-bit form: bit-pair levels isolated by masks, v_dot4_i32_i8 into four accumulators carrying 1, 4, 16, 16.
 * Five per byte: see bl_t5_digits for the byte; two permutes take a byte's number 0..8 as a selector into eight-byte tables, the
 * first and the second digit of four weights each, against k = 20 * word + 4 * i + 0..3.  A selector of 8 replicates the sign of
 * table byte 1, so the tables hold c - 3 (entry 8 is then -1 and byte 1 negative, as it has to be); sum_k (c - 3) q = sum_k c q - 3 sum_k q.
 * LDS image: 2-bit form: per chunk 20 dwords (16 + 4 of padding so that the eight chunks a wave reads together fall on
 * different banks), dword s * 4 + d = the bytes that pair with bit-pair level s of packed word d; five per byte: the int8 row as
 * it is, 20 dwords per chunk and 4 of padding; zeros to the end of the last chunk and one zero chunk behind it for lanes whose
 * load is clamped. */
#pragma once

template <int FORM>
constexpr int bl_dot_stride() { return FORM == BL_FORM_TRIT5 ? 24 : 20; }      /* dwords of a chunk in LDS */

/* Sum over aligned groups of 1 << lgG lanes (8, 16, 32 or 64), result in every lane. */
__device__ __forceinline__ int bl_group_sum_rt(int v, int lgG) {
    v = bl_group_sum<8>(v);
    if (lgG >= 4) v += bl_dpp<BL_DPP_ROW_MIRROR>(v);
    if (lgG >= 5) v += __shfl_xor(v, 16);
    if (lgG >= 6) v += __shfl_xor(v, 32);
    return v;
}

/* Sixteen activations (16-byte group u of the row) into the image. */
template <int FORM>
__device__ __forceinline__ void bl_dot_put(int* __restrict__ Qs, int u, int layout, bl_v4i v) {
    if constexpr (FORM == BL_FORM_TRIT5) {
        *(bl_v4i*)(Qs + (u / 5) * bl_dot_stride<FORM>() + (u % 5) * 4) = v;
    } else {
        uint32_t a0 = (uint32_t)v[0], a1 = (uint32_t)v[1], a2 = (uint32_t)v[2], a3 = (uint32_t)v[3];
        if (layout == 0) bl_transpose4x4(a0, a1, a2, a3);
        int* dst = Qs + (u >> 2) * bl_dot_stride<FORM>() + (u & 3);
        dst[0] = (int)a0;
        dst[4] = (int)a1;
        dst[8] = (int)a2;
        dst[12] = (int)a3;
    }
}

/* Stages the activation row of P: Qs = the image above, misc[0] = sum_k q, misc[1] = token part of the rescale factor (float
 * bits).  Ends with a barrier. */
template <int FORM>
__device__ __forceinline__ void bl_dot_stage(const bl_stream_item& P, int* __restrict__ Qs, int* __restrict__ misc, bool owner) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int groups = P.qgroups;
    float* fs = (float*)(misc + 2);
    int* ssum = misc + 6;
    if constexpr (FORM == BL_FORM_TRIT5) {
        for (int u = groups + tid; u < (P.nchunks + 1) * 5; u += 256) bl_dot_put<FORM>(Qs, u, 0, bl_v4i{0, 0, 0, 0});
    } else {
        if (tid < bl_dot_stride<FORM>()) Qs[P.nchunks * bl_dot_stride<FORM>() + tid] = 0;
    }
    int part = 0;
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
        if (lane == 0) fs[w] = mx;
        __syncthreads();
        const float gamma = bl_max_pos(bl_max_pos(fs[0], fs[1]), bl_max_pos(fs[2], fs[3]));   /* (NaN is the largest) */
        float gg = fmaxf(gamma, 1e-5f);
        const float inv = bl_div_rn(127.0f, gg);
        auto put = [&](int u, uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3) {
            part += bl_sum16(a0, a1, a2, a3);
            const bl_v4i qv = {(int)a0, (int)a1, (int)a2, (int)a3};
            if (owner && P.q_out) *(bl_gv4i*)(P.q_out + u * 16) = qv;
            bl_dot_put<FORM>(Qs, u, P.layout, qv);
        };
        for (int u = tid; u < groups; u += 256) {
            uint32_t a0, a1, a2, a3;
            bl_quant8_words(ld(2 * u), inv, a0, a1);
            bl_quant8_words(ld(2 * u + 1), inv, a2, a3);
            put(u, a0, a1, a2, a3);
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
                    if (lane == 0) fs[w] = v;
                    __syncthreads();
                    return bl_max_pos(bl_max_pos(fs[0], fs[1]), bl_max_pos(fs[2], fs[3]));
                },
                put);
        }
        if (tid == 0) {
            const float sc = bl_div_rn(gg, 127.0f);
            misc[1] = __float_as_int(P.fixed_scale > 0.0f ? P.fixed_scale : sc);
            if (owner && P.scale_out) *(float BL_G*)P.scale_out = sc;
        }
        part = bl_wave_sum(part);
        if (lane == 0) ssum[w] = part;
        __syncthreads();
        if (tid == 0) misc[0] = (ssum[0] + ssum[1]) + (ssum[2] + ssum[3]);
    } else {
        const bl_gv4i* qg = (const bl_gv4i*)P.q;
        for (int u = tid; u < groups; u += 256) bl_dot_put<FORM>(Qs, u, P.layout, qg[u]);
        if (tid == 0) {
            misc[0] = *(const int32_t BL_G*)P.rowsum;
            misc[1] = P.scale ? __float_as_int(*(const float BL_G*)P.scale) : 0;
        }
    }
    __syncthreads();
}

/* One 16-byte load of a lane, p, against its activations at a (LDS); A carries the lane's sums. */
template <int FORM>
__device__ __forceinline__ void bl_dot_load(const bl_v4i p, const int* a, int* A) {
    if constexpr (FORM == BL_FORM_TRIT5) {
        bl_v4i q[5];
#pragma unroll
        for (int t = 0; t < 5; ++t) q[t] = *(const bl_v4i*)(a + t * 4);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t w = (uint32_t)p[d];
            uint32_t e = w & 0x00FF00FFu, o = (w >> 8) & 0x00FF00FFu;
            auto dot = [&](uint32_t dg, int i) { A[0] = __builtin_amdgcn_sdot4((int)dg, q[(5 * d + i) >> 2][(5 * d + i) & 3], A[0], false); };
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                e = (e << 3) + e;
                o = (o << 3) + o;
                const uint32_t t = __builtin_amdgcn_perm(o, e, 0x07030501u);    /* bits 8..15 of the four lanes */
                dot(__builtin_amdgcn_perm(0xFFFFFEFEu, 0xFEFDFDFDu, t), i);     /* t / 3 - 3 */
                dot(__builtin_amdgcn_perm(0xFEFDFFFEu, 0xFDFFFEFDu, t), i + 1); /* t % 3 - 3 */
                e &= 0x00FF00FFu;
                o &= 0x00FF00FFu;
            }
            e = (e << 1) + e;
            o = (o << 1) + o;
            dot(__builtin_amdgcn_perm(o, e, 0x07030501u) + 0xFDFDFDFDu, 4);
        }
    } else {
        bl_v4i q[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) q[s] = *(const bl_v4i*)(a + s * 4);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t w = (uint32_t)p[d];
                const uint32_t lv = s == 0 ? (w & 0x03030303u)
                                  : s == 1 ? (w & 0x0C0C0C0Cu)
                                  : s == 2 ? (w & 0x30303030u)
                                           : ((w >> 2) & 0x30303030u);
                A[s] = __builtin_amdgcn_sdot4((int)lv, q[s][d], A[s], false);
            }
    }
}

/* One product slice [ub, ue) of row groups; the four waves take them round-robin and keep one in flight while another is
 * multiplied.  Every load of the steady loop is unconditional (out-of-range lanes read a clamped, valid address and meet the
 * zero chunk, or are never stored); the residual value of a row travels with the row's weights (without one every lane reads beta). */
template <int FORM, int LP>
__device__ __forceinline__ void bl_dot_slice(const bl_stream_item& P, const int ub, const int ue, int* __restrict__ Qs,
                                              int* __restrict__ misc, const bool restage) {
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = P.N, nchunks = P.nchunks, lgG = P.lgG;
    const int R = 64 >> lgG;
    const int r = lane >> lgG, g = lane & ((1 << lgG) - 1);
    const bl_gv4i* const wbase = (const bl_gv4i*)P.packed;
    int32_t BL_G* const acc_g = (int32_t BL_G*)P.acc;
    float BL_G* const y_g = (float BL_G*)P.y;
    const float BL_G* const res_g = (const float BL_G*)P.residual;
    const float BL_G* const res_base = res_g ? res_g : (const float BL_G*)P.beta;
    int coff[LP], qoff[LP];                              /* clamped k chunk of each load; its LDS image */
#pragma unroll
    for (int i = 0; i < LP; ++i) {
        const int chunk = g + (i << lgG);
        coff[i] = chunk < nchunks ? chunk : nchunks - 1;
        qoff[i] = (chunk < nchunks ? chunk : nchunks) * bl_dot_stride<FORM>();
    }
    auto issue = [&](bl_v4i* p, float& rv, int rg) {
        int n = rg * R + r;
        n = n < N ? n : N - 1;
        const bl_gv4i* wrow = wbase + (int64_t)n * nchunks;
#pragma unroll
        for (int i = 0; i < LP; ++i) p[i] = __builtin_nontemporal_load(wrow + coff[i]);
        rv = res_base[res_g ? n : 0];
    };
    bl_v4i pa[LP], pb[LP];
    float ra, rb;
    int u = ub + w;                                      /* this wave's row group */
    if (u < ue) issue(pa, ra, u);                        /* in flight during the staging */
    if (restage) __syncthreads();                        /* every wave is done with the previous image */
    bl_dot_stage<FORM>(P, Qs, misc, ub == 0);
    if (u >= ue) return;
    const int rs = misc[0];
    float cf = 0.0f;
    if (y_g) cf = *(const float BL_G*)P.beta * __int_as_float(misc[1]);
    auto finish = [&](const bl_v4i* p, const float rv, int rg) {
        int A[4] = {0, 0, 0, 0};
        /* The image does not change inside the loop, so the compiler would hoist these reads out of it and hold them in
         * 16 * LP registers: the address is hidden from it. */
#pragma unroll
        for (int i = 0; i < LP; ++i) {
            int qo = qoff[i];
            asm volatile("" : "+v"(qo));
            bl_dot_load<FORM>(p[i], Qs + qo, A);
        }
        int v = FORM == BL_FORM_TRIT5 ? A[0] : A[0] + (A[1] >> 2) + ((A[2] + A[3]) >> 4);
        v = bl_group_sum_rt(v, lgG);
        const int n = rg * R + r;
        if (g == 0 && n < N) {
            const int val = FORM == BL_FORM_TRIT5 ? v + 2 * rs : v - rs;   /* sum (c - 3) q + 3 sum q - sum q */
            if (acc_g) acc_g[n] = val;
            if (y_g) {
                const float t = (float)val * cf;
                y_g[n] = res_g ? rv + t : t;
            }
        }
    };
    for (;;) {
        if (u + 4 >= ue) { finish(pa, ra, u); break; }
        issue(pb, rb, u + 4);
        finish(pa, ra, u);
        u += 4;
        if (u + 4 >= ue) { finish(pb, rb, u); break; }
        issue(pa, ra, u + 4);
        finish(pb, rb, u);
        u += 4;
    }
}

/* Persistent grid as bl_stream_m1.  Two loop shapes cover every product: five loads per lane and row, and up to four (a
 * product with fewer leaves slots idle). */
template <int FORM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
void bl_stream_dot(const bl_stream_item* __restrict__ items, const int2* __restrict__ wgstart, const int q_ints) {
    extern __shared__ __attribute__((aligned(16))) int lds[];   /* q_ints ints of image + 16 */
    int* Qs = lds;
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
        if (P.lp == 5) bl_dot_slice<FORM, 5>(P, ub, ue, Qs, misc, staged);
        else bl_dot_slice<FORM, 4>(P, ub, ue, Qs, misc, staged);
        staged = true;
    }
}
