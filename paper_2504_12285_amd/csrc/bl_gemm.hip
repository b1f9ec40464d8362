/* Prefill-side W1.58A8 product (Section 5.1 of the BitNet b1.58 2B4T report):
 * a dense int8 contraction on the CDNA4 matrix cores.  Packed 2-bit weight
 * tiles go HBM -> LDS still packed (a quarter of the int8 bytes), each wave
 * expands the words it needs to int8 in registers with shift+mask behind the
 * v_mfma_i32_32x32x32_i8 in front, and the activations stream through LDS as int8
 * (bl_gemm_pipe.h).  Codes c = Wt + 1 are contracted as they are; the epilogue subtracts
 * rowsum[m] = sum_k q[m][k] (exact int32 identity), then rescales.
 */
#include "bl_device.h"
#include "bl_gemm_choice.h"
#include "bl_gemm_pipe.h"
#include "bl_host.h"

#include <atomic>

/* Outputs of the fused producer epilogues (device pointers; see bl_gemm_pipe). */
struct bl_epi_args {
    uint16_t* xb;
    int* absmax;
};

/* ---- few tiles: the k loop split over the waves of a workgroup -------------------------------
 * With few tokens (65 .. a few hundred) a product has fewer 64 x 128 tiles than the chip has compute
 * units, and its time is one tile's serial chain of k steps (about 600 clocks each, of which the matrix
 * cores work 256).  Here a workgroup owns a 64 x 32 tile and each of its four waves takes every fourth
 * k step of it alone: four times the workgroups, a quarter of the chain, and no barrier inside the loop (a
 * wave's stages in LDS are its own; it waits for its own loads).  The four partial tiles meet in LDS and
 * each wave finishes a quarter of the rows.  The weights cost the same bytes as before, the activations
 * are fetched by four times as many workgroups, from the L2.
 * Same LDS layout, swizzles, k mapping and order of bits as bl_gemm_pipe (one wave: pieces of
 * eight activation rows and one of 32 weight rows).
 * Measured (us, 64 x 128 tiles of bl_gemm_pipe / this kernel): 40 tiles 128 x 6912 -> 2560 19.8 / 11.2, 80 tiles 256 x 2560 ->
 * 2560 10.0 / 8.3, 104 tiles 800 x 7000 -> 1024 20.5 / 17.1, 160 tiles 512 x 2560 -> 2560 10.4 / 12.9: there the tiles fill the chip. */
#define KS_STAGE (64 * GP_BK + 32 * GP_BK / 4)

template <int LAYOUT>
__global__ __launch_bounds__(256, 2) void bl_gemm_ksplit(const uint8_t* __restrict__ packed, const int8_t* __restrict__ q,
                                                         const int32_t* __restrict__ rowsum, const float* __restrict__ beta,
                                                         const float* __restrict__ scale, int M, int N, int K, int tiles_m,
                                                         int tiles, int across, const float* __restrict__ residual,
                                                         int32_t* __restrict__ acc, float* __restrict__ y,
                                                         long long* __restrict__ stamps) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];      /* [wave][stage] */
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    /* workgroup L runs on XCD L % 8: each XCD takes one eighth of the tiles, row tiles fastest or (across: the tiles across N)
     * column tiles fastest, whichever makes an XCD read less */
    const int share = (tiles + 7) >> 3, at = ((int)blockIdx.x & 7) * share + ((int)blockIdx.x >> 3);
    if (((int)blockIdx.x >> 3) >= share || at >= tiles) return;         /* the whole workgroup (never workgroup 0) */
    const bool stamp = stamps != nullptr && blockIdx.x == 0;            /* measurement hook, as in bl_gemm_pipe */
    long long c_start = 0, w_start = 0;
    if (stamp) {
        c_start = clock64();
        w_start = wall_clock64();
    }
    const int along = across ? across : tiles_m, major = at / along, minor = at - major * along;
    const int m0 = (across ? major : minor) * 64, n0 = (across ? minor : major) * 32;
    const int steps = (K + GP_BK - 1) / GP_BK;
    const bool half = (K & 64) != 0;

    /* what the rows this wave finishes need: rows (w >> 1) * 32 + (v >> 2) * 8 + h * 4 + (v & 3), v = 8 (w & 1) .. + 7 */
    int rs[8];
    float sc[8], rr[8];
    const int n = n0 + l32;
    const float bt = y ? *beta : 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int v = (w & 1) * 8 + i;
        int m = m0 + (w >> 1) * 32 + (v >> 2) * 8 + h * 4 + (v & 3);
        m = m < M ? m : M - 1;
        rs[i] = rowsum[m];
        sc[i] = y ? scale[m] : 0.0f;
        rr[i] = y && residual ? residual[(int64_t)m * N + (n < N ? n : N - 1)] : 0.0f;
    }

    const uint8_t* asrc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int row = j * 8 + (lane >> 3), u = (lane & 7) ^ ((row >> 1) & 7);
        const int m = m0 + row < M ? m0 + row : M - 1;
        asrc[j] = (const uint8_t*)q + (int64_t)m * K + u * 16;
    }
    const int wrow = n0 + (lane >> 1) < N ? n0 + (lane >> 1) : N - 1, wu = (lane & 1) ^ ((lane >> 4) & 1);
    const uint8_t* const wsrc = packed + (int64_t)wrow * (K / 4) + wu * 16;
    uint8_t* const base = smem + w * 2 * KS_STAGE;
    auto issue = [&](int kk, int buf) {
        uint8_t* st = base + buf * KS_STAGE;
        const bool last = half && kk == steps - 1;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int back = last ? (((lane >> 2) ^ j) & 1) * 64 : 0;   /* units of the second half: from the first */
            __builtin_amdgcn_global_load_lds((bl_gptr)(asrc[j] + ((int64_t)kk * GP_BK - back)), (bl_lptr)(st + j * 1024), 16, 0, 0);
        }
        __builtin_amdgcn_global_load_lds((bl_gptr)(wsrc + ((int64_t)kk * (GP_BK / 4) - (last ? wu * 16 : 0))),
                                         (bl_lptr)(st + 64 * GP_BK), 16, 0, 0);
    };
    const int a_off = l32 * GP_BK, a_swz = (l32 >> 1) & 7;
    const int w_off = 64 * GP_BK + (l32 * 2 + (h ^ ((l32 >> 3) & 1))) * 16;

    bl_v16i C[2];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int v = 0; v < 16; ++v) C[mi][v] = 0;
    int buf = 0;
    if (w < steps) issue(w, 0);
    for (int kk = w; kk < steps; kk += 4) {
        /* the other buffer's reads (the step before) have been performed before loads overwrite it */
        BL_WAIT_LGKM0();
        asm volatile("" ::: "memory");
        if (kk + 4 < steps) {
            issue(kk + 4, buf ^ 1);
            BL_WAIT_VM(9);                                              /* all but the nine just issued */
        } else {
            BL_WAIT_VM(0);
        }
        asm volatile("" ::: "memory");
        const uint8_t* st = base + buf * KS_STAGE;
        bl_v4i wq = *(const bl_v4i*)(st + w_off), a[4][2];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) a[ks][mi] = *(const bl_v4i*)(st + a_off + mi * 32 * GP_BK + (((4 * h + ks) ^ a_swz) * 16));
        __builtin_amdgcn_sched_barrier(0);                              /* one wait for the step, not one per read */
        if (half && kk == steps - 1 && h == 1) wq = bl_v4i{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const bl_v4i bop = bl_unpack16(LAYOUT == 0 ? bl_word_to_k16((uint32_t)wq[ks]) : (uint32_t)wq[ks]);
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) C[mi] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks][mi], bop, C[mi], 0, 0, 0);
        }
        buf ^= 1;
    }
    bl_mfma_fence();
    /* the partial tiles meet (a wave's part lies in its own stages, which it has read) */
    BL_WAIT_LGKM0();
    asm volatile("" ::: "memory");
    int* const part = (int*)base;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int v = 0; v < 16; ++v) part[(mi * 16 + v) * 64 + lane] = C[mi][v];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int v = (w & 1) * 8 + i, m = m0 + (w >> 1) * 32 + (v >> 2) * 8 + h * 4 + (v & 3);
        int sum = -rs[i];
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) sum += ((const int*)(smem + ww * 2 * KS_STAGE))[((w >> 1) * 16 + v) * 64 + lane];
        if (m < M && n < N) {
            if (acc) acc[(int64_t)m * N + n] = sum;
            if (y) {
                const float t = (float)sum * (bt * sc[i]);
                y[(int64_t)m * N + n] = residual ? rr[i] + t : t;
            }
        }
    }
    if (stamp && threadIdx.x == 0) {
        stamps[0] = clock64() - c_start;
        stamps[1] = wall_clock64() - w_start;
    }
}

template <int LAYOUT>
static bl_status launch_ksplit(const uint8_t* packed, const float* beta, const int8_t* q, const float* scale,
                               const int32_t* rowsum, int m, int n, int k, const float* residual, int32_t* acc, float* y,
                               hipStream_t st) {
    constexpr int lds = 8 * KS_STAGE;
    auto kern = bl_gemm_ksplit<LAYOUT>;
    static std::atomic<bool> attr_set;
    if (!attr_set.load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess) return BL_ERR_HIP;
        attr_set.store(true, std::memory_order_release);
    }
    const int tiles_m = (m + 63) / 64, tiles_n = (n + 31) / 32, tiles = tiles_m * tiles_n, share = (tiles + 7) / 8;
    kern<<<share * 8, 256, lds, st>>>(packed, q, rowsum, beta, scale, m, n, k, tiles_m, tiles, bl_ksplit_order_of(m, n).across ? tiles_n : 0, residual, acc, y,
                                                 (long long*)bl_clock_stamps());
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}

/* Launch of bl_gemm_pipe: a persistent grid of the workgroups that are resident at once. */
template <int MI, int NI, int WM, int WN, int S, int OCC, int EPI, int LAYOUT, bool ODD = false>
static bl_status launch_pipe(const uint8_t* packed, const float* beta, const int8_t* q, const float* scale, const int32_t* rowsum,
                             int M, int N, int K, const float* residual, int32_t* acc, float* y, hipStream_t st,
                             bl_epi_args ep = bl_epi_args{nullptr, nullptr}) {
    using G = bl_pipe_geom<MI, NI, WM, WN, S>;
    const auto kern = bl_gemm_pipe<MI, NI, WM, WN, S, OCC, EPI, LAYOUT, false, ODD>;
    static std::atomic<int> cached{0};
    int blocks = cached.load(std::memory_order_acquire);
    if (blocks == 0) {
        int dev = 0, cus = 0, per_cu = 0;
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kern, G::THREADS, G::LDS) != hipSuccess ||
            cus < 1 || per_cu < 1)
            return BL_ERR_HIP;
        blocks = cus * per_cu < 8 ? 8 : cus * per_cu / 8 * 8;      /* (a multiple of 8 keeps a workgroup on its XCD's share) */
        cached.store(blocks, std::memory_order_release);
    }
    const int tiles_m = (M + G::BM - 1) / G::BM, out = EPI == 2 ? N / 2 : N, cover = EPI == 2 ? G::BN / 2 : G::BN;
    const int tiles_n = (out + cover - 1) / cover;
    if ((int64_t)tiles_m * tiles_n > ((int64_t)1 << 28)) return BL_ERR_SHAPE;
    const bl_tile_order o = bl_tile_order_of(tiles_m, tiles_n, G::BM, K);
    if (blocks > o.vgrid) blocks = o.vgrid;
    kern<<<blocks, G::THREADS, G::LDS, st>>>(packed, q, rowsum, beta, scale, M, N, K, tiles_m, tiles_n, o.gm ? 3 - __builtin_ctz(o.gm) : -1, o.band, o.vgrid, blocks,
                                             residual, acc, y, ep.xb, ep.absmax, (long long*)bl_clock_stamps(), nullptr, nullptr, nullptr);
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}

/* Table walk (batched decode of a stack, more than 32 tokens, see mb_tile_route): one launch over every tile of 64 x BL_TILE_ROWS of every product
 * (see bl_gemm_pipe); M <= 64 tokens, the same for every product; the host balances the k steps over the workgroups.  Thirty
 * 2560 / 6912 layers at 64 tokens 182 us (64 x 128 tiles with two stages, four workgroups to a unit: 220; this kernel with tiles of
 * 64 x 128 206, x 384 189, x 512 235; weights not kept in the caches 323: a line holds four k steps of a row).
 * bl_gemm_table_blocks: the persistent grid (resident workgroups), 0 on error. */
static std::atomic<int> g_table_blocks{0};

int bl_gemm_table_blocks(void) {
    int blocks = g_table_blocks.load(std::memory_order_acquire);
    if (blocks > 0) return blocks;
    const auto kern = bl_gemm_pipe<2, 2, 1, 4, 4, 2, 0, 1, true>;
    using G = bl_pipe_geom<2, 2, 1, 4, 4>;
    static_assert(G::BM == BL_STACK_MAX_TOKENS && G::BN == BL_TILE_ROWS, "");
    int dev = 0, cus = 0, per_cu = 0;
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kern, G::THREADS, G::LDS) != hipSuccess ||
        cus < 1 || per_cu < 1)
        return 0;
    blocks = cus * per_cu;
    g_table_blocks.store(blocks, std::memory_order_release);
    return blocks;
}

bl_status bl_gemm_table_launch(const bl_tile_item* items, int M, int blocks, const int* wg_start, const int* tile_list, bl_stream s) {
    if (g_table_blocks.load(std::memory_order_acquire) == 0) return BL_ERR_VALUE;   /* no table was built in this process */
    using G = bl_pipe_geom<2, 2, 1, 4, 4>;
    bl_gemm_pipe<2, 2, 1, 4, 4, 2, 0, 1, true><<<blocks, G::THREADS, G::LDS, (hipStream_t)s>>>(
        nullptr, nullptr, nullptr, nullptr, nullptr, M, 0, GP_BK, 1, 0, 0, 1, 0, 1, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
        items, wg_start, tile_list);
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}

/* rowsum[m] = sum_k q[m][k]; one wave per row. */
__global__ __launch_bounds__(256) void bl_rowsum_kernel(const int8_t* __restrict__ q, int M, int K,
                                                         int32_t* __restrict__ rowsum) {
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (m >= M) return;
    const uint4* row = (const uint4*)(q + (int64_t)m * K);
    int s = 0;
    for (int i = lane; i < K / 16; i += 64) {
        const uint4 v = row[i];
        s = __builtin_amdgcn_sdot4((int)v.x, 0x01010101, s, false);
        s = __builtin_amdgcn_sdot4((int)v.y, 0x01010101, s, false);
        s = __builtin_amdgcn_sdot4((int)v.z, 0x01010101, s, false);
        s = __builtin_amdgcn_sdot4((int)v.w, 0x01010101, s, false);
    }
    s = bl_wave_sum(s);
    if (lane == 0) rowsum[m] = s;
}

template <int LAYOUT>
static bl_status launch_plain(const uint8_t* packed, const float* beta, const int8_t* q, const float* scale,
                              const int32_t* rowsum, int m, int n, int k, const float* residual, int32_t* acc, float* y,
                              hipStream_t st) {
    switch (bl_plain_kernel(m, n, k, residual != nullptr, acc != nullptr, y != nullptr)) {
        case 0: return launch_pipe<2, 4, 2, 2, 3, 2, 0, LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
        case 1: return launch_pipe<2, 3, 2, 2, 3, 2, 0, LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
        case 2: return launch_pipe<2, 3, 2, 2, 4, 1, 0, LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
        case 3: return launch_pipe<2, 2, 2, 2, 3, 2, 0, LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
        case 4: return launch_pipe<2, 1, 1, 4, 3, 4, 0, LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
        default: return launch_ksplit<LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
    }
}

/* Arguments already validated by the public entry points. */
bl_status bl_gemm_dispatch(const uint8_t* packed, const float* beta, int layout, const int8_t* q,
                           const float* scale, const int32_t* rowsum, int64_t M, int64_t N, int64_t K,
                           const float* residual, int32_t* acc, float* y, void* workspace, hipStream_t st) {
    if (!rowsum) {
        if (!workspace) return BL_ERR_WORKSPACE;
        if (!bl_aligned(workspace, 4)) return BL_ERR_ALIGN;
        int32_t* rs = (int32_t*)workspace;
        bl_rowsum_kernel<<<(unsigned)((M + 3) / 4), 256, 0, st>>>(q, (int)M, (int)K, rs);
        rowsum = rs;
    }
    const int m = (int)M, n = (int)N, k = (int)K;              /* k: a multiple of 64 */
    if (layout == 1) return launch_plain<1>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
    return launch_plain<0>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
}

extern "C" bl_status bl_gemm_w158a8_res(const uint8_t* packed, const float* beta, int layout, const int8_t* q,
                                        const float* scale, const int32_t* rowsum, int64_t M, int64_t N, int64_t K,
                                        const float* residual, int32_t* acc, float* y, void* workspace,
                                        bl_stream s) {
    if (!packed || !beta || !q) return BL_ERR_NULL;
    if (!acc && !y) return BL_ERR_NULL;
    if (y && !scale) return BL_ERR_NULL;
    if (M < 1 || M > BL_MAX_DIM || !bl_shape_ok(N, K)) return BL_ERR_SHAPE;
    if (layout != BL_LAYOUT_ROWMAJOR && layout != BL_LAYOUT_K16) return BL_ERR_LAYOUT;
    if (!bl_aligned(packed, 16) || !bl_aligned(q, 16) || !bl_aligned(acc, 4) || !bl_aligned(y, 4) ||
        !bl_aligned(scale, 4) || !bl_aligned(beta, 4) || !bl_aligned(rowsum, 4) || !bl_aligned(residual, 4))
        return BL_ERR_ALIGN;
    return bl_gemm_dispatch(packed, beta, layout, q, scale, rowsum, M, N, bl_kpad(K), residual, acc, y, workspace,
                            (hipStream_t)s);
}

extern "C" bl_status bl_gemm_w158a8(const uint8_t* packed, const float* beta, int layout, const int8_t* q,
                                    const float* scale, const int32_t* rowsum, int64_t M, int64_t N, int64_t K,
                                    int32_t* acc, float* y, void* workspace, bl_stream s) {
    return bl_gemm_w158a8_res(packed, beta, layout, q, scale, rowsum, M, N, K, nullptr, acc, y, workspace, s);
}

/* Prefill product with a fused producer epilogue (see bl_gemm_pipe, EPI = 1 and 2). */
extern "C" bl_status bl_gemm_w158a8_fused(const uint8_t* packed, const float* beta, int layout, const int8_t* q,
                                          const float* scale, const int32_t* rowsum, int64_t M, int64_t N, int64_t K,
                                          const bl_gemm_epilogue* ep, int32_t* acc, bl_stream s) {
    if (!packed || !beta || !q || !scale || !rowsum || !ep) return BL_ERR_NULL;
    if (!ep->x_bf16 || !ep->absmax) return BL_ERR_NULL;
    if (ep->kind != BL_EPI_RESIDUAL && ep->kind != BL_EPI_RELU2_GATE) return BL_ERR_VALUE;
    if (ep->kind == BL_EPI_RESIDUAL && !ep->residual) return BL_ERR_NULL;
    if (M < 1 || M > BL_MAX_DIM || !bl_shape_ok(N, K) || K % GP_BK != 0 || N % 4 != 0) return BL_ERR_SHAPE;
    if (ep->kind == BL_EPI_RELU2_GATE && N % 128 != 0) return BL_ERR_SHAPE;   /* N/2 gate columns in tiles of 64 */
    if (layout != BL_LAYOUT_K16) return BL_ERR_LAYOUT;
    if (!bl_aligned(packed, 16) || !bl_aligned(q, 16) || !bl_aligned(acc, 4) || !bl_aligned(ep->y, 4) ||
        !bl_aligned(scale, 4) || !bl_aligned(beta, 4) || !bl_aligned(rowsum, 4) || !bl_aligned(ep->residual, 4) ||
        !bl_aligned(ep->x_bf16, 2) || !bl_aligned(ep->absmax, 4))
        return BL_ERR_ALIGN;
    const bl_epi_args ea = {ep->x_bf16, (int*)ep->absmax};
    hipStream_t st = (hipStream_t)s;
    const int m = (int)M, n = (int)N, k = (int)K;
    if (!bl_aligned(ep->x_bf16, 4)) {                          /* (rare: one tile, the smallest, for every size) */
        if (ep->kind == BL_EPI_RESIDUAL)
            return launch_pipe<1, 2, 2, 2, 3, 4, 1, 1, true>(packed, beta, q, scale, rowsum, m, n, k, ep->residual, acc, ep->y, st, ea);
        return launch_pipe<1, 2, 2, 2, 3, 4, 2, 1, true>(packed, beta, q, scale, rowsum, m, n, k, nullptr, acc, ep->y, st, ea);
    }
    if (ep->kind == BL_EPI_RESIDUAL) {
        switch (bl_residual_kernel(m, n, k)) {
            case 0: return launch_pipe<2, 4, 2, 2, 3, 2, 1, 1>(packed, beta, q, scale, rowsum, m, n, k, ep->residual, acc, ep->y, st, ea);
            case 1: return launch_pipe<2, 2, 2, 2, 3, 2, 1, 1>(packed, beta, q, scale, rowsum, m, n, k, ep->residual, acc, ep->y, st, ea);
            default: return launch_pipe<1, 2, 2, 2, 3, 4, 1, 1>(packed, beta, q, scale, rowsum, m, n, k, ep->residual, acc, ep->y, st, ea);
        }
    }
    if (bl_gate_kernel(m, n, k) == 0)
        return launch_pipe<2, 4, 2, 2, 3, 2, 2, 1>(packed, beta, q, scale, rowsum, m, n, k, nullptr, acc, ep->y, st, ea);
    return launch_pipe<1, 2, 2, 2, 3, 4, 2, 1>(packed, beta, q, scale, rowsum, m, n, k, nullptr, acc, ep->y, st, ea);
}

/* ---- entry point that allocates nothing ---------------------------------------------------
 * bl_gemm_w158a8 needs device scratch for the row sums sum_k q[m][k] when the caller brings
 * none.  Here that scratch is a static device array: every GPU the library runs on holds its
 * own copy, at its own address, until the process ends.  In host code the array's name is only
 * a stand-in: the device address comes from hipGetSymbolAddress, once per device, and that
 * pointer is what the kernels receive. */
#define BL_NOALLOC_MAX_DEVICES 64
static __device__ __align__(256) int32_t scratch[BL_NOALLOC_MAX_M];
static std::atomic<int32_t*> bl_scratch_ptr[BL_NOALLOC_MAX_DEVICES];

static bl_status bl_scratch_for_current_device(int32_t** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= BL_NOALLOC_MAX_DEVICES) return BL_ERR_HIP;
    int32_t* p = bl_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        /* two threads racing here both obtain the same address: the symbol has one copy per device */
        void* sym = nullptr;
        if (hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)) != hipSuccess || !sym) return BL_ERR_HIP;
        p = (int32_t*)sym;
        bl_scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return BL_OK;
}

extern "C" bl_status bl_gemm_w158a8_noalloc(const uint8_t* packed, const float* beta, int layout, const int8_t* q,
                                            const float* scale, int64_t M, int64_t N, int64_t K, int32_t* acc,
                                            float* y, bl_stream s) {
    if (!packed || !beta || !q) return BL_ERR_NULL;
    if (!acc && !y) return BL_ERR_NULL;
    if (y && !scale) return BL_ERR_NULL;
    if (M < 1 || M > BL_NOALLOC_MAX_M || !bl_shape_ok(N, K)) return BL_ERR_SHAPE;
    if (layout != BL_LAYOUT_ROWMAJOR && layout != BL_LAYOUT_K16) return BL_ERR_LAYOUT;
    if (!bl_aligned(packed, 16) || !bl_aligned(q, 16) || !bl_aligned(acc, 4) || !bl_aligned(y, 4) ||
        !bl_aligned(scale, 4) || !bl_aligned(beta, 4))
        return BL_ERR_ALIGN;
    int32_t* rs = nullptr;
    const bl_status st = bl_scratch_for_current_device(&rs);
    if (st != BL_OK) return st;
    /* the row-sum kernel overwrites entries 0..M-1 and nothing reads beyond them, so what an
     * earlier (larger) call left behind needs no clearing */
    return bl_gemm_dispatch(packed, beta, layout, q, scale, nullptr, M, N, bl_kpad(K), nullptr, acc, y, rs, (hipStream_t)s);
}
