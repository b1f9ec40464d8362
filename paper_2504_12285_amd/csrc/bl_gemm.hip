/* Prefill-side W1.58A8 product (Section 5.1 of the BitNet b1.58 2B4T report):
 * a dense int8 contraction on the CDNA4 matrix cores.  Packed 2-bit weight
 * tiles go HBM -> LDS still packed (a quarter of the int8 bytes), each wave
 * expands the words it needs to int8 in registers with shift+mask behind the
 * v_mfma_i32_32x32x32_i8 in front, and the activations stream through LDS as int8
 * (bl_gemm_pipe.h).  Codes c = Wt + 1 are contracted as they are; the epilogue subtracts
 * rowsum[m] = sum_k q[m][k] (exact int32 identity), then rescales.
 */
#include "bl_device.h"
#include "bl_gemm_pipe.h"
#include "bl_host.h"

#include <atomic>

/* Outputs of the fused producer epilogues (device pointers; see bl_gemm_pipe). */
struct bl_epi_args {
    uint16_t* xb;
    int* absmax;
};

/* Order of the tiles (see bl_gemm_pipe).  Rows of activations per band: at most ~1.5 MB of int8 (measured, medians of six
 * interleaved rounds at M = 2048: +7 % on the 13824-wide shape against bands of all rows, equal on the others).  A rectangle
 * per XCD unless its size means more tiles for the busiest of an XCD's 32 compute units than an even share
 * does: 2140 x 3840 -> 13458 (17 row tiles, bands of 3: two XCDs idle) 148 / 122 us, 1100 x 2560 -> 7000 (70
 * tiles against 62) 36 / 27.5; 777 x 2999 -> 5003 with its quantiser (70 and 60 tiles against 65: three on
 * the busiest unit either way) 28.1 / 30.6 (tiles of 128 x 128 and 64 x 128). */
struct bl_tile_order {
    int gm, band, vgrid;
};
static bl_tile_order tile_order(int tiles_m, int tiles_n, int BM, int K) {
    int gm = 1;
    while (gm < 8 && (int64_t)((tiles_m + gm - 1) / gm) * BM * K > (3 << 19)) gm *= 2;
    int band = (tiles_m + gm - 1) / gm;
    const int rect = band * ((tiles_n + 8 / gm - 1) / (8 / gm)), share = (tiles_m * tiles_n + 7) / 8;
    if ((rect + 31) / 32 <= (share + 31) / 32) return {gm, band, 8 * rect};
    int64_t most = (3 << 19) / ((int64_t)BM * K);
    if (most < 1) most = 1;
    const int bands = (int)((tiles_m + most - 1) / most);
    band = (tiles_m + bands - 1) / bands;
    return {0, band, 8 * share};
}

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

/* The order of the tiles and what an XCD reads: bytes per k of its share, 64 to a row tile, 8 to a column tile; a share in
 * one order is whole lines in the other.  3931 x 4480 -> 256 (62 row tiles and 8 column tiles; row tiles fastest, every XCD reads
 * all activations) 24.5 us, columns fastest 13.1; 2528 x 1877 -> 320 10.7 / 7.7. */
struct bl_ksplit_order {
    bool across;
    int64_t bytes;
};
static bl_ksplit_order ksplit_order(int m, int n) {
    const int64_t tm = (m + 63) / 64, tn = (n + 31) / 32, share = (tm * tn + 7) / 8;
    const int64_t down = (share < tm ? share : tm) * 64 + (share + tm - 1) / tm * 8, over = (share < tn ? share : tn) * 8 + (share + tn - 1) / tn * 64;
    const bool across = over * 2 < down;                       /* (rows first otherwise: 395 x 2176 -> 1600 8.0 us, 8.7 across) */
    return {across, across ? over : down};
}
/* Its time (us), for the tile choice below: rounds of 512 workgroups, and what an XCD reads. */
static float ksplit_us(int m, int n, int k) {
    const int64_t tiles = (int64_t)((m + 63) / 64) * ((n + 31) / 32);
    const float rounds = (float)((tiles + 511) / 512), steps = (float)((k + GP_BK - 1) / GP_BK);
    return 1.81f + rounds * (steps * .091f + 1.83f) + 2.18e-6f * (float)ksplit_order(m, n).bytes * (float)k + 1.31e-6f * (float)m * (float)n;
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
    /* bytes per k that an XCD reads: 64 to a row tile, 8 to a column tile; a share of one order is whole lines of the other */
    const int64_t down = (int64_t)(share < tiles_m ? share : tiles_m) * 64 + (int64_t)((share + tiles_m - 1) / tiles_m) * 8;
    const int64_t over = (int64_t)(share < tiles_n ? share : tiles_n) * 8 + (int64_t)((share + tiles_n - 1) / tiles_n) * 64;
    kern<<<share * 8, 256, lds, st>>>(packed, q, rowsum, beta, scale, m, n, k, tiles_m, tiles, over < down ? tiles_n : 0, residual, acc, y,
                                                 (long long*)bl_clock_stamps());
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}

/* Launch of bl_gemm_pipe: a persistent grid of the workgroups that are resident at once. */
template <int MI, int NI, int WM, int WN, int S, int OCC, int EPI, int LAYOUT>
static bl_status launch_pipe(const uint8_t* packed, const float* beta, const int8_t* q, const float* scale, const int32_t* rowsum,
                             int M, int N, int K, const float* residual, int32_t* acc, float* y, hipStream_t st,
                             bl_epi_args ep = bl_epi_args{nullptr, nullptr}) {
    using G = bl_pipe_geom<MI, NI, WM, WN, S>;
    const auto kern = bl_gemm_pipe<MI, NI, WM, WN, S, OCC, EPI, LAYOUT>;
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
    const bl_tile_order o = tile_order(tiles_m, tiles_n, G::BM, K);
    if (blocks > o.vgrid) blocks = o.vgrid;
    kern<<<blocks, G::THREADS, G::LDS, st>>>(packed, q, rowsum, beta, scale, M, N, K, tiles_m, tiles_n, o.gm ? 3 - __builtin_ctz(o.gm) : -1, o.band, o.vgrid, blocks,
                                             residual, acc, y, ep.xb, ep.absmax, (long long*)bl_clock_stamps(), nullptr, nullptr, nullptr);
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}

/* Table walk (batched decode of a stack, more than 48 tokens): one launch over every tile of 64 x BL_TILE_ROWS of every product
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

/* Tile choice of a plain product: the kernel with the least time by this estimate (us),
 *     fixed + busiest * (steps * (step + lone) + tile) + 2^-20 outputs,
 * busiest = tiles of the busiest of 256 compute units, lone (to `step`) only where no unit has more than one.  Fitted to 200 shapes in
 * both layouts (65 .. 4096 x 300 .. 14000, K 256 .. 7000): the choice takes 1.005 times the time of the best of the six, and
 * .86 of that of the kernels before them (128 x 128 with deferred stores, 64 x 128 with two or four stages, a
 * register-staged 128 x 128; worst 1.12, 4072 x 640 -> 1915).  Where each is the best (us; in brackets the kernels before):
 *   128 x 256, two workgroups to a unit: many tiles (4096 x 2560 -> 13824 117; 128 x 192 122, 128 x 128 129, 64 x 128 151 [149]);
 *   128 x 192, two workgroups: where it fills the units better (2048 x 2560 -> 13824 63.6; 128 x 256 68, 64 x 128 79 [72]);
 *   128 x 192, one workgroup with four stages: at most one tile to a unit (2048 x 6912 -> 2560 37.2; 128 x 256 44.5, 128 x 128 40.6,
 *     64 x 128 42.2 [43.2]);
 *   128 x 128, two workgroups: two tiles to a unit (2048 x 2560 -> 3840 22.3; 128 x 256 25.4, 64 x 128 25.7 [25.2]);
 *   64 x 128, four workgroups: few tokens (512 x 2560 -> 3840 10.4; 128 x 128 12.5 [14.1]);
 *   the k loop split over the waves (bl_gemm_ksplit): fewer tiles than units (512 tiles of 64 x 32 in a round; 128 x 2560 -> 3840
 *     6.6, 64 x 128 8.7). */
struct bl_tile_cost {
    int bm, bn;
    float fixed, step, lone, tile, out;
    float us(int m, int n, int k) const {
        const int64_t tiles = (int64_t)((m + bm - 1) / bm) * ((n + bn - 1) / bn), busiest = (tiles + 255) / 256;
        const float steps = (float)((k + GP_BK - 1) / GP_BK);
        return fixed + (float)busiest * (steps * (step + (busiest == 1 ? lone : 0.0f)) + tile) + out * 1e-6f * (float)m * (float)n;
    }
};
/* the kernel of the least cost: its place in the list */
template <int COUNT>
static int least(const bl_tile_cost (&cost)[COUNT], int m, int n, int k, float* us = nullptr) {
    int best = 0;
    float t = cost[0].us(m, n, k);
    for (int i = 1; i < COUNT; ++i) {
        const float ti = cost[i].us(m, n, k);
        if (ti < t) {
            t = ti;
            best = i;
        }
    }
    if (us) *us = t;
    return best;
}
static constexpr bl_tile_cost plain_cost[5] = {{128, 256, 4.55f, .616f, .093f, .252f, .515f}, {128, 192, 4.05f, .508f, .110f, .317f, .505f},
                                               {128, 192, 2.96f, .564f, 0.0f, 2.01f, .465f}, {128, 128, 4.16f, .351f, .066f, 0.0f, .553f},
                                               {64, 128, 3.70f, .225f, .068f, 0.0f, .492f}};

template <int LAYOUT>
static bl_status launch_plain(const uint8_t* packed, const float* beta, const int8_t* q, const float* scale,
                              const int32_t* rowsum, int m, int n, int k, const float* residual, int32_t* acc, float* y,
                              hipStream_t st) {
    float us;
    const int kernel = least(plain_cost, m, n, k, &us);
    /* (fitted with fp32 output alone; the split k loop has the residual at hand when its sums are ready, and writes two outputs at
     * once: 663 x 781 -> 1088 5.9 us with residual, 64 x 128 tiles 8.0; 436 x 576 -> 2330 with both 6.2 / 6.9) */
    us += residual ? 2.0f : acc && y ? 0.8f : 0.0f;
    if (ksplit_us(m, n, k) < us) return launch_ksplit<LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
    switch (kernel) {
        case 0: return launch_pipe<2, 4, 2, 2, 3, 2, 0, LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
        case 1: return launch_pipe<2, 3, 2, 2, 3, 2, 0, LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
        case 2: return launch_pipe<2, 3, 2, 2, 4, 1, 0, LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
        case 3: return launch_pipe<2, 2, 2, 2, 3, 2, 0, LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
        default: return launch_pipe<2, 1, 1, 4, 3, 4, 0, LAYOUT>(packed, beta, q, scale, rowsum, m, n, k, residual, acc, y, st);
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

/* The tile of a fused epilogue, by the same estimate (gate: tiles of outputs), fitted to 140 shapes; the choice takes 1.003 times
 * the time of the best, .80 (residual) and .88 (gate) of that of the 128 x 128 and 64 x 128 tiles before it.  us [before]:
 *   residual 4096 x 2560 -> 2560 40 [45], 4096 x 6912 -> 2560 88 [93], 1000 x 2560 -> 2560 15.7 [20.1], 128 x 6912 -> 2560 21.2 [26.7];
 *   gate 2560 -> 13824 at 4096 tokens 120 [142], 2048 70 [72.6], 1000 38.5 [48.5], 128 18.2 [19.5].
 * Slower than before: gates of short rows with few tiles (834 x 256 -> 3328 6.7 [6.0], 94 x 1024 -> 6400 9.9 [9.5]). */
static constexpr bl_tile_cost residual_cost[3] = {{128, 256, 0.0f, .450f, .207f, 8.97f, .929f}, {128, 128, 3.26f, .266f, .103f, 3.68f, .988f},
                                                  {64, 128, 3.84f, .193f, .112f, .966f, 1.17f}};
static constexpr bl_tile_cost gate_cost[2] = {{128, 128, 6.24f, .614f, .072f, 0.0f, .756f}, {64, 64, 4.52f, .230f, .056f, 0.0f, .872f}};

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
    if (ep->kind == BL_EPI_RESIDUAL) {
        switch (least(residual_cost, m, n, k)) {
            case 0: return launch_pipe<2, 4, 2, 2, 3, 2, 1, 1>(packed, beta, q, scale, rowsum, m, n, k, ep->residual, acc, ep->y, st, ea);
            case 1: return launch_pipe<2, 2, 2, 2, 3, 2, 1, 1>(packed, beta, q, scale, rowsum, m, n, k, ep->residual, acc, ep->y, st, ea);
            default: return launch_pipe<1, 2, 2, 2, 3, 4, 1, 1>(packed, beta, q, scale, rowsum, m, n, k, ep->residual, acc, ep->y, st, ea);
        }
    }
    if (least(gate_cost, m, n / 2, k) == 0)
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
