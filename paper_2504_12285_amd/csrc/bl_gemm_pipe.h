/* The pipelined tile kernel of the prefill product (included by bl_gemm.hip).
 *
 * A workgroup of four waves owns a tile of BM tokens x BN weight rows; k step 128; S stages in LDS filled by direct
 * global -> LDS loads.  One k step of a wave is 4 * MI * NI MFMAs in a fixed order, and everything else a step needs is
 * placed behind single MFMAs, so that the matrix core always has the next one:
 *   - the codes of the next 32 weight rows are opened (bl_unpack16, 7 instructions) behind the MFMAs of the ones before;
 *   - the activations of sub-step ks + 1 are read from LDS behind the first MFMAs of sub-step ks;
 *   - in front of the last sub-step the wave waits for the NEXT stage and passes the step's one barrier, and the last
 *     sub-step's MFMAs cover the reads of that stage's codes and first activations;
 *   - behind the barrier the loads of stage t + S - 1 are issued (its buffer was read last a step ago).
 * The k steps of a workgroup's tiles are one sequence: the loads run S - 1 steps ahead of the matrix cores across tile
 * borders, the row terms (row sums, scales) of a tile travel with its first stage, and behind the last tile the loads go
 * on with an empty range, so that every wait is a constant.
 * Loads go through buffer descriptors: a lane's offset inside a tile never changes, a tile is a scalar base, a k step a
 * scalar offset, and rows past the end of a matrix are out of range (zeros) without a clamp.
 *
 * What bounds it: a compute unit takes 59 B/clk of direct loads (24 KB in 416 clocks, LDS reads beside them for nothing) and its
 * matrix cores 32 clocks for four 32x32x32.  A 128 x 256 tile in 2 x 2 waves of 64 x 128 needs 24 KB of loads and 48 KB of LDS reads
 * for 1024 clocks of MFMA, 128 x 128 in waves of 64 x 64 20 KB and 40 KB for 512: the wide tile is what lets the matrix
 * cores run, and the fixed order is what lets two waves per SIMD (its registers) be enough.  Without output stores it reaches
 * 2.9 POP/s (8192 x 4096 -> 8192 at 1.73 GHz: the power management; the bare MFMA loop reaches 3.4 - 3.6), the
 * kernel of 128 x 128 tiles before it 2.3.  One wave per SIMD issues an MFMA every 41 clocks (two: 35), which is all that a lone
 * 128 x 192 tile loses in its loop (0.51 us a step, without loads, reads and unpacking 0.50); eight waves on the same tile gain nothing.
 *
 * LDS stage = A part (BM rows x 128 int8, 16-byte units XOR-swizzled by (row/2)%8) + W part (BN rows x 32 packed bytes =
 * two units, swapped by row/8%2): sixteen consecutive lanes of a ds_read_b128 fall on sixteen different 16-byte bank
 * groups.  A direct load writes 64 consecutive units, so the swizzle is applied to the global address.
 * k mapping inside a step: MFMA sub-step ks, lane half h  <->  the 16 k of packed word 4h+ks.
 *
 * K a multiple of 64.  With an odd multiple the last step takes the last 128 columns, whose first 64 have
 * been multiplied: lane half 0 (the first unit of a weight row) gets zeros for codes.  (K = 64: one step, lane half 1 gets
 * the zeros and loads the next row, or nothing behind the last.)
 * LAYOUT 0: the activations' bytes are transposed 4 x 4 in registers (weight i of a word lies at bits 2i, so that
 * (word >> 2s) & 0x03030303 holds the codes of k = s, 4 + s, 8 + s, 12 + s): 8 instructions per 16 activations, which NI
 * MFMAs share, against 12 per word shared by MI (one block of 32 rows per wave: the words are turned, bl_word_to_k16).
 *
 * EPI: 0 = int32 and/or fp32 outputs, optional residual; 1 = "residual": t = residual + product as fp32 (y, optional) and
 * bf16 (xb), the row maximum of |bf16(t)| folded into absmax; 2 = "squared-ReLU gate": a wave's NI blocks of 32 weight
 * rows are NI/2 blocks of gate rows and the NI/2 matching blocks of up rows (n and N/2 + n), t = (relu(g)*relu(g))*u.
 * ODD: an xb that starts at an odd multiple of two bytes, stored value by value (a dword store has to be aligned).
 *
 * TABLE: the tiles of a whole table of products of at most BM tokens (device arrays: items; workgroup b takes tile_list[wg_start[b] ..
 * wg_start[b+1]), an entry = product << BL_TILE_BITS | block of BN weight rows): the batched decode of a stack of BitLinears
 * in one launch whose weights are read once.  K, N and the pointers are then those of the product in hand; rows are whole
 * k steps, layout 1, plain epilogue. */
#pragma once
#include "bl_device.h"
#include "bl_gemm_choice.h"
#include "bl_host.h"

#include <type_traits>

template <int MI, int NI, int WM, int WN, int S>
struct bl_pipe_geom {
    static constexpr int BM = WM * MI * 32, BN = WN * NI * 32, THREADS = WM * WN * 64;
    static constexpr int A_BYTES = BM * GP_BK, W_BYTES = BN * GP_BK / 4, STAGE = A_BYTES + W_BYTES;
    static constexpr int SETS = S + 1;                      /* of row terms: the tile in its epilogue and those that the loads may have reached */
    static constexpr int LDS = S * STAGE + SETS * (BM * 8 + WM * WN * 16);
};

template <int MI, int NI, int WM, int WN, int S, int OCC, int EPI, int LAYOUT, bool TABLE = false, bool ODD = false>
__global__ __launch_bounds__(WM * WN * 64, OCC) void bl_gemm_pipe(const uint8_t* __restrict__ packed, const int8_t* __restrict__ q,
                                                                  const int32_t* __restrict__ rowsum, const float* __restrict__ beta,
                                                                  const float* __restrict__ scale, int M, int N, int K, int tiles_m,
                                                                  int tiles_n, int gs, int band, int vgrid, int grid,
                                                                  const float* __restrict__ residual, int32_t* __restrict__ acc,
                                                                  float* __restrict__ y, uint16_t* __restrict__ xb,
                                                                  int* __restrict__ absmax, long long* __restrict__ stamps,
                                                                  const bl_tile_item* __restrict__ items, const int* __restrict__ wg_start,
                                                                  const int* __restrict__ tile_list) {
#if defined(__HIP_DEVICE_COMPILE__)   /* (the host has no type for a buffer descriptor) */
    using G = bl_pipe_geom<MI, NI, WM, WN, S>;
    constexpr int SETS = G::SETS, NW = WM * WN, BM = G::BM, BN = G::BN, STAGE = G::STAGE, AB = G::A_BYTES;
    constexpr int AL = AB / 1024 / NW, WP = G::W_BYTES / 1024, WL = (WP + NW - 1) / NW, LOADS = AL + WL;
    constexpr int SL = MI * NI;                              /* MFMAs of a sub-step */
    static_assert(AB % (1024 * NW) == 0 && S >= 3 && (S - 1) * LOADS < 64, "whole loads per wave; vmcnt is a 6-bit count");
    static_assert(EPI != 2 || NI % 2 == 0, "gate and up blocks in pairs");
    constexpr bool TURN_A = LAYOUT == 0 && NI > 1, TURN_W = LAYOUT == 0 && NI == 1;
    typedef __attribute__((address_space(3))) void* lds_p;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    int* const terms = (int*)(smem + S * STAGE);             /* SETS sets of BM row sums and BM scales */
    int* const ahead = terms + SETS * 2 * BM;                /* each wave's tiles that the loads have reached: SETS of four ints (tm, tn; TABLE: steps) */
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int wm0 = (wave / WN) * (MI * 32), wn0 = (wave % WN) * (NI * 32);
    static_assert(!TABLE || (EPI == 0 && LAYOUT == 1 && WM == 1), "one block of rows, plain epilogue");
    /* of the product whose tile the loads have reached (one product: of all) */
    int lN = N, lK = K;
    const uint8_t* lpacked = packed;
    const int8_t* lq = q;
    const int32_t* lrowsum = rowsum;
    const float* lscale = scale;
    int steps = (K + GP_BK - 1) / GP_BK, lsteps = steps;
    /* at the end of step `zstep` of a tile the codes at hand are those of a half step */
    const int zstep = TABLE || K % GP_BK == 0 ? -1 : max(steps - 2, 0), dead = !TABLE && K < GP_BK ? 1 : 0;
    float bt = !TABLE && (EPI != 0 || y != nullptr) ? *beta : 0.0f;

    /* XCD-aware tile order: workgroup L runs on XCD L%8.  The row tiles are cut into bands so narrow that
     * a band's activation panel stays in an XCD's 4 MB L2 while its weight tiles stream through, row tiles
     * fastest.  Either a rectangle per XCD (8 >> gs bands x 1 << gs column blocks), or (gs < 0) the tiles are
     * numbered band by band and each XCD takes one eighth of the sequence; the host chooses.  The grid is persistent:
     * a workgroup takes virtual blocks vb = blockIdx.x, + grid, .. (grid is a multiple of 8). */
    auto tile_of = [&](int vb, int& tm, int& tn) {
        const int xcd = vb & 7, idx = vb >> 3;
        if (gs >= 0) {
            const int cols = (tiles_n + (1 << gs) - 1) >> gs, col = idx / band;
            tm = (xcd >> gs) * band + (idx - col * band);
            tn = (xcd & ((1 << gs) - 1)) * cols + col;
            return col < cols && tm < tiles_m && tn < tiles_n;
        }
        const int tiles = tiles_m * tiles_n, share = (tiles + 7) >> 3, band_tiles = band * tiles_n;
        const int at = xcd * share + idx;
        if (idx >= share || at >= tiles) return false;
        const int b = at / band_tiles, in = at - b * band_tiles;
        const int rows = min(band, tiles_m - b * band);
        tn = in / rows;
        tm = b * band + (in - tn * rows);
        return true;
    };
    int vend = vgrid;
    if constexpr (TABLE) vend = wg_start[blockIdx.x + 1];
    auto next_tile = [&](int vb, int& tm, int& tn) {
        if constexpr (TABLE) {                               /* vb: position in the list; tm: the product */
            if (vb >= vend) return -1;
            const int e = tile_list[vb];
            tm = e >> BL_TILE_BITS;
            tn = e & ((1 << BL_TILE_BITS) - 1);
            return vb;
        }
        for (; vb < vgrid; vb += grid)
            if (tile_of(vb, tm, tn)) return vb;
        return -1;
    };
    auto rsrc = [](const void* p, uint32_t bytes) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
    };

    /* A stage is BM/8 pieces of eight activation rows and WP pieces of 32 weight rows, 1 KB each.  Where the weight pieces
     * don't divide among the waves the last ones are fetched twice (the same bytes to the same place), so that every wave has
     * the same count in flight. */
    auto wpiece = [&](const int j) __attribute__((always_inline)) {
        return (j + 1) * NW <= WP ? j * NW + wave : j * NW + wave % (WP - j * NW > 0 ? WP - j * NW : 1);
    };
    uint32_t ao[AL], wo[WL];
    auto offsets = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < AL; ++j) {
            const int row = (j * NW + wave) * 8 + (lane >> 3);
            ao[j] = (uint32_t)row * (uint32_t)lK + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
        }
#pragma unroll
        for (int j = 0; j < WL; ++j)                         /* (inside the piece) */
            wo[j] = (uint32_t)(lane >> 1) * (uint32_t)(lK / 4) + (uint32_t)(((lane & 1) ^ ((lane >> 4) & 1)) * 16);
    };
    if constexpr (!TABLE) offsets();

    /* the load cursor: tile, k step, buffer, set of row terms */
    int lvb, ltm = 0, ltn = 0, lkk = 0, lbuf = 0, lset = 0;
    decltype(rsrc(nullptr, 0)) ra, rw[WL];
    auto setup = [&]() {
        if constexpr (TABLE) {
            const bl_tile_item it = items[ltm];
            lpacked = it.packed;
            lq = it.q;
            lrowsum = it.rowsum;
            lscale = it.scale;
            lN = it.N;
            lK = it.K;
            lsteps = lK / GP_BK;
            offsets();
        }
        const int m0 = TABLE ? 0 : ltm * BM, rows = min(BM, M - m0), kb = lK / 4;
        ra = rsrc(lq + (int64_t)m0 * lK, (uint32_t)rows * (uint32_t)lK);
#pragma unroll
        for (int j = 0; j < WL; ++j) {
            const int p = wpiece(j);
            int n;
            if (EPI == 2)      /* blocks of a wave: NI/2 of gate rows, then the matching up rows */
                n = (p % NI >= NI / 2 ? N / 2 : 0) + ltn * (BN / 2) + (p / NI) * (NI * 16) + (p % (NI / 2 > 0 ? NI / 2 : 1)) * 32;
            else
                n = ltn * BN + p * 32;
            if (n > lN - 32) n = max(min(n, lN - 1) & ~31, 0);          /* blocks past the end: the last one again */
            rw[j] = rsrc(lpacked + (int64_t)n * kb, (uint32_t)min(32, lN - n) * (uint32_t)kb);
        }
    };
    auto setup_terms = [&]() __attribute__((always_inline)) {
        const int m0 = TABLE ? 0 : ltm * BM, rows = min(BM, M - m0);
#pragma unroll
        for (int j = 0; j < (2 * BM + NW * 64 - 1) / (NW * 64); ++j) {
            const int g = (j * NW + wave) * 64;
            if (g >= 2 * BM) break;
            const bool s = g >= BM;
            const void* src = s ? (const void*)(lscale + m0) : (const void*)(lrowsum + m0);
            const auto rt = rsrc(src, s && !lscale ? 0 : rows * 4);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rt, (lds_p)(terms + lset * 2 * BM + g), 4, ((s ? g - BM : g) + lane) * 4, 0, 0, 0);
        }
    };
    uint8_t* lst = smem;
    int lko = 0;
    auto advance = [&](const bool first) __attribute__((always_inline)) {
        if (!first) {
            lbuf = lbuf + 1 == S ? 0 : lbuf + 1;
            if (++lkk == lsteps) {
                lkk = 0;
                if (lvb >= 0) {
                    lvb = next_tile(lvb + (TABLE ? 1 : grid), ltm, ltn);
                    lset = lset + 1 == SETS ? 0 : lset + 1;
                    if (lvb >= 0) {
                        setup();
                        setup_terms();
                    } else {
                        ra = rsrc(lq, 0);
#pragma unroll
                        for (int j = 0; j < WL; ++j) rw[j] = rsrc(lpacked, 0);
                        ltm = -1;
                    }
                    int* const slot = ahead + (wave * SETS + lset) * 4;
                    slot[0] = ltm;
                    slot[1] = ltn;
                    if constexpr (TABLE) slot[2] = lsteps;
                }
            }
        }
        lst = smem + lbuf * STAGE;
        lko = lvb < 0 ? 0 : max(min(lkk * GP_BK, lK - GP_BK), 0);
    };
    auto load = [&](const int j) __attribute__((always_inline)) {
        if (j < AL)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_p)(lst + (j * NW + wave) * 1024), 16, ao[j < AL ? j : 0], lko, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw[j >= AL ? j - AL : 0], (lds_p)(lst + AB + wpiece(j - AL) * 1024), 16, wo[j >= AL ? j - AL : 0], lko / 4, 0, 0);
    };
    /* With three stages a stage's loads are issued at once behind the barrier (they have one step to arrive), with more they
     * are spread over the MFMAs up to the next barrier: 2048 x 2560 -> 2560 in 128 x 192 tiles, four stages 16.8 / 17.8 us, and
     * in 128 x 256 tiles with three 23.3 / 20.6. */
    constexpr bool SPREAD = S > 3;
    /* DEEP: with few MFMAs to a sub-step they don't cover an LDS read, so a wave reads a whole step's operands one step ahead;
     * the step's barrier then stands in front of it, and the buffer of the step itself is free for loads (stage t + S). */
    constexpr bool DEEP = SL <= 4;
    constexpr int FIRST = SPREAD && !DEEP ? (LOADS + 3) / 4 : LOADS;            /* in the sub-step behind the barrier */
    constexpr int GAP = LOADS > FIRST ? 3 * SL / (LOADS - FIRST) : 1;           /* MFMAs between the others */
    static_assert(FIRST <= SL || !SPREAD || DEEP, "one load per MFMA");
    constexpr int INIT = DEEP ? S : S - 1;                                      /* stages on their way in front of the first step */

    /* per-lane LDS read offsets inside a stage */
    const int a_off = (wm0 + l32) * GP_BK, a_swz = (l32 >> 1) & 7;
    const int w_off = AB + ((wn0 + l32) * 2 + (h ^ ((l32 >> 3) & 1))) * 16;
    int au[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) au[ks] = a_off + ((4 * h + ks) ^ a_swz) * 16;

    int tm, tn;
    lvb = next_tile(TABLE ? wg_start[blockIdx.x] : (int)blockIdx.x, ltm, ltn);
    if (lvb < 0) return;
    /* measurement hook: workgroup 0 counts shader clocks and wall-clock ticks over its lifetime */
    const bool stamp = stamps != nullptr && blockIdx.x == 0;
    long long c_start = 0, w_start = 0;
    if (stamp) {
        c_start = clock64();
        w_start = wall_clock64();
    }
    tm = ltm;
    tn = ltn;
    setup();
    if constexpr (TABLE) steps = lsteps;
    if (steps >= INIT) {
#pragma unroll
        for (int s = 0; s < INIT; ++s) {
            lst = smem + s * STAGE;
            lko = min(s * GP_BK, max(lK - GP_BK, 0));
#pragma unroll
            for (int j = 0; j < (s < INIT - 1 ? LOADS : FIRST); ++j) load(j);
            if (s == 0) setup_terms();                       /* (behind the loads that are waited for first) */
        }
        lkk = lbuf = INIT - 1;
    } else {                                                 /* rows of few k steps: the first stages are of several tiles */
        setup_terms();
#pragma nounroll
        for (int s = 0; s < INIT; ++s) {
            advance(s == 0);
#pragma unroll
            for (int j = 0; j < FIRST; ++j) load(j);
            if (s < INIT - 1) {
#pragma unroll
                for (int j = FIRST; j < LOADS; ++j) load(j);
            }
        }
    }
    int stage_at = 0, set = 0;
    BL_WAIT_VM((INIT - 2) * LOADS + FIRST);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    bl_v4i wq[DEEP ? 2 : 1][NI], a[DEEP ? 8 : 2][MI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) wq[0][ni] = *(const bl_v4i*)(smem + w_off + ni * 1024);
#pragma unroll
    for (int ks = 0; ks < (DEEP ? 4 : 1); ++ks)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) a[ks][mi] = *(const bl_v4i*)(smem + au[ks] + mi * 32 * GP_BK);
    if (!TABLE && K < GP_BK && h == 1) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) wq[0][ni] = bl_v4i{0, 0, 0, 0};
    }
    /* LAYOUT 0: half (0, 1) of the 4 x 4 byte transpose of sixteen activations */
    auto turn = [&](bl_v4i& v, const int half) __attribute__((always_inline)) {
        uint32_t x0 = (uint32_t)v[0], x1 = (uint32_t)v[1], x2 = (uint32_t)v[2], x3 = (uint32_t)v[3], r0, r1, r2, r3;
        if (half == 0) {
            r0 = __builtin_amdgcn_perm(x1, x0, 0x05010400u);
            r1 = __builtin_amdgcn_perm(x1, x0, 0x07030602u);
            r2 = __builtin_amdgcn_perm(x3, x2, 0x05010400u);
            r3 = __builtin_amdgcn_perm(x3, x2, 0x07030602u);
        } else {
            r0 = __builtin_amdgcn_perm(x2, x0, 0x05040100u);
            r1 = __builtin_amdgcn_perm(x2, x0, 0x07060302u);
            r2 = __builtin_amdgcn_perm(x3, x1, 0x05040100u);
            r3 = __builtin_amdgcn_perm(x3, x1, 0x07060302u);
        }
        asm volatile("" : "+v"(r0), "+v"(r1), "+v"(r2), "+v"(r3));
        v = bl_v4i{(int)r0, (int)r1, (int)r2, (int)r3};
    };
    /* the transposes of a sub-step's activations lie in its last MFMAs: halves where there is room */
    constexpr bool HALVES = SL >= 4 * MI;
    auto turn_at = [&](bl_v4i (&v)[MI], const int sl) __attribute__((always_inline)) {
        if constexpr (TURN_A) {
            if (HALVES) {
                const int i = sl - (SL - 2 * MI);
                if (i >= 0) turn(v[i >= 0 ? i / 2 : 0], i & 1);
            } else {
                const int i = sl - (SL - MI);
                if (i >= 0) {
                    turn(v[i >= 0 ? i : 0], 0);
                    turn(v[i >= 0 ? i : 0], 1);
                }
            }
        }
    };
    if constexpr (TURN_A) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            turn(a[0][mi], 0);
            turn(a[0][mi], 1);
        }
    }
    bl_v4i bop = bl_unpack16(TURN_W ? bl_word_to_k16((uint32_t)wq[0][0][0]) : (uint32_t)wq[0][0][0]);

    while (true) {
        const int m0 = TABLE ? 0 : tm * BM, n0 = tn * BN;
        if constexpr (TABLE) {                               /* what the epilogue stores to arrives under the k loop */
            const bl_tile_item it = items[tm];
            N = it.N;
            acc = it.acc;
            y = it.y;
            residual = it.residual;
            bt = y ? *bl_gc<float>(it.beta) : 0.0f;
        }
        bl_v16i C[MI][NI];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) C[mi][ni][v] = 0;

        /* MI MFMAs of one block of 32 weight rows; behind each: `extra`, and a part of the next block's codes opened
         * (w, or with last >= 0 the first word of the next stage, from wq[last]) */
        auto chunk = [&](const int ab, const int ni, const uint32_t w, const int last, auto&& extra) __attribute__((always_inline)) {
            bl_v4i nx;
            uint32_t x = w;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                C[mi][ni] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ab][mi], bop, C[mi][ni], 0, 0, 0);
                extra(ni * MI + mi);
                if (last >= 0) x = (uint32_t)wq[last >= 0 ? last : 0][0][0];
                if (TURN_W && (mi == 0 || last >= 0)) x = bl_word_to_k16(x);
#pragma unroll
                for (int j = mi * 4 / MI; j < (mi + 1) * 4 / MI; ++j) {
                    int t = (int)((x >> 2 * j) & 0x03030303u);
                    asm volatile("" : "+v"(t));              /* (or the compiler moves it to its use) */
                    nx[j] = t;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            bop = nx;
        };
        auto clear = [&](bl_v4i (&w)[NI]) __attribute__((always_inline)) {
            const bool z = h == dead;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int i = 0; i < 4; ++i) w[ni][i] = z ? 0 : w[ni][i];
#pragma unroll
            for (int i = 0; i < 4; ++i) bop[i] = z ? 0 : bop[i];
        };
        if constexpr (DEEP) {
            /* one step: multiplies set P of the operands and reads the next step's into set 1 - P */
            auto step = [&](auto p, const int kk) __attribute__((always_inline)) {
                constexpr int P = decltype(p)::value, Q = 1 - P;
                const int ahead_at = stage_at + STAGE == S * STAGE ? 0 : stage_at + STAGE;
                /* this step's operands are in registers; the next stage has landed, the S - 2 behind it may stay in flight */
                BL_WAIT_LGKM0();
                BL_WAIT_VM((S - 2) * LOADS);
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                const uint8_t* sn = smem + ahead_at;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
                        chunk(P * 4 + ks, ni, (uint32_t)(ni + 1 < NI ? wq[P][ni + 1 < NI ? ni + 1 : 0][ks] : ks < 3 ? wq[P][0][ks < 3 ? ks + 1 : 0] : 0),
                              ks == 3 && ni + 1 == NI ? Q : -1, [&](const int sl) __attribute__((always_inline)) {
                                  constexpr int SLOTS = 4 * SL - 1, READS = NI + 4 * MI, RPER = (READS + SLOTS - 2) / (SLOTS - 1);
                                  const int at = ks * SL + sl;
                                  /* reads from the first MFMA on, so that they have the step to arrive */
#pragma unroll
                                  for (int r0 = 0; r0 < RPER; ++r0) {
                                      const int r = at * RPER + r0;
                                      if (r < NI) wq[Q][r < NI ? r : 0] = *(const bl_v4i*)(sn + w_off + r * 1024);
                                      else if (r < READS) a[Q * 4 + (r - NI) / MI % 4][(r - NI) % MI >= 0 ? (r - NI) % MI : 0] = *(const bl_v4i*)(sn + au[(r - NI) / MI % 4] + (r - NI) % MI * 32 * GP_BK);
                                  }
                                  if (at == 0) advance(false);
                                  if (at > 0) {
#pragma unroll
                                      for (int j = 0; j < LOADS; ++j)
                                          if (at == 1 + j * SLOTS / LOADS) load(j);
                                  }
                                  turn_at(ks < 3 ? a[P * 4 + (ks < 3 ? ks + 1 : 0)] : a[Q * 4], sl);
                              });
                stage_at = ahead_at;
                if (kk == zstep) clear(wq[Q]);
                __builtin_amdgcn_sched_barrier(0);
            };
            int kk = 0;
            for (; kk + 1 < steps; kk += 2) {
                step(std::integral_constant<int, 0>{}, kk);
                step(std::integral_constant<int, 1>{}, kk + 1);
            }
            if (kk < steps) {                                /* an odd step, and every tile starts with set 0 */
                step(std::integral_constant<int, 0>{}, kk);
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) wq[0][ni] = wq[DEEP ? 1 : 0][ni];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi) a[ks][mi] = a[DEEP ? 4 + ks : 0][mi];
            }
        } else {
        for (int kk = 0; kk < steps; ++kk) {
            const uint8_t* st = smem + stage_at;
            const int ahead_at = stage_at + STAGE == S * STAGE ? 0 : stage_at + STAGE;
#pragma unroll
            for (int ks = 0; ks < 3; ++ks)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    chunk(ks & 1, ni, (uint32_t)(ni + 1 < NI ? wq[0][ni + 1 < NI ? ni + 1 : 0][ks] : wq[0][0][ks + 1]), -1,
                          [&](const int sl) __attribute__((always_inline)) {
                              const int at = ks * SL + sl;
                              if (LOADS > FIRST && at % GAP == 0 && FIRST + at / GAP < LOADS) load(FIRST + at / GAP);
                              if (sl < MI) a[(ks + 1) & 1][sl < MI ? sl : 0] = *(const bl_v4i*)(st + au[ks + 1] + sl * 32 * GP_BK);
                              turn_at(a[(ks + 1) & 1], sl);
                          });
            __builtin_amdgcn_sched_barrier(0);
            /* the next stage has landed; the S - 3 behind it may stay in flight */
            BL_WAIT_VM((S - 3) * LOADS);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const uint8_t* sn = smem + ahead_at;             /* (behind the last step of all: zeros or an old stage, unused) */
            uint32_t w3[NI];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) w3[ni] = (uint32_t)wq[0][ni][3];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                chunk(1, ni, ni + 1 < NI ? w3[ni + 1 < NI ? ni + 1 : 0] : 0u, ni + 1 == NI ? 0 : -1, [&](const int sl) __attribute__((always_inline)) {
                    /* (scalar work between the barrier and the first MFMA would hold up both) */
                    if (sl == 0) advance(false);
                    if constexpr (!SPREAD) {
                        if (sl == 1) {
#pragma unroll
                            for (int j = 0; j < LOADS; ++j) load(j);
                        }
                    } else {
                        constexpr int E = SL / FIRST;
                        if (sl % E == E - 1 && sl / E < FIRST) load(sl / E);
                        static_assert(E > 1, "behind advance");
                    }
                    /* first code word, activations, the other words */
                    constexpr int PER = (NI + MI + SL - 1) / SL;
#pragma unroll
                    for (int r0 = 0; r0 < PER; ++r0) {
                        const int r = sl * PER + r0;
                        if (r >= 1 && r <= MI) {
                            a[0][r >= 1 && r <= MI ? r - 1 : 0] = *(const bl_v4i*)(sn + au[0] + (r - 1) * 32 * GP_BK);
                        } else if (r < NI + MI) {
                            const int wi = r == 0 ? 0 : r - MI;
                            wq[0][wi < NI ? wi : 0] = *(const bl_v4i*)(sn + w_off + wi * 1024);
                        }
                    }
                    turn_at(a[0], sl);
                });
            stage_at = ahead_at;
            if (kk == zstep) clear(wq[0]);
            __builtin_amdgcn_sched_barrier(0);
        }
        }

        /* Epilogue: the loads of the next tile's first stages travel meanwhile. */
        bl_mfma_fence();
        const int* const rs_s = terms + set * 2 * BM;
        const float* const sc_s = (const float*)(rs_s + BM);
        /* Outputs through descriptors of the tile's rows: rows past M are out of their range, columns past the last get an
         * offset out of any range, so one form without branches serves every tile (a form per output with a condition per value
         * is so much code, each of it met once per tile, that fetching it took longer than the tile's k loop:
         * 1000 x 2560 -> 3840 in 128 x 128 tiles 20.5 / 14.7 us). */
        constexpr uint32_t NOWHERE = 0x80000000u;
        constexpr int NT = 2;                                 /* non-temporal */
        constexpr int AHEAD = SL > 4 ? 2 : MI == 1 ? 3 : 4;   /* groups of residual values on their way (more spill) */
        /* A descriptor of the eight rows of group g of the wave (rows of `bytes` bytes), none past M. */
        auto span = [&](const void* p, const uint32_t bytes, const int g) __attribute__((always_inline)) {
            const int m = m0 + wm0 + g * 8, left = __builtin_amdgcn_readfirstlane(max(min(8, M - m), 0));
            return rsrc((const uint8_t*)p + (int64_t)m * bytes, (uint32_t)left * bytes);
        };
        /* every row of the lane, four to a group: before(g), row(g, mi, v, v4, row sum, factor), after(g, its first row in the tile) */
        auto rows = [&](auto&& before, auto&& row, auto&& after) __attribute__((always_inline)) {
#pragma unroll
            for (int g = 0; g < 4 * MI; ++g) {
                int ml = wm0 + g * 8 + h * 4;
                if (SL > 4) asm volatile("" : "+v"(ml));     /* (large tiles: keeps the groups apart, or registers spill) */
                before(g);
                const bl_v4i rs = *(const bl_v4i*)(rs_s + ml);
                const bl_v4f sc = *(const bl_v4f*)(sc_s + ml);
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) row(g, g / 4, (g % 4) * 4 + v4, v4, rs[v4], bt * sc[v4]);
                after(g, ml);
                if (SL > 4) __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto nothing = [](auto...) __attribute__((always_inline)) {};
        const uint32_t wide = (uint32_t)N * 4;
        decltype(rsrc(nullptr, 0)) ro, rr;
        if (acc) {
            uint32_t col[NI];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int n = EPI == 2 ? tn * (BN / 2) + wn0 / 2 + ni % (NI / 2 > 0 ? NI / 2 : 1) * 32 + l32 : n0 + wn0 + ni * 32 + l32;
                const bool up = EPI == 2 && ni >= NI / 2;
                col[ni] = (n < (EPI == 2 ? N / 2 : N) ? (uint32_t)(up ? N / 2 + n : n) * 4 : NOWHERE) + (uint32_t)(h * 4) * wide;
            }
            rows([&](const int g) __attribute__((always_inline)) { ro = span(acc, wide, g); },
                 [&](const int, const int mi, const int v, const int v4, const int rs, const float) __attribute__((always_inline)) {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) __builtin_amdgcn_raw_buffer_store_b32(C[mi][ni][v] - rs, ro, col[ni] + (uint32_t)v4 * wide, 0, 0);
            }, nothing);
        }
        if constexpr (EPI == 0) {
            uint32_t col[NI];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int n = n0 + wn0 + ni * 32 + l32;
                col[ni] = (n < N ? (uint32_t)n * 4 : NOWHERE) + (uint32_t)(h * 4) * wide;
            }
            auto plain = [&](auto nt) __attribute__((always_inline)) {
                rows([&](const int g) __attribute__((always_inline)) { ro = span(y, wide, g); },
                     [&](const int, const int mi, const int v, const int v4, const int rs, const float c) __attribute__((always_inline)) {
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int((float)(C[mi][ni][v] - rs) * c), ro, col[ni] + (uint32_t)v4 * wide, 0, decltype(nt)::value);
                }, nothing);
            };
            if (y && !residual) {
                if (bl_past_caches(M, N, acc != nullptr)) plain(std::integral_constant<int, NT>{});
                else plain(std::integral_constant<int, 0>{});
            } else if (y) {
                /* the residual values are requested ahead of their rows */
                constexpr int RING = AHEAD;
                float res[RING][4][NI];
                auto fetch = [&](const int g) __attribute__((always_inline)) {
                    rr = span(residual, wide, g);
#pragma unroll
                    for (int v4 = 0; v4 < 4; ++v4)
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni)
                            res[g % RING][v4][ni] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rr, col[ni] + (uint32_t)v4 * wide, 0, 0));
                };
#pragma unroll
                for (int g = 0; g < RING; ++g) fetch(g);
                rows([&](const int g) __attribute__((always_inline)) { ro = span(y, wide, g); },
                     [&](const int g, const int mi, const int v, const int v4, const int rs, const float c) __attribute__((always_inline)) {
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(res[g % RING][v4][ni] + (float)(C[mi][ni][v] - rs) * c), ro, col[ni] + (uint32_t)v4 * wide, 0, NT);
                }, [&](const int g, const int) __attribute__((always_inline)) {
                    if (g + RING < 4 * MI) fetch(g + RING);
                });
            }
        } else {
            /* fused producer epilogue: glue value t, its bf16 narrowing (the next BitLinear's input before quantisation) and the
             * row maximum of |bf16(t)|: over the lane's columns, then over the 32 lanes of a half wave (DPP), then one atomic
             * max for the eight rows of a group on the float bits (non-negative floats order like integers, so the result does
             * not depend on the order).  Two rows at a time: a lane narrows its column of both in one instruction, trades with
             * its neighbour and stores two columns of one row, and the maxima are taken on 16-bit patterns, both rows at once. */
            typedef short v2s __attribute__((ext_vector_type(2)));
            constexpr int MAG = 0x007F007F;           /* added to magnitudes: infinity is the largest int16, a NaN negative */
            constexpr int NO = EPI == 2 ? NI / 2 : NI;
            const int NOUT = EPI == 2 ? N / 2 : N;
            const uint32_t narrow = (uint32_t)NOUT * 2;
            uint32_t colx[NO], coly[NO];
            int in[NO];
#pragma unroll
            for (int ni = 0; ni < NO; ++ni) {
                const int n = (EPI == 2 ? tn * (BN / 2) + wn0 / 2 : n0 + wn0) + ni * 32 + l32;
                in[ni] = n < NOUT ? 0x7FFF7FFF : 0;
                coly[ni] = (n < NOUT ? (uint32_t)n * 4 : NOWHERE) + (uint32_t)(h * 4) * narrow * 2;
                colx[ni] = (n < NOUT ? (uint32_t)(ODD ? n : n & ~1) * 2 : NOWHERE) + (uint32_t)(h * 4 + (ODD ? 0 : lane & 1)) * narrow;
            }
            const uint32_t pick = lane & 1 ? 0x03020706u : 0x05040100u;
            decltype(rsrc(nullptr, 0)) rx;
            /* EPI 1: the residual values are requested ahead */
            constexpr int RING = AHEAD;
            float res[RING][4][EPI == 1 ? NI : 1];
            auto fetch = [&](const int g) __attribute__((always_inline)) {
                rr = span(residual, narrow * 2, g);
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4)
#pragma unroll
                    for (int ni = 0; ni < NO; ++ni)
                        res[g % RING][v4][EPI == 1 ? ni : 0] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rr, coly[ni] + (uint32_t)v4 * narrow * 2, 0, 0));
            };
            if constexpr (EPI == 1) {
#pragma unroll
                for (int g = 0; g < RING; ++g) fetch(g);
            }
            float first[NO];
            int most[2];
            auto gated = [&](const int mi, const int ni, const int v, const int rs, const float c) __attribute__((always_inline)) {
                const float t = (float)(C[mi][ni][v] - rs) * c, u = (float)(C[mi][ni + (EPI == 2 ? NO : 0)][v] - rs) * c;
                const float r = fmaxf(t, 0.0f);
                const float r2 = r * r;
                return r2 * u;
            };
            if (EPI == 2 && y) {
                rows([&](const int g) __attribute__((always_inline)) { ro = span(y, narrow * 2, g); },
                     [&](const int, const int mi, const int v, const int v4, const int rs, const float c) __attribute__((always_inline)) {
#pragma unroll
                    for (int ni = 0; ni < NO; ++ni)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(gated(mi, ni, v, rs, c)), ro, coly[ni] + (uint32_t)v4 * narrow * 2, 0, NT);
                }, nothing);
            }
            rows([&](const int g) __attribute__((always_inline)) {
                rx = span(xb, narrow, g);
                if (EPI == 1) ro = span(y, y ? narrow * 2 : 0, g);      /* (no fp32 output: nothing in range) */
            }, [&](const int g, const int mi, const int v, const int v4, const int rs, const float c) __attribute__((always_inline)) {
                v2s mx = __builtin_bit_cast(v2s, MAG);
#pragma unroll
                for (int ni = 0; ni < NO; ++ni) {
                    const float o = EPI == 1 ? res[g % RING][v4][EPI == 1 ? ni : 0] + (float)(C[mi][ni][v] - rs) * c : gated(mi, ni, v, rs, c);
                    if (EPI == 1) __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(o), ro, coly[ni] + (uint32_t)v4 * narrow * 2, 0, NT);
                    if (v4 % 2 == 0) {
                        first[ni] = o;
                    } else {
                        const uint32_t two = bl_pack2_bf16(first[ni], o);
                        if constexpr (ODD) {
                            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)two, rx, colx[ni] + (uint32_t)(v4 - 1) * narrow, 0, 0);
                            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(two >> 16), rx, colx[ni] + (uint32_t)v4 * narrow, 0, 0);
                        } else {
                            const uint32_t other = (uint32_t)bl_dpp<BL_DPP_QUAD_XOR1>((int)two);
                            __builtin_amdgcn_raw_buffer_store_b32((int)__builtin_amdgcn_perm(other, two, pick), rx, colx[ni] + (uint32_t)(v4 - 1) * narrow, 0, 0);
                        }
                        const v2s mag = __builtin_bit_cast(v2s, (int)two & in[ni]) + __builtin_bit_cast(v2s, MAG);
                        mx = __builtin_elementwise_max(mx, mag);
                    }
                }
                if (v4 % 2 == 1) most[v4 / 2] = __builtin_bit_cast(int, mx);
            }, [&](const int g, const int ml) __attribute__((always_inline)) {
                if constexpr (EPI == 1) {
                    if (g + RING < 4 * MI) fetch(g + RING);
                }
                auto larger = [](const int a, const int b) __attribute__((always_inline)) {
                    return __builtin_bit_cast(int, __builtin_elementwise_max(__builtin_bit_cast(v2s, a), __builtin_bit_cast(v2s, b)));
                };
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    int m = most[i];
                    m = larger(m, bl_dpp<BL_DPP_QUAD_XOR1>(m));
                    m = larger(m, bl_dpp<BL_DPP_QUAD_XOR2>(m));
                    m = larger(m, bl_dpp<BL_DPP_ROW_HALF_MIRROR>(m));
                    m = larger(m, bl_dpp<BL_DPP_ROW_MIRROR>(m));
                    const auto t = __builtin_amdgcn_permlane16_swap((uint32_t)m, (uint32_t)m, false, false);
                    most[i] = __builtin_bit_cast(int, __builtin_bit_cast(v2s, larger((int)t[0], (int)t[1])) - __builtin_bit_cast(v2s, MAG));
                }
                /* lane v4 of a half stands for row v4: one atomic instruction for eight rows, which travels under the groups
                 * behind it (all of them behind the last group are waited for by themselves: gate 74 x 384 -> 2560 6.0 us, so 5.5,
                 * 834 x 256 -> 3328 6.9 / 6.3, 764 x 896 -> 10240 15.8 / 14.1; residual 65 x 2560 -> 2560 11.5 / 10.8, at 2048 tokens 22.9 / 23.3) */
                if (l32 < 4) {
                    const int m = m0 + ml + l32, pair = l32 < 2 ? most[0] : most[1];
                    if (m < M) atomicMax(absmax + m, l32 & 1 ? pair & (int)0xFFFF0000 : pair << 16);
                }
            });
        }
        set = set + 1 == SETS ? 0 : set + 1;
        const int* const slot = ahead + (wave * SETS + set) * 4;
        const int ntm = __builtin_amdgcn_readfirstlane(slot[0]);
        if (ntm < 0) {
            /* No load may write to LDS once the workgroup has gone: those behind the last tile are older than the tile's
             * outputs, of which there are at least OUT (a wait for those would be half a microsecond). */
            constexpr int OUT = EPI == 0 ? 16 * MI * NI : EPI == 1 ? 24 * MI * NI : 4 * MI * NI, MAXES = EPI == 0 ? 0 : 4 * MI;
            if (m0 + BM <= M) BL_WAIT_VM(OUT + MAXES < 63 ? OUT + MAXES : 63);
            else BL_WAIT_VM(OUT < 63 ? OUT : 63);
            break;
        }
        tm = ntm;
        tn = __builtin_amdgcn_readfirstlane(slot[1]);
        if constexpr (TABLE) steps = __builtin_amdgcn_readfirstlane(slot[2]);
    }
    if (stamp && tid == 0) {
        stamps[0] = clock64() - c_start;
        stamps[1] = wall_clock64() - w_start;
    }
#endif
}
