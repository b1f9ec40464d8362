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
 * What bounds it: the LDS serves arriving direct loads at about 48 B/clk and reads at about 138 B/clk, one after the other,
 * and the matrix cores of a CU take 32 clocks for four 32x32x32.  A 128 x 256 tile in 2 x 2 waves of 64 x 128 needs 500 + 348
 * clocks of LDS for 1024 of MFMA, 128 x 128 in waves of 64 x 64 417 + 290 for 512: the wide tile is what lets the matrix
 * cores run, and the fixed order is what lets two waves per SIMD (its registers) be enough.  Without output stores it reaches
 * 2.9 POP/s (8192 x 4096 -> 8192; 1.74 GHz under power management, where the bare MFMA loop reaches 3.4 - 3.6), the
 * kernel of 128 x 128 tiles before it 2.3.
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
 * rows are NI/2 blocks of gate rows and the NI/2 matching blocks of up rows (n and N/2 + n), t = (relu(g)*relu(g))*u. */
#pragma once
#include "bl_device.h"

#include <type_traits>

#define GP_BK 128

/* sets of row terms: the tile in its epilogue and those that the loads may have reached */
template <int MI, int NI, int WM, int WN, int S>
struct bl_pipe_geom {
    static constexpr int BM = WM * MI * 32, BN = WN * NI * 32, THREADS = WM * WN * 64;
    static constexpr int A_BYTES = BM * GP_BK, W_BYTES = BN * GP_BK / 4, STAGE = A_BYTES + W_BYTES;
    static constexpr int LDS = S * STAGE + S * BM * 8 + S * WM * WN * 8;
};

template <int MI, int NI, int WM, int WN, int S, int OCC, int EPI, int LAYOUT>
__global__ __launch_bounds__(WM * WN * 64, OCC) void bl_gemm_pipe(const uint8_t* __restrict__ packed, const int8_t* __restrict__ q,
                                                                  const int32_t* __restrict__ rowsum, const float* __restrict__ beta,
                                                                  const float* __restrict__ scale, int M, int N, int K, int tiles_m,
                                                                  int tiles_n, int gm, int band, int vgrid, int grid,
                                                                  const float* __restrict__ residual, int32_t* __restrict__ acc,
                                                                  float* __restrict__ y, uint16_t* __restrict__ xb,
                                                                  int* __restrict__ absmax, long long* __restrict__ stamps) {
#if defined(__HIP_DEVICE_COMPILE__)   /* (the host has no type for a buffer descriptor) */
    using G = bl_pipe_geom<MI, NI, WM, WN, S>;
    constexpr int NW = WM * WN, BM = G::BM, BN = G::BN, STAGE = G::STAGE, AB = G::A_BYTES;
    constexpr int AL = AB / 1024 / NW, WP = G::W_BYTES / 1024, WL = (WP + NW - 1) / NW, LOADS = AL + WL;
    constexpr int SL = MI * NI;                              /* MFMAs of a sub-step */
    static_assert(AB % (1024 * NW) == 0 && S >= 3 && (S - 2) * LOADS < 64, "whole loads per wave; vmcnt is a 6-bit count");
    static_assert(EPI != 2 || NI % 2 == 0, "gate and up blocks in pairs");
    constexpr bool TURN_A = LAYOUT == 0 && NI > 1, TURN_W = LAYOUT == 0 && NI == 1;
    typedef __attribute__((address_space(3))) void* lds_p;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    int* const terms = (int*)(smem + S * STAGE);             /* S sets of BM row sums and BM scales */
    int* const ahead = terms + S * 2 * BM;                   /* each wave's tiles that the loads have reached: S of (tm, tn) */
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int wm0 = (wave / WN) * (MI * 32), wn0 = (wave % WN) * (NI * 32);
    const int kb = K / 4, steps = (K + GP_BK - 1) / GP_BK;
    /* at the end of step `zstep` of a tile the codes at hand are those of a half step */
    const int zstep = K % GP_BK == 0 ? -1 : max(steps - 2, 0), dead = K < GP_BK ? 1 : 0;
    const float bt = (EPI != 0 || y != nullptr) ? *beta : 0.0f;

    /* XCD-aware tile order: workgroup L runs on XCD L%8.  The row tiles are cut into bands so narrow that
     * a band's activation panel stays in an XCD's 4 MB L2 while its weight tiles stream through, row tiles
     * fastest.  Either a rectangle per XCD (gm bands x 8 / gm column blocks), or (gm = 0) the tiles are
     * numbered band by band and each XCD takes one eighth of the sequence; the host chooses.  The grid is persistent:
     * a workgroup takes virtual blocks vb = blockIdx.x, + grid, .. (grid is a multiple of 8). */
    const int tiles = tiles_m * tiles_n, share = (tiles + 7) >> 3, band_tiles = band * tiles_n;
    const int gn = gm ? 8 / gm : 1, cols = (tiles_n + gn - 1) / gn;
    auto tile_of = [&](int vb, int& tm, int& tn) {
        const int xcd = vb & 7, idx = vb >> 3;
        if (gm) {
            tm = (xcd / gn) * band + idx % band;
            tn = (xcd % gn) * cols + idx / band;
            return idx < band * cols && tm < tiles_m && tn < tiles_n;
        }
        const int at = xcd * share + idx;
        if (idx >= share || at >= tiles) return false;
        const int b = at / band_tiles, in = at - b * band_tiles;
        const int rows = min(band, tiles_m - b * band);
        tn = in / rows;
        tm = b * band + (in - tn * rows);
        return true;
    };
    auto next_tile = [&](int vb, int& tm, int& tn) {
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
#pragma unroll
    for (int j = 0; j < AL; ++j) {
        const int row = (j * NW + wave) * 8 + (lane >> 3);
        ao[j] = (uint32_t)row * (uint32_t)K + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
    }
#pragma unroll
    for (int j = 0; j < WL; ++j)                             /* (inside the piece) */
        wo[j] = (uint32_t)(lane >> 1) * (uint32_t)kb + (uint32_t)(((lane & 1) ^ ((lane >> 4) & 1)) * 16);

    /* the load cursor: tile, k step, buffer, set of row terms */
    int lvb, ltm = 0, ltn = 0, lkk = 0, lbuf = 0, lset = 0;
    decltype(rsrc(nullptr, 0)) ra, rw[WL];
    auto setup = [&]() {
        const int m0 = ltm * BM, rows = min(BM, M - m0);
        ra = rsrc(q + (int64_t)m0 * K, (uint32_t)rows * (uint32_t)K);
#pragma unroll
        for (int j = 0; j < WL; ++j) {
            const int p = wpiece(j);
            int n;
            if (EPI == 2)      /* blocks of a wave: NI/2 of gate rows, then the matching up rows */
                n = (p % NI >= NI / 2 ? N / 2 : 0) + ltn * (BN / 2) + (p / NI) * (NI * 16) + (p % (NI / 2 > 0 ? NI / 2 : 1)) * 32;
            else
                n = ltn * BN + p * 32;
            if (n > N - 32) n = max(min(n, N - 1) & ~31, 0);          /* blocks past the end: the last one again */
            rw[j] = rsrc(packed + (int64_t)n * kb, (uint32_t)min(32, N - n) * (uint32_t)kb);
        }
#pragma unroll
        for (int j = 0; j < (2 * BM + NW * 64 - 1) / (NW * 64); ++j) {
            const int g = (j * NW + wave) * 64;
            if (g >= 2 * BM) break;
            const bool s = g >= BM;
            const void* src = s ? (const void*)(scale + m0) : (const void*)(rowsum + m0);
            const auto rt = rsrc(src, s && !scale ? 0 : rows * 4);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rt, (lds_p)(terms + lset * 2 * BM + g), 4, ((s ? g - BM : g) + lane) * 4, 0, 0, 0);
        }
    };
    uint8_t* lst = smem;
    int lko = 0;
    auto advance = [&](const bool first) __attribute__((always_inline)) {
        if (!first) {
            lbuf = lbuf + 1 == S ? 0 : lbuf + 1;
            if (++lkk == steps) {
                lkk = 0;
                if (lvb >= 0) {
                    lvb = next_tile(lvb + grid, ltm, ltn);
                    lset = lset + 1 == S ? 0 : lset + 1;
                    if (lvb >= 0) {
                        setup();
                    } else {
                        ra = rsrc(q, 0);
#pragma unroll
                        for (int j = 0; j < WL; ++j) rw[j] = rsrc(packed, 0);
                        ltm = -1;
                    }
                    int* const slot = ahead + (wave * S + lset) * 2;
                    slot[0] = ltm;
                    slot[1] = ltn;
                }
            }
        }
        lst = smem + lbuf * STAGE;
        lko = lvb < 0 ? 0 : max(min(lkk * GP_BK, K - GP_BK), 0);
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
    constexpr int FIRST = SPREAD ? (LOADS + 3) / 4 : LOADS;                     /* in the sub-step behind the barrier */
    constexpr int GAP = LOADS > FIRST ? 3 * SL / (LOADS - FIRST) : 1;           /* MFMAs between the others */
    static_assert(FIRST <= SL || !SPREAD, "one load per MFMA");

    /* per-lane LDS read offsets inside a stage */
    const int a_off = (wm0 + l32) * GP_BK, a_swz = (l32 >> 1) & 7;
    const int w_off = AB + ((wn0 + l32) * 2 + (h ^ ((l32 >> 3) & 1))) * 16;
    int au[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) au[ks] = a_off + ((4 * h + ks) ^ a_swz) * 16;

    int tm, tn;
    lvb = next_tile((int)blockIdx.x, ltm, ltn);
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
#pragma nounroll
    for (int s = 0; s < S - 1; ++s) {
        advance(s == 0);
#pragma unroll
        for (int j = 0; j < FIRST; ++j) load(j);
        if (s < S - 2) {
#pragma unroll
            for (int j = FIRST; j < LOADS; ++j) load(j);
        }
    }
    int buf = 0, set = 0;
    BL_WAIT_VM((S - 3) * LOADS + FIRST);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    bl_v4i wq[NI], a[2][MI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) wq[ni] = *(const bl_v4i*)(smem + w_off + ni * 1024);
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) a[0][mi] = *(const bl_v4i*)(smem + au[0] + mi * 32 * GP_BK);
    if (K < GP_BK && h == 1) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) wq[ni] = bl_v4i{0, 0, 0, 0};
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
    bl_v4i bop = bl_unpack16(TURN_W ? bl_word_to_k16((uint32_t)wq[0][0]) : (uint32_t)wq[0][0]);

    while (true) {
        const int m0 = tm * BM, n0 = tn * BN;
        bl_v16i C[MI][NI];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) C[mi][ni][v] = 0;

        /* MI MFMAs of one block of 32 weight rows; behind each: `extra`, and a part of the next block's codes opened
         * (w, or with `last` the first word of the next stage) */
        auto chunk = [&](const int ab, const int ni, const uint32_t w, const bool last, auto&& extra) __attribute__((always_inline)) {
            bl_v4i nx;
            uint32_t x = w;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                C[mi][ni] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ab][mi], bop, C[mi][ni], 0, 0, 0);
                extra(ni * MI + mi);
                if (last) x = (uint32_t)wq[0][0];
                if (TURN_W && (mi == 0 || last)) x = bl_word_to_k16(x);
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
        for (int kk = 0; kk < steps; ++kk) {
            const uint8_t* st = smem + buf * STAGE;
#pragma unroll
            for (int ks = 0; ks < 3; ++ks)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    chunk(ks & 1, ni, (uint32_t)(ni + 1 < NI ? wq[ni + 1 < NI ? ni + 1 : 0][ks] : wq[0][ks + 1]), false,
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
            advance(false);
            __builtin_amdgcn_sched_barrier(0);
            buf = buf + 1 == S ? 0 : buf + 1;
            const uint8_t* sn = smem + buf * STAGE;          /* (behind the last step of all: zeros or an old stage, unused) */
            uint32_t w3[NI];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) w3[ni] = (uint32_t)wq[ni][3];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                chunk(1, ni, ni + 1 < NI ? w3[ni + 1 < NI ? ni + 1 : 0] : 0u, ni + 1 == NI, [&](const int sl) __attribute__((always_inline)) {
                    if constexpr (!SPREAD) {
                        if (sl == 0) {
#pragma unroll
                            for (int j = 0; j < LOADS; ++j) load(j);
                        }
                    } else {
                        constexpr int E = SL / FIRST;
                        if (sl % E == E - 1 && sl / E < FIRST) load(sl / E);
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
                            wq[wi < NI ? wi : 0] = *(const bl_v4i*)(sn + w_off + wi * 1024);
                        }
                    }
                    turn_at(a[0], sl);
                });
            if (kk == zstep && h == dead) {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) wq[ni] = bl_v4i{0, 0, 0, 0};
                bop = bl_v4i{0, 0, 0, 0};
            }
            __builtin_amdgcn_sched_barrier(0);
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
                asm volatile("" : "+v"(ml));
                before(g);
                const bl_v4i rs = *(const bl_v4i*)(rs_s + ml);
                const bl_v4f sc = *(const bl_v4f*)(sc_s + ml);
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) row(g, g / 4, (g % 4) * 4 + v4, v4, rs[v4], bt * sc[v4]);
                after(g, ml);
                __builtin_amdgcn_sched_barrier(0);
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
                /* A non-temporal store of part of a line goes to memory as part of a line once the output outgrows the L2
                 * (3812 x 677 -> 6613 51.1 us, plain stores 35.0; 2048 x 2560 -> 13826 77.2 / 73.0; whole and half lines or
                 * outputs that fit gain by it: 2048 x 2560 -> 13840 66.7 / 69.3, 1000 x 2560 -> 3850 15.1 / 15.9). */
                if (N % 16 == 0 || (int64_t)M * N <= (8 << 20)) plain(std::integral_constant<int, NT>{});
                else plain(std::integral_constant<int, 0>{});
            } else if (y) {
                /* the residual values of four rows first, then their stores back to back: a load
                 * between two stores would make each store wait for the one before it */
                float res[4][NI];
                rows([&](const int g) __attribute__((always_inline)) {
                    ro = span(y, wide, g);
                    rr = span(residual, wide, g);
#pragma unroll
                    for (int v4 = 0; v4 < 4; ++v4)
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni)
                            res[v4][ni] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rr, col[ni] + (uint32_t)v4 * wide, 0, 0));
                }, [&](const int, const int mi, const int v, const int v4, const int rs, const float c) __attribute__((always_inline)) {
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(res[v4][ni] + (float)(C[mi][ni][v] - rs) * c), ro, col[ni] + (uint32_t)v4 * wide, 0, NT);
                }, nothing);
            }
        } else {
            /* fused producer epilogue: glue value t, its bf16 narrowing (the next BitLinear's input before quantisation) and the
             * row maximum of |bf16(t)|: over the lane's columns, then over the 32 lanes of a half wave (DPP), then one atomic
             * max for the eight rows of a group on the float bits (non-negative floats order like integers, so the result does
             * not depend on the order). */
            constexpr int MAG0 = 0x007F0000;          /* added to a magnitude's bits: infinity is the largest int, a NaN negative */
            constexpr int NO = EPI == 2 ? NI / 2 : NI;
            const int NOUT = EPI == 2 ? N / 2 : N;
            const uint32_t narrow = (uint32_t)NOUT * 2;
            uint32_t colb[NO];
            bool in[NO];
#pragma unroll
            for (int ni = 0; ni < NO; ++ni) {
                const int n = (EPI == 2 ? tn * (BN / 2) + wn0 / 2 : n0 + wn0) + ni * 32 + l32;
                in[ni] = n < NOUT;
                colb[ni] = (in[ni] ? (uint32_t)n * 2 : NOWHERE / 2) + (uint32_t)(h * 4) * narrow;
            }
            decltype(rsrc(nullptr, 0)) rx;
            /* EPI 1: the residual values of two groups are requested ahead */
            float res[2][4][EPI == 1 ? NI : 1];
            auto fetch = [&](const int g) __attribute__((always_inline)) {
                rr = span(residual, narrow * 2, g);
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4)
#pragma unroll
                    for (int ni = 0; ni < NO; ++ni)
                        res[g & 1][v4][EPI == 1 ? ni : 0] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rr, (colb[ni] + (uint32_t)v4 * narrow) * 2, 0, 0));
            };
            if constexpr (EPI == 1) {
                fetch(0);
                fetch(1);
            }
            float rowmax[4];
            rows([&](const int g) __attribute__((always_inline)) {
                rx = span(xb, narrow, g);
                ro = span(y, y ? narrow * 2 : 0, g);          /* (no fp32 output: nothing in range) */
            }, [&](const int g, const int mi, const int v, const int v4, const int rs, const float c) __attribute__((always_inline)) {
                int mx = MAG0;
#pragma unroll
                for (int ni = 0; ni < NO; ++ni) {
                    const float t = (float)(C[mi][ni][v] - rs) * c;
                    float o;
                    if (EPI == 1) {
                        o = res[g & 1][v4][EPI == 1 ? ni : 0] + t;
                    } else {
                        const float u = (float)(C[mi][ni + (EPI == 2 ? NO : 0)][v] - rs) * c;
                        const float r = fmaxf(t, 0.0f);
                        const float r2 = r * r;
                        o = r2 * u;
                    }
                    if (EPI == 1 || y) __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(o), ro, (colb[ni] + (uint32_t)v4 * narrow) * 2, 0, NT);
                    const uint32_t bits = bl_pack2_bf16(o, o);
                    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)bits, rx, colb[ni] + (uint32_t)v4 * narrow, 0, 0);
                    const int mag = (int)(((bits << 16) & 0x7FFF0000u) + (uint32_t)MAG0);
                    mx = max(mx, in[ni] ? mag : MAG0);
                }
                rowmax[v4] = __int_as_float(mx - MAG0);
            }, [&](const int g, const int ml) __attribute__((always_inline)) {
                if constexpr (EPI == 1) {
                    if (g + 2 < 4 * MI) fetch(g + 2);
                }
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) rowmax[v4] = bl_half_max(rowmax[v4]);
                /* lane v4 of a half stands for row v4: one atomic instruction for eight rows */
                const float mine = l32 == 0 ? rowmax[0] : l32 == 1 ? rowmax[1] : l32 == 2 ? rowmax[2] : rowmax[3];
                if (l32 < 4 && m0 + ml + l32 < M) atomicMax(absmax + m0 + ml + l32, __float_as_int(mine));
            });
        }
        set = set + 1 == S ? 0 : set + 1;
        const int* const slot = ahead + (wave * S + set) * 2;
        tm = __builtin_amdgcn_readfirstlane(slot[0]);
        tn = __builtin_amdgcn_readfirstlane(slot[1]);
        if (tm < 0) break;
    }
    BL_WAIT_VM(0);
    if (stamp && tid == 0) {
        stamps[0] = clock64() - c_start;
        stamps[1] = wall_clock64() - w_start;
    }
#endif
}
