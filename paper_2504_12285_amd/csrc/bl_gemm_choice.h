/* Which kernel a prefill product takes and in which order its tiles are walked (bl_gemm.hip); host code without the runtime, so
 * that a host program can ask it (tests/gemm_choice_driver.cpp). */
#pragma once
#include <stdint.h>

#define GP_BK 128   /* columns of a k step */

/* Order of the tiles (see bl_gemm_pipe).  Rows of activations per band: at most ~1.5 MB of int8 (measured, medians of six
 * interleaved rounds at M = 2048: +7 % on the 13824-wide shape against bands of all rows, equal on the others).  A rectangle
 * per XCD unless its size means more tiles for the busiest of an XCD's 32 compute units than an even share
 * does: 2140 x 3840 -> 13458 (17 row tiles, bands of 3: two XCDs idle) 148 / 122 us, 1100 x 2560 -> 7000 (70
 * tiles against 62) 36 / 27.5; 777 x 2999 -> 5003 with its quantiser (70 and 60 tiles against 65: three on
 * the busiest unit either way) 28.1 / 30.6 (tiles of 128 x 128 and 64 x 128). */
struct bl_tile_order {
    int gm, band, vgrid;
};
static inline bl_tile_order bl_tile_order_of(int tiles_m, int tiles_n, int BM, int K) {
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

/* Order of the split k loop's tiles (64 x 32) and what an XCD then reads for its eighth of them, bytes per k: 64 to a row tile, 8 to a
 * column tile.  A share is a run of whole and partial lines in one order, and all that lies along a line in the other.  Columns first (across)
 * where that takes a quarter off the bytes.  us, rows first / across: 3931 x 4480 -> 256 (62 row tiles and 8 column tiles: rows
 * first, every XCD reads all activations) 24.4 / 12.5, 2528 x 1877 -> 320 10.5 / 7.3, 512 x 2560 -> 1024 6.8 / 6.5, 408 x 3519 -> 925 8.0 / 7.6; nearer
 * to even it gains nothing and loses where K is long: 395 x 2176 -> 1600 7.7 / 8.3, 329 x 4794 -> 1438 11.5 / 14.2 (130 shapes: at
 * most three quarters 0.60 - 1.00 of the time, from there to even 0.98 - 1.24). */
struct bl_ksplit_order {
    bool across;
    int64_t bytes;
};
static inline bl_ksplit_order bl_ksplit_order_of(int m, int n) {
    const int64_t tm = (m + 63) / 64, tn = (n + 31) / 32, share = (tm * tn + 7) / 8;
    /* lines of `along` tiles that a share touches, of `all` */
    auto lines = [=](int64_t along, int64_t all) {
        const int64_t l = share % along == 0 ? share / along : along % share == 0 ? 1 : (share - 1) / along + 2;
        return l < all ? l : all;
    };
    const int64_t down = (share < tm ? share : tm) * 64 + lines(tm, tn) * 8, over = (share < tn ? share : tn) * 8 + lines(tn, tm) * 64;
    const bool across = 4 * over <= 3 * down;
    return {across, across ? over : down};
}

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
static inline int bl_least(const bl_tile_cost (&cost)[COUNT], int m, int n, int k, float* us = nullptr) {
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

/* Tile choice of a plain product: the kernel with the least time by this estimate (us),
 *     fixed + busiest * (steps * (step + lone) + tile) + 2^-20 outputs,
 * busiest = tiles of the busiest of 256 compute units, lone (to `step`) only where no unit has more than one.  Fitted to 200 shapes in
 * both layouts (65 .. 4096 x 300 .. 14000, K 256 .. 7000).  Over 380 products of other shapes, K 64 .. 7000, the choice (with the split k
 * loop) takes 1.010 times the time of the best of the six, and .87 of that of the kernels before them (128 x 128 with deferred stores, 64 x
 * 128 with two or four stages, a register-staged 128 x 128); up to 1.05 where K <= 256 makes a launch one of stores (2067 x 256 ->
 * 12928 27.0 / 28.5).  Where each is the best (us; in brackets the kernels before):
 *   128 x 256, two workgroups to a unit: many tiles (4096 x 2560 -> 13824 117; 128 x 192 122, 128 x 128 129, 64 x 128 151 [149]);
 *   128 x 192, two workgroups: where it fills the units better (1616 x 4800 -> 5154 48.9; 128 x 256 58.0, 128 x 128 54.2, 64 x 128
 *     59.0 [62.8]);
 *   128 x 192, one workgroup with four stages: at most one tile to a unit (2048 x 6912 -> 2560 37.2; 128 x 256 44.5, 128 x 128 40.6,
 *     64 x 128 42.2 [43.2]);
 *   128 x 128, two workgroups: two tiles to a unit (2048 x 2560 -> 3840 22.3; 128 x 256 25.4, 64 x 128 25.7 [25.2]), and where it ends
 *     evenly (2048 x 2560 -> 13824 70.2; 128 x 192 69.0, 128 x 256 74.8, 64 x 128 86.8 [79.0]);
 *   64 x 128, four workgroups: few tokens (512 x 2560 -> 3840 10.4; 128 x 128 12.5 [14.1]);
 *   the k loop split over the waves (bl_gemm_ksplit): fewer tiles than units (512 tiles of 64 x 32 in a round; 128 x 2560 -> 3840
 *     6.6, 64 x 128 8.7). */
static constexpr bl_tile_cost bl_plain_cost[5] = {{128, 256, 4.55f, .616f, .093f, .252f, .515f}, {128, 192, 4.05f, .508f, .110f, .317f, .505f},
                                               {128, 192, 2.96f, .564f, 0.0f, 2.01f, .465f}, {128, 128, 4.16f, .351f, .066f, 0.0f, .553f},
                                               {64, 128, 3.70f, .225f, .068f, 0.0f, .492f}};
/* The split k loop's time (us): rounds of 512 workgroups, two to a unit, whose k steps share its matrix cores, and what an XCD reads
 * (361 shapes in the order that is launched: within 2.7 % in the mean, 15 % at most). */
static inline float bl_ksplit_us(int m, int n, int k) {
    const int64_t tiles = (int64_t)((m + 63) / 64) * ((n + 31) / 32);
    const float rounds = (float)((tiles + 511) / 512), steps = (float)((k + GP_BK - 1) / GP_BK);
    return 1.97f + rounds * (steps * (tiles > 256 ? .174f : .105f) + 1.83f) + .50e-6f * (float)bl_ksplit_order_of(m, n).bytes * (float)k +
           .94e-6f * (float)m * (float)n;
}
/* The kernel of a plain product: its place in the list of costs, or 5, the split k loop.  The lists are fitted with fp32 output alone;
 * against the split k loop the tiles take longer with a residual (it has that at hand when its sums are ready: 663 x 781 -> 1088
 * 5.9 us, 64 x 128 tiles 8.0), with both outputs (which it writes at once: 436 x 576 -> 2330 6.2 / 6.9), and where rows of fp32 start inside
 * a line, which the few tiles of such a launch write past the caches in parts and it does not (909 x 256 -> 460 4.4 / 5.0, 293 x 448 ->
 * 3082 5.2 / 5.7, 357 x 256 -> 1001 4.4 / 4.9; but 242 x 256 -> 4032 5.0 / 4.7). */
static inline int bl_plain_kernel(int m, int n, int k, bool residual, bool acc, bool y) {
    float us;
    const int kernel = bl_least(bl_plain_cost, m, n, k, &us);
    us += residual ? 2.0f : acc && y ? 0.8f : y && n % 16 != 0 ? 0.5f : 0.0f;
    return bl_ksplit_us(m, n, k) < us ? 5 : kernel;
}

/* Whether the tile kernels store fp32 output past the caches (non-temporal).  Whole and half lines gain by it (2048 x 2560 -> 13840 66.7 us,
 * plain stores 69.3).  Rows that start inside a line write lines in parts: such a store goes to memory as a part once the output
 * outgrows the L2s, from about 5 M values (2106 x 256 -> 3705 15.9 / 10.4, 4072 x 640 -> 1915 17.2 / 13.3, 2242 x 192 -> 2986 12.4 / 10.4, 3812 x 677 ->
 * 6613 51.1 / 35.0), and up to there gains where the k loop is long (422 x 1280 -> 4751 8.3 / 8.9, 387 x 2560 -> 7778 14.2 / 14.9) and loses
 * less where it is short (734 x 256 -> 2034 5.7 / 5.3).  Beside an int32 output only whole and half lines. */
static constexpr bool bl_past_caches(int m, int n, bool acc) { return n % 16 == 0 || (!acc && (int64_t)m * n <= (4 << 20)); }

/* The tile of a fused epilogue, by the same estimate (gate: tiles of outputs), fitted to 140 shapes; over 210 others the choice takes
 * 1.005 times the time of the best, .78 (residual) and .87 (gate) of that of the 128 x 128 and 64 x 128 tiles before it.  us [before]:
 *   residual 4096 x 2560 -> 2560 40 [45], 4096 x 6912 -> 2560 86 [93], 1000 x 2560 -> 2560 15.9 [20.4], 128 x 6912 -> 2560 20.9 [26.8];
 *   gate 2560 -> 13824 at 4096 tokens 120 [142], 2048 69 [72], 1500 49 [65], 65 17.6 [18.3].
 * Slower than before: the gate at 834 x 256 -> 3328 6.3 [6.0], 199 x 256 -> 6144 7.9 [7.7], 3736 x 1664 -> 2176 21.2 [20.0]. */
static constexpr bl_tile_cost bl_residual_cost[3] = {{128, 256, 0.0f, .450f, .207f, 8.97f, .929f}, {128, 128, 3.26f, .266f, .103f, 3.68f, .988f},
                                                  {64, 128, 3.84f, .193f, .112f, .966f, 1.17f}};
static constexpr bl_tile_cost bl_gate_cost[2] = {{128, 128, 6.24f, .614f, .072f, 0.0f, .756f}, {64, 64, 4.52f, .230f, .056f, 0.0f, .872f}};
static inline int bl_residual_kernel(int m, int n, int k) { return bl_least(bl_residual_cost, m, n, k); }
static inline int bl_gate_kernel(int m, int n, int k) { return bl_least(bl_gate_cost, m, n / 2, k); }

/* Whether a table of 33 to 48 tokens is walked by the tile kernel: entries = its tiles of 64 x 256, steps = the k steps of all of them,
 * chain = of the longest.  Not below 128 entries.  us: the tiles take a lone tile's chain, slower where units share two, or their even
 * share; the form with the tokens in LDS (two groups of them) a row's staging and its share.  LDS form / tiles over 33, 36, .. 48 tokens:
 * three layers of 2560 / 6912 27 - 35 / 33 - 35 (267 entries), four 34 - 42 / 34 - 36, eight 60 - 70 / 50; one of 4096 / 11008 29 - 31 / 36, two 48 -
 * 51 / 48 - 51, three 70 - 76 / 52; four of 2048 / 5632 25 - 31 / 28 - 29, eight 43 - 48 / 32; four of 896 / 2560 20 - 28 / 12.  Even within 10 %
 * either way: two layers of 2560 / 6912 (23 - 29 / 25), three of 2048 / 5632 (23 - 26 / 23 - 24). */
static inline bool bl_table_in_tiles(int64_t entries, int64_t steps, int64_t chain) {
    const float share = (float)steps / 256.0f, alone = (float)chain * (entries > 256 ? .58f : .39f);
    const float tiles = 2.0f + (alone > .72f * share ? alone : .72f * share), few = 18.0f + .35f * share, many = 4.0f + 1.05f * share;
    return entries >= 128 && tiles <= (few > many ? few : many);
}
