/* Walks the index rules of the one-token stream (csrc/bl_stream_index.h) over the shapes that the library takes and
 * reports every read outside its row, matrix or vector; and the shares of the workgroups (csrc/bl_stream_cut.h).
 * argv[1]: activations | issue | cut. */
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "bl_host.h"
#include "bl_stream_cut.h"
#include "bl_stream_index.h"

static long bad = 0;
static void expect(bool ok, const char* what, long a, long b, long c, long d) {
    if (!ok && ++bad <= 20) printf("%s: %ld %ld %ld %ld\n", what, a, b, c, d);
}

/* Every word that a thread stages or requests ahead (words 0 .. 4 * chunks - 1 of the packed row). */
template <int UD>
static void activations(int64_t K) {
    const int dwords = (int)(bl_kpad(K) / 4);
    const int words = (int)(UD == 5 ? bl_kpad5(K) / 20 : bl_kpad(K) / 16);
    for (int wd = 0; wd < words; ++wd)
        for (int i = 0; i < UD; ++i) {
            const int valid = bl_word_valid<UD>(wd, dwords);
            const int at = bl_word_first<UD>(wd, dwords) + bl_word_dword(i, valid);
            expect(at >= 0 && at < dwords, "activation (words per unit, K, word, dword)", UD, (long)K, wd, at);
            if (wd * UD + i < dwords) expect(i < valid && at == wd * UD + i, "wrong activation", UD, (long)K, wd, at);
            else expect(i >= valid, "not masked", UD, (long)K, wd, i);
        }
}

/* The requests of one wave: row groups first .. first + mine - 1 of N rows of n chunks, parts of lp loads, and the one
 * part more.  Cursor and lane offsets as in bl_stream_slice. */
static void wave(int N, int n, int lq, int mod, int lead, int lp, int first, int mine) {
    const int parts = ((n + lead + 7) / 8 + lp - 1) / lp, row_bytes = n * 16, bias = lead * 16;
    int irg = first, ipart = 0, rows = N - bl_group_base(first, lq);
    for (int k = 0; k <= mine * parts; ++k) {
        const bool over = irg == first + mine;
        const int at = ipart * lp * 128, base_row = N - rows;
        const int limit = over ? 0 : bl_part_limit(rows, row_bytes, at, bias, lq);
        const int back = bl_group_next(irg - 1, lq);
        const int64_t base = (int64_t)base_row * row_bytes - bias + (over ? bias - back * row_bytes : at);
        for (int lane = 0; lane < 64; ++lane) {
            const int h = lane >> 5, u = lane & 7, r = bl_group_row((lane >> 3) & 3, h, lq), shift = bl_group_shift(irg, h, lq, mod);
            const int end = r * row_bytes + row_bytes - 16 + bias - at;
            for (int i = 0; i < lp; ++i) {
                const int off = std::min(std::min(r * row_bytes + (u - shift) * 16 + bias + i * 128, end), limit);
                const int64_t x = base + (uint32_t)off;
                expect(x >= 0 && x + 16 <= (int64_t)N * row_bytes, "weights (N, chunks, row group, byte)", N, n, irg, (long)x);
                /* a live lane reads its own chunk, shifted ones whole lines */
                const int chunk = ipart * lp * 8 + i * 8 + u - shift;
                if (!over && base_row + r < N && chunk >= 0 && chunk < n)
                    expect(x == ((int64_t)base_row + r) * row_bytes + chunk * 16, "wrong chunk", N, n, irg, (long)x);
                if (lead || n % 8 == 0) expect((n * (base_row + r) + chunk) % 8 == u || over, "not a line", N, n, irg, chunk);
            }
            const int64_t v = base_row + std::min(r, over ? -back : rows - 1);
            expect(v >= 0 && v < N, "residual (N, chunks, row group, element)", N, n, irg, (long)v);
            if (!over && base_row + r < N) expect(v == base_row + r, "wrong residual", N, n, irg, (long)v);
        }
        if (!over && ++ipart == parts) {
            rows -= bl_group_next(irg, lq);
            ipart = 0;
            ++irg;
        }
    }
}
/* Every row is in one row group. */
static void groups(int N, int lq) {
    std::vector<int> seen(N, 0);
    for (int g = 0; g < bl_groups(N, lq); ++g) {
        expect(bl_group_base(g, lq) < N, "empty row group", N, lq, g, bl_group_base(g, lq));
        expect(bl_group_base(g + 1, lq) == bl_group_base(g, lq) + bl_group_next(g, lq), "next row group", N, lq, g, 0);
        for (int i = 0; i < 8; ++i) {
            const int row = bl_group_base(g, lq) + bl_group_row(i >> 1, i & 1, lq);
            if (row < N) ++seen[row];
        }
    }
    for (int r = 0; r < N; ++r) expect(seen[r] == 1, "row", N, lq, r, seen[r]);
}

/* Slices are contiguous, cover the table once, and none costs more than a fair share (a quarter more: the bisection is taken for a fifth less),
 * a row group for each wave and two entries (its own and the one that stopped its neighbour). */
static void cut(const std::vector<int>& units, const std::vector<int64_t>& uc, const std::vector<int64_t>& ec, int blocks, int waves) {
    const std::vector<bl_cut_pos> wg = bl_cut_slices(units, uc, ec, blocks, waves);
    const int count = (int)units.size();
    int64_t all = 0, uc_max = 0, ec_max = 0;
    for (int i = 0; i < count; ++i) {
        all += units[i] * uc[i] + ec[i];
        uc_max = std::max(uc_max, uc[i]);
        ec_max = std::max(ec_max, ec[i]);
    }
    int pi = 0, unit = 0;
    for (int b = 0; b < blocks; ++b) {
        int64_t cost = 0;
        /* as the kernels walk it */
        for (int p = wg[b].x; p <= wg[b + 1].x; ++p) {
            if (p == wg[b + 1].x && wg[b + 1].y == 0) break;
            const int ub = p == wg[b].x ? wg[b].y : 0, ue = p == wg[b + 1].x ? wg[b + 1].y : units[p];
            if (ub >= ue) continue;
            if (unit == units[pi]) ++pi, unit = 0;
            expect(p == pi && ub == unit, "gap (products, blocks, block, product)", count, blocks, b, p);
            unit = ue;
            cost += ec[p] + (ue - ub) * uc[p];
        }
        expect(cost <= all / blocks / 4 * 5 + uc_max * waves + 2 * ec_max + 1, "share (products, blocks, block, cost)", count, blocks, b, (long)cost);
    }
    expect(pi == count - 1 && unit == units[pi], "rest", count, blocks, pi, unit);
}

int main(int argc, char** argv) {
    if (argc < 2) return 2;
    if (!strcmp(argv[1], "activations")) {
        for (int64_t K = 1; K <= 20480; K += K < 2000 ? 1 : K % 64 == 0 ? 1 : 63) {
            activations<4>(K);
            activations<5>(K);
        }
    } else if (!strcmp(argv[1], "issue")) {
        for (int n : {1, 2, 3, 4, 5, 7, 8, 11, 12, 20, 23, 32, 36, 40, 43, 44, 50, 60, 62, 87, 108, 113, 132, 253, 256, 317, 320})
            for (int form = 0; form < 2; ++form) {
                const int lq = form == 0 ? 0 : bl_row_classes(n), mod = form == 0 && n % 4 ? 0 : n % 8, lead = bl_row_lead(mod);
                for (int lp = 3; lp <= 5; ++lp)
                    for (int N : {1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 29, 37, 64, 100, 2564, 5003}) {
                        const int units = bl_groups(N, lq);
                        /* every slice of a small product; the last ones of a large one */
                        for (int ub = units > 9 ? units - 9 : 0; ub < units; ++ub)
                            for (int ue = ub + 1; ue <= units; ++ue)
                                for (int w = 0; w < 4; ++w) {
                                    const int each = (ue - ub) >> 2, extra = (ue - ub) & 3;
                                    wave(N, n, lq, mod, lead, lp, ub + w * each + std::min(w, extra), each + (w < extra ? 1 : 0));
                                }
                    }
            }
        for (int lq = 0; lq < 3; ++lq)
            for (int N = 1; N < 300; ++N) groups(N, lq);
    } else if (!strcmp(argv[1], "cut")) {
        cut(std::vector<int>(12, 512), std::vector<int64_t>(12, 9472), std::vector<int64_t>(12, 36 << 10), 1024, 4);
        cut(std::vector<int>(54, 512), std::vector<int64_t>(54, 8960), std::vector<int64_t>(54, 36 << 10), 1024, 4);
        cut({1728}, {128}, {36 << 10}, 432, 4);
        cut({1}, {128}, {36 << 10}, 1, 4);
        uint32_t x = 12345;
        auto rnd = [&x](int lo, int hi) {
            x = x * 1664525u + 1013904223u;
            return lo + (int)((uint64_t)(x >> 8) * (uint64_t)(hi - lo + 1) >> 24);
        };
        for (int k = 0; k < 400; ++k) {
            const int count = rnd(1, k % 4 ? 40 : 1024);
            std::vector<int> units(count);
            std::vector<int64_t> uc(count), ec(count);
            int64_t total = 0;
            for (int i = 0; i < count; ++i) {
                units[i] = rnd(1, 4000) >> rnd(0, 10);
                units[i] += units[i] == 0;
                uc[i] = (int64_t)rnd(1, 320) * 128;
                ec[i] = (int64_t)rnd(0, 36) << 10;
                total += units[i];
            }
            cut(units, uc, ec, (int)std::min<int64_t>(rnd(1, 4096), (total + 3) / 4), k % 2 ? 4 : 8);
        }
    } else {
        return 2;
    }
    printf(bad ? "%ld outside\n" : "walk ok\n", bad);
    return bad != 0;
}
