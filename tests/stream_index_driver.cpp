/* Walks the index rules of the one-token stream (csrc/bl_stream_index.h) over the shapes that the library takes and
 * reports every read outside its row, matrix or vector.  argv[1]: activations | issue. */
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>

#include "bl_host.h"
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

/* The requests of one wave: row groups first .. first + mine - 1 of N rows of nchunks chunks, parts of lp loads, and
 * the one part more.  Cursor and lane offsets as in bl_stream_slice. */
static void wave(int N, int nchunks, int lp, int first, int mine) {
    const int shift = nchunks % 8 == 4 ? 4 : 0, parts = ((nchunks + shift + 7) / 8 + lp - 1) / lp, row_bytes = nchunks * 16;
    int irg = first, ipart = 0;
    for (int k = 0; k <= mine * parts; ++k) {
        const bool over = irg == first + mine;
        const int rows = N - irg * 8, at = ipart * lp * 128;
        const bl_part_window win = bl_part_of(rows, row_bytes, at, over);
        for (int lane = 0; lane < 64; ++lane) {
            const int r = ((lane >> 2) & 6) | (lane >> 5), u16 = (lane & 7) * 16 - (lane >> 5 ? shift * 16 : 0);
            const int end = std::max(r * row_bytes + row_bytes - 16 - at, 0);
            for (int i = 0; i < lp; ++i) {
                const int64_t x = (int64_t)irg * 8 * row_bytes + win.off + std::min(std::min(r * row_bytes + u16 + i * 128, end), win.limit);
                expect(x >= 0 && x + 16 <= (int64_t)N * row_bytes, "weights (N, chunks, row group, byte)", N, nchunks, irg, (long)x);
                /* a live lane reads its own chunk */
                const int chunk = ipart * lp * 8 + i * 8 + (lane & 7) - (lane >> 5 ? shift : 0);
                if (!over && irg * 8 + r < N && chunk >= 0 && chunk < nchunks)
                    expect(x == ((int64_t)irg * 8 + r) * row_bytes + chunk * 16, "wrong chunk", N, nchunks, irg, (long)x);
            }
            const int64_t v = (int64_t)irg * 8 + std::min(r, bl_last_residual(rows));
            expect(v >= 0 && v < N, "residual (N, chunks, row group, element)", N, nchunks, irg, (long)v);
            if (!over && irg * 8 + r < N) expect(v == irg * 8 + r, "wrong residual", N, nchunks, irg, (long)v);
        }
        if (!over && ++ipart == parts) {
            ipart = 0;
            ++irg;
        }
    }
}

int main(int argc, char** argv) {
    if (argc < 2) return 2;
    if (!strcmp(argv[1], "activations")) {
        for (int64_t K = 1; K <= 20480; K += K < 2000 ? 1 : K % 64 == 0 ? 1 : 63) {
            activations<4>(K);
            activations<5>(K);
        }
    } else if (!strcmp(argv[1], "issue")) {
        for (int nchunks : {1, 2, 3, 4, 5, 7, 8, 11, 12, 20, 23, 32, 36, 40, 44, 60, 87, 108, 132, 256, 320})
            for (int lp = 3; lp <= 5; ++lp)
                for (int N : {1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 29, 37, 64, 100, 2564, 5003}) {
                    const int units = (N + 7) / 8;
                    /* every slice of a small product; the last ones of a large one */
                    for (int ub = units > 9 ? units - 9 : 0; ub < units; ++ub)
                        for (int ue = ub + 1; ue <= units; ++ue)
                            for (int w = 0; w < 4; ++w) {
                                const int each = (ue - ub) >> 2, extra = (ue - ub) & 3;
                                wave(N, nchunks, lp, ub + w * each + std::min(w, extra), each + (w < extra ? 1 : 0));
                            }
                }
    } else {
        return 2;
    }
    printf(bad ? "%ld outside\n" : "walk ok\n", bad);
    return bad != 0;
}
