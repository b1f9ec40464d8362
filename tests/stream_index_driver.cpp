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

int main(int argc, char** argv) {
    if (argc < 2) return 2;
    if (!strcmp(argv[1], "activations")) {
        for (int64_t K = 1; K <= 20480; K += K < 2000 ? 1 : K % 64 == 0 ? 1 : 63) {
            activations<4>(K);
            activations<5>(K);
        }
    } else {
        return 2;
    }
    printf(bad ? "%ld outside\n" : "walk ok\n", bad);
    return bad != 0;
}
