/* Where the one-token stream reads (bl_stream.hip), apart from the kernels so that a host program can walk every
 * index (tests/stream_index_driver.cpp). */
#pragma once

#if defined(__HIPCC__)
#define BL_INDEX __host__ __device__ __forceinline__
#else
#define BL_INDEX static inline
#endif

/* A packed word of five per byte meets five dwords of four activations; 2-bit words meet four.  The packed row is a
 * multiple of 80 weights, the activation row one of 64: its last words may end behind it (up to three of them lie
 * behind it as a whole: K = 256, word 13 of 16).  First dword of word wd's activations, with those that it has: the
 * row's first one where it has none. */
template <int UD>
BL_INDEX int bl_word_first(int wd, int dwords) { return wd * UD < dwords ? wd * UD : 0; }
template <int UD>
BL_INDEX int bl_word_valid(int wd, int dwords) { return dwords - wd * UD; }
/* Dword i of the word, from its first one; what is not valid is read as the first again and not used. */
BL_INDEX int bl_word_dword(int i, int valid) { return i < valid ? i : 0; }

/* Row groups of eight weight rows.  A row of `chunks` 16-byte chunks starts (chunks * row) % 8 chunks behind the start of a
 * 128-byte line.  A wave-wide load covers eight lines where every row is read from the start of its line, but the products allow two
 * such shifts in a load (even lanes' half and odd one).  So the rows of a group are those of two classes: with 2^lq groups to a
 * block of 8 * 2^lq rows, group g holds rows base + 2 * 2^lq * j + h (j = 0 .. 3, h = 0, 1), base = bl_group_base.  lq = 0: eight
 * consecutive rows. */
BL_INDEX int bl_group_base(int g, int lq) { return ((g >> lq) << (3 + lq)) + 2 * (g & ((1 << lq) - 1)); }
BL_INDEX int bl_group_row(int j, int h, int lq) { return (j << (1 + lq)) + h; }
BL_INDEX int bl_group_span(int lq) { return (6 << lq) + 2; }              /* rows from the first one to behind the last */
BL_INDEX int bl_groups(int N, int lq) {
    const int block = 8 << lq, rest = ((N & (block - 1)) + 1) >> 1;
    return ((N / block) << lq) + (rest < 1 << lq ? rest : 1 << lq);
}
/* Rows from this group's base to the next one's. */
BL_INDEX int bl_group_next(int g, int lq) { return ((g + 1) & ((1 << lq) - 1)) ? 2 : bl_group_span(lq); }
/* Chunks that the loads of half h of group g start in front of their rows, with mod = chunks % 8 (0: rows that are not
 * shifted), and the largest of them. */
BL_INDEX int bl_row_classes(int chunks) { return chunks % 4 == 0 ? 0 : chunks % 2 == 0 ? 1 : 2; }
BL_INDEX int bl_row_lead(int mod) { return mod == 0 ? 0 : mod % 4 == 0 ? 4 : mod % 2 == 0 ? 6 : 7; }
BL_INDEX int bl_group_shift(int g, int h, int lq, int mod) { return (mod * (2 * (g & ((1 << lq) - 1)) + h)) & 7; }

/* The lanes' byte offsets count from `bias` = 16 * lead bytes in front of the part's place in the group's first row, so that they
 * are never negative; the last 16 bytes that may be read of a part `at` bytes into its rows, `rows` rows in front of the matrix's end. */
BL_INDEX int bl_part_limit(int rows, int row_bytes, int at, int bias, int lq) {
    return rows >= bl_group_span(lq) ? 0x7FFFFFFF : rows * row_bytes - 16 - at + bias;
}
