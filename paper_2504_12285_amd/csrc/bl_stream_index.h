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

/* One part of a row group of eight weight rows, `rows` rows in front of the matrix's end; `over`: behind the
 * wave's last row group, where the loop requests one part more than it multiplies (every lane reads the first bytes of the row
 * group in front of it).  Byte offsets from the row group: where the part starts, and, from there, the last 16 bytes that
 * may be read.  `at`: first byte of the part in its row. */
struct bl_part_window {
    int off, limit;
};
BL_INDEX bl_part_window bl_part_of(int rows, int row_bytes, int at, bool over) {
    const int limit = rows >= 8 ? 0x7FFFFFFF : rows * row_bytes - 16 - at;
    return {over ? -8 * row_bytes : limit < 0 ? 0 : at, over || limit < 0 ? 0 : limit};
}
/* The last row's residual value, from the row group's first one; behind the wave's last row group too, where that may
 * be the matrix's end (the value is not used). */
BL_INDEX int bl_last_residual(int rows) { return rows - 1; }
