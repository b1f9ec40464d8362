/* Internal device helpers shared by the HIP kernels of the BitLinear library
 * (not part of the public boundary).  gfx950 only: 64-lane wavefronts. */
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bitlinear.h"

typedef int bl_v4i __attribute__((ext_vector_type(4)));
typedef int bl_v16i __attribute__((ext_vector_type(16)));

typedef float bl_v4f __attribute__((ext_vector_type(4)));
typedef uint32_t bl_v2u __attribute__((ext_vector_type(2)));

#define BL_WAVE 64

/* A pointer that reached a kernel inside a structure is generic to the compiler once it has been
 * pinned or read from memory: its loads become flat_* instructions, which count on both counters
 * and are waited for all at once.  Casting it to the global address space gives global_* with
 * exact waits. */
#define BL_G __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ T BL_G* bl_g(T* p) { return (T BL_G*)p; }
template <typename T>
__device__ __forceinline__ const T BL_G* bl_gc(const void* p) { return (const T BL_G*)p; }

/* bf16 bit pattern -> fp32 (exact). */
__device__ __forceinline__ float bl_bf16_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

/* Two fp32 -> packed bf16 bit patterns (a in the low half), round to nearest even: one
 * instruction, the bits of that definition for every finite input (tests/test_gpu_rounding.py goes through all). */
typedef __bf16 bl_v2bf __attribute__((ext_vector_type(2)));
typedef float bl_v2f __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bl_pack2_bf16(float a, float b) {
    const bl_v2f v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bl_v2bf));
}

/* Correctly rounded fp32 quotient (IEEE division: about ten fp32 instructions; by way of an fp64
 * quotient, the same bits, it took about three times as long). */
__device__ __forceinline__ float bl_div_rn(float a, float b) { return a / b; }

/* DPP cross-lane moves inside a row of 16 lanes (old value = 0 for disabled lanes). */
template <int CTRL>
__device__ __forceinline__ int bl_dpp(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
#define BL_DPP_QUAD_XOR1 0xB1   /* quad_perm [1,0,3,2] */
#define BL_DPP_QUAD_XOR2 0x4E   /* quad_perm [2,3,0,1] */
#define BL_DPP_ROW_HALF_MIRROR 0x141
#define BL_DPP_ROW_MIRROR 0x140

/* Sum over aligned groups of G lanes (G = 4, 8 or 16), result in every lane of
 * the group.  DPP only: quad butterflies, then half-row / row mirrors (after a
 * quad sum all four lanes of a quad agree, so a mirror pairs distinct quads). */
template <int G>
__device__ __forceinline__ int bl_group_sum(int v) {
    static_assert(G == 1 || G == 2 || G == 4 || G == 8 || G == 16, "group size");
    if (G >= 2) v += bl_dpp<BL_DPP_QUAD_XOR1>(v);
    if (G >= 4) v += bl_dpp<BL_DPP_QUAD_XOR2>(v);
    if (G >= 8) v += bl_dpp<BL_DPP_ROW_HALF_MIRROR>(v);
    if (G >= 16) v += bl_dpp<BL_DPP_ROW_MIRROR>(v);
    return v;
}

/* Sum over the 64 lanes, the same in every lane. */
__device__ __forceinline__ int bl_wave_sum(int v) {
    v = bl_group_sum<16>(v);
    return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
           (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}
/* Maximum of NON-NEGATIVE floats (they order like their bit patterns: no canonicalising moves),
 * over 16 lanes and over the 64 lanes of a wave: DPP inside the rows of 16, then four readlanes. */
__device__ __forceinline__ float bl_max_pos(float a, float b) {
    const uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
    return __uint_as_float(x > y ? x : y);
}
template <int CTRL>
__device__ __forceinline__ float bl_dppf(float v) {
    return __int_as_float(bl_dpp<CTRL>(__float_as_int(v)));
}
__device__ __forceinline__ float bl_lane_f(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ float bl_row_max(float v) {
    v = bl_max_pos(v, bl_dppf<BL_DPP_QUAD_XOR1>(v));
    v = bl_max_pos(v, bl_dppf<BL_DPP_QUAD_XOR2>(v));
    v = bl_max_pos(v, bl_dppf<BL_DPP_ROW_HALF_MIRROR>(v));
    return bl_max_pos(v, bl_dppf<BL_DPP_ROW_MIRROR>(v));
}
__device__ __forceinline__ float bl_wave_max(float v) {
    v = bl_row_max(v);
    return bl_max_pos(bl_max_pos(bl_lane_f(v, 0), bl_lane_f(v, 16)), bl_max_pos(bl_lane_f(v, 32), bl_lane_f(v, 48)));
}

/* 4x4 byte transpose of four dwords: out[s].byte[b] = in[b].byte[s]. */
__device__ __forceinline__ void bl_transpose4x4(uint32_t& a0, uint32_t& a1, uint32_t& a2, uint32_t& a3) {
    const uint32_t t0 = __builtin_amdgcn_perm(a1, a0, 0x05010400u);
    const uint32_t t1 = __builtin_amdgcn_perm(a1, a0, 0x07030602u);
    const uint32_t t2 = __builtin_amdgcn_perm(a3, a2, 0x05010400u);
    const uint32_t t3 = __builtin_amdgcn_perm(a3, a2, 0x07030602u);
    a0 = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
    a1 = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
    a2 = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
    a3 = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
}

/* Direct global->LDS loads (16 bytes per lane): the LDS destination is a wave-uniform
 * base, lane l's bytes land at base + 16*l.  They count on vmcnt like any load. */
typedef const __attribute__((address_space(1))) void* bl_gptr;
typedef __attribute__((address_space(3))) void* bl_lptr;

/* s_waitcnt vmcnt(n) only, n < 64: expcnt = 7, lgkmcnt = 15 left open (gfx9 encoding:
 * vmcnt bits 3:0 in imm[3:0], bits 5:4 in imm[15:14]) */
#define BL_WAIT_VM(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))
/* s_waitcnt lgkmcnt(0) only (vmcnt = 63 and expcnt = 7 left open): a wave's own LDS writes have
 * been performed.  A raw s_barrier does not imply it, so a wave that hands data to other waves
 * through LDS waits with this in front of the barrier. */
#define BL_WAIT_LGKM0() __builtin_amdgcn_s_waitcnt(0xC07F)

/* Waits until at most r stages of LOADS direct loads each are still in flight (r <= J). */
template <int J, int LOADS>
__device__ __forceinline__ void bl_wait_stages(int r) {
    if (r >= J) {
        BL_WAIT_VM(J * LOADS);
    } else {
        if constexpr (J > 0) bl_wait_stages<J - 1, LOADS>(r);
    }
}

/* Expand one packed word (16 weights, layout-1 digit order) into the sixteen
 * int8 codes of 16 consecutive k: three shifts and four masks. */
__device__ __forceinline__ bl_v4i bl_unpack16(uint32_t p) {
    bl_v4i b;
    b[0] = (int)(p & 0x03030303u);
    b[1] = (int)((p >> 2) & 0x03030303u);
    b[2] = (int)((p >> 4) & 0x03030303u);
    b[3] = (int)((p >> 6) & 0x03030303u);
    return b;
}

/* A packed word of layout 0 (weight i at bits 2i) in layout-1 order (at bits 8(i%4) + 2(i/4)): the
 * transpose of a 4 x 4 matrix of bit pairs, two delta swaps of six cheap instructions each. */
__device__ __forceinline__ uint32_t bl_word_to_k16(uint32_t p) {
    uint32_t t = ((p >> 12) ^ p) & 0x0000F0F0u;
    p = p ^ t ^ (t << 12);
    t = ((p >> 6) ^ p) & 0x00CC00CCu;
    return p ^ t ^ (t << 6);
}

/* Wait for in-flight matrix-core results before ordinary vector instructions
 * read an accumulator.  The hardware has no interlock for that read, and the
 * compiler's wait-state count for the gfx950 16x16x64 int8 MFMA proved too
 * short on hardware (the last result rows were read before they were written).
 * 32 idle issue cycles cover the longest (16-pass) MFMA; the scheduling
 * barriers keep every MFMA before and every reader after this point. */
__device__ __forceinline__ void bl_mfma_fence() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
