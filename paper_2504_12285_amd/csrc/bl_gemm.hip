/* Prefill-side W1.58A8 product (Section 5.1 of the BitNet b1.58 2B4T report):
 * a dense int8 contraction on the CDNA4 matrix cores.  Packed 2-bit weight
 * tiles go HBM -> LDS still packed (a quarter of the int8 bytes), each wave
 * expands the words it needs to int8 in registers with shift+mask right before
 * v_mfma_i32_32x32x32_i8, and the activations stream through LDS as int8.
 * Codes c = Wt + 1 are contracted as they are; the epilogue subtracts
 * rowsum[m] = sum_k q[m][k] (exact int32 identity), then rescales.
 */
#include "bl_device.h"
#include "bl_gemm_pipe.h"
#include "bl_host.h"

#include <atomic>
#include <type_traits>

/* ---- tile kernel ------------------------------------------------------------
 * BM x BN output tile per workgroup, k step 128, STAGES LDS stages filled by direct
 * global->LDS loads (no register staging) ahead of the matrix cores; one barrier per
 * k step.  WM x WN waves.
 *
 * LDS stage = A part (BM rows x 128 int8, 16-byte units XOR-swizzled by
 * (row/2)%8) + W part (BN rows x 32 packed bytes = two units, swapped by row/8%2): with these
 * two patterns sixteen consecutive lanes of a ds_read_b128 fall on sixteen different 16-byte
 * bank groups (measured on a read-only loop, 8 waves per CU: 152 - 154 B/clk/CU against 113 - 116
 * for swizzles by row%8 and row/4%2, which are conflict-free only over eight lanes).
 * A direct load writes 64 consecutive units per wave, so the swizzle is applied
 * to the GLOBAL address each lane fetches, not to the LDS address.
 *
 * k mapping inside a k step: MFMA sub-step ks, lane half h  <->  the 16 k of
 * packed word 4h+ks (bytes 16*(4h+ks).. of the activation row).  Lane half h
 * therefore needs exactly unit h of a weight row: one ds_read_b128 per 32 rows
 * and k step, and one per (32 rows, sub-step) for the activations.
 *
 * K a multiple of 64 (HALF: an odd one); layout 1, or 0 through bl_word_to_k16. */
#define G3_BK 128


/* EPI: 0 = plain epilogue (int32 and/or fp32 outputs, optional residual); 1 = fused producer
 * epilogue "residual": t = residual + product, written as fp32 (y, optional) and as bf16 (xb) with
 * the row maximum of |bf16(t)| folded into absmax[m]; 2 = "squared-ReLU gate": the tile's 128 weight
 * rows are 2 x 32 gate rows and the 2 x 32 matching up rows (n and N/2 + n), t = (relu(g)*relu(g))*u
 * for N/2 output columns, written as bf16 with its row maximum (Section 2: ReLU^2 in the FFN,
 * per-token absmax quantisation of the next BitLinear's input). */
/* TABLE: the persistent grid walks the tiles of a whole TABLE of products (device array `items`,
 * tile0[i] = first virtual tile of product i; at most BM token rows, so a tile is one block of
 * BN weight rows of one product) instead of the tiles of the one product in the arguments: the
 * batched decode of a stack of BitLinears in one launch whose weights are read once. */
/* DEFER: the fp32 outputs of a tile are not stored in a burst behind its k loop (every workgroup of
 * a launch reaches that point together, the chip then writes at the HBM rate while its matrix cores
 * idle: measured 19 - 23 thousand clocks of stores per 128 x 128 tile against 28 - 31 thousand of k
 * loop) but kept in registers and stored a few rows per k step during the NEXT tile of the
 * workgroup, behind that step's operand loads and behind its last MFMA (the matrix core works on
 * while the wave issues them).  Vector memory operations retire in order, so the wait in front of
 * the following step leaves exactly those stores in flight.  Interior tiles
 * with a following tile only; edge tiles and a workgroup's last tile store at once.  fp32 output
 * alone (no int32 output, no residual). */
/* HALF: K is an odd multiple of 64, so the last k step has only its first 64 columns: lane half 1 (the
 * second unit of a weight row) multiplies nothing there, its weights are set to zero and its loads go to
 * the step's first half (inside the row): 777 x 2999 -> 5003 with its quantiser 28.8 us against 38.4 on a
 * register-staged kernel of 128 x 128 tiles, one workgroup per compute unit.  (With deferred stores it spills nine
 * registers, and is the fastest form all the same: 4096 x 2112 -> 7040 76 us, 83 with stores at once.)  LAYOUT 0: a packed word is turned into layout-1 order in the
 * register before it is opened (bl_word_to_k16): 1000 x 2560 -> 3840 24.0 us against 29.2. */
template <int BM, int BN, int STAGES, int WM, int WN, int EPI, bool TABLE = false, bool DEFER = false, bool HALF = false, int LAYOUT = 1>
__global__ __launch_bounds__(WM * WN * 64, (DEFER && BM * BN >= 128 * 128 ? 2 : BM * BN >= 128 * 128 ? 3 : 4)) void bl_gemm_tile256(const uint8_t* __restrict__ packed,
                                                                const int8_t* __restrict__ q,
                                                                const int32_t* __restrict__ rowsum,
                                                                const float* __restrict__ beta,
                                                                const float* __restrict__ scale, int M, int N,
                                                                int K, int tiles_m, int tiles_n, int gm, int band,
                                                                int vgrid, const float* __restrict__ residual,
                                                                int32_t* __restrict__ acc, float* __restrict__ y,
                                                                uint16_t* __restrict__ xb, int* __restrict__ absmax,
                                                                long long* __restrict__ stamps,
                                                                const bl_tile_item* __restrict__ items,
                                                                const int* __restrict__ tile0, int nitems,
                                                                const int* __restrict__ wg_start,
                                                                const int* __restrict__ tile_list) {
    static_assert(!TABLE || EPI == 0, "the table walk has the plain epilogue only");
    static_assert(!(HALF || LAYOUT == 0) || (EPI == 0 && !TABLE), "ragged K and layout 0: plain products");
    static_assert(!DEFER || (EPI == 0 && !TABLE && STAGES == 2), "deferred stores: plain epilogue, two stages");
    static_assert(EPI != 2 || (BN == 128 && WN == 2 && BN / WN / 32 == 2), "the gate epilogue pairs ni = 0 with ni = 1");
    constexpr int NW = WM * WN, THREADS = NW * 64;
    constexpr int G3_BM = BM, G3_A_BYTES = BM * G3_BK;
    constexpr int G3_W_BYTES = BN * G3_BK / 4, G3_STAGE_BYTES = G3_A_BYTES + G3_W_BYTES;
    constexpr int MI = G3_BM / WM / 32, NI = BN / WN / 32;
    constexpr int A_LOADS = G3_A_BYTES / 16 / THREADS;      /* direct loads per thread and stage */
    constexpr int W_LOADS = G3_W_BYTES / 16 / THREADS;
    constexpr int LOADS = A_LOADS + W_LOADS;
    static_assert((STAGES - 2) * LOADS < 64, "vmcnt is a 6-bit count");
    static_assert(THREADS >= BM, "one thread per tile row fetches the row terms");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    /* behind the stages: the per-row terms of the tile in flight (row sum, beta*scale) */
    /* (DEFER: two sets, the second for the tile whose stores are still pending) */
    int* const rs_base = (int*)(smem + STAGES * G3_STAGE_BYTES);
    int* rs_s = rs_base;
    float* cf_s = (float*)(rs_base + G3_BM);
    /* (one product in 64 x 128 tiles: the wave's number as a scalar, so that where the direct loads write is scalar
     * arithmetic, 1 - 2 %; the table of products loses 2 % by it, the 128 x 128 kernels nothing to 2 %) */
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = BM < 128 && !TABLE ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
    const int l32 = lane & 31, h = lane >> 5;
    const int wm0 = (wave / WN) * (MI * 32), wn0 = (wave % WN) * (NI * 32);
    /* fixed for the launch, or (TABLE) those of the product whose tile is set up next */
    int kb = K / 4;
    int steps = HALF ? (K + G3_BK - 1) / G3_BK : K / G3_BK;
    bool want_cf = EPI != 0 || y != nullptr;            /* the fused epilogues always rescale */
    float bt = (!TABLE && want_cf) ? *beta : 0.0f;
    /* what the epilogue of the tile in flight stores to (TABLE: set when that tile was set up) */
    int eN = N;
    /* (cast to the global address space: read from the table they would be generic, see BL_G) */
    const float BL_G* eres = bl_gc<float>(residual);
    int32_t BL_G* eacc = bl_g(acc);
    float BL_G* ey = bl_g(y);
    const int32_t BL_G* rowsum_g = bl_gc<int32_t>(rowsum);
    const float BL_G* scale_g = bl_gc<float>(scale);
    int nN = N, nsteps = steps;
    const float BL_G* nres = eres;
    int32_t BL_G* nacc = eacc;
    float BL_G* ny = ey;
    auto load_item = [&](int vb, int& tn) {
        int lo = 0, hi = nitems - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tile0[mid] <= vb) lo = mid; else hi = mid - 1;
        }
        const bl_tile_item it = items[lo];
        tn = vb - tile0[lo];
        packed = it.packed;
        q = it.q;
        rowsum_g = bl_gc<int32_t>(it.rowsum);
        scale_g = bl_gc<float>(it.scale);
        N = nN = it.N;
        K = it.K;
        kb = K / 4;
        nsteps = K / G3_BK;
        nres = bl_gc<float>(it.residual);
        nacc = bl_g(it.acc);
        ny = bl_g(it.y);
        want_cf = it.y != nullptr;
        bt = want_cf ? *bl_gc<float>(it.beta) : 0.0f;
    };

    /* XCD-aware tile order: workgroup L runs on XCD L%8.  The row tiles are cut into bands so narrow that
     * a band's activation panel stays in an XCD's 4 MB L2 while its weight tiles stream through, row tiles
     * fastest.  Either a rectangle per XCD (gm bands x 8 / gm column blocks), or (gm = 0) the tiles are
     * numbered band by band and each XCD takes one eighth of the sequence, so that the XCDs are even whatever
     * the tile counts; the host chooses.  The grid is persistent: a workgroup takes virtual blocks
     * vb = blockIdx.x, + gridDim.x, .. (gridDim.x is a multiple of 8, so it stays on its XCD's share). */
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
    int vend = vgrid;
    if constexpr (TABLE) vend = wg_start[blockIdx.x + 1];
    /* the next virtual block of this workgroup that maps to a real tile, or -1 */
    auto next_tile = [&](int vb, int& tm, int& tn) {
        if constexpr (TABLE) {                      /* vb: position in this workgroup's tile list */
            if (vb >= vend) return -1;
            tm = 0;
            load_item(tile_list[vb], tn);
            return vb;
        }
        for (; vb < vgrid; vb += (int)gridDim.x)
            if (tile_of(vb, tm, tn)) return vb;
        return -1;
    };

    /* per-lane global sources of the direct loads of the tile (tm, tn) */
    const uint8_t* asrc[A_LOADS];
    const uint8_t* wsrc[W_LOADS];
    int row_rs = 0;
    float row_cf = 0.0f;
    auto setup = [&](int tm, int tn) {
        const int m0 = tm * G3_BM, n0 = tn * BN;
#pragma unroll
        for (int j = 0; j < A_LOADS; ++j) {
            const int row = (j * NW + wave) * 8 + (lane >> 3);          /* row of the tile */
            const int u = (lane & 7) ^ ((row >> 1) & 7);
            int m = m0 + row;
            if (m >= M) m = M - 1;
            asrc[j] = (const uint8_t*)q + (int64_t)m * K + u * 16;
        }
        const int u = (lane & 1) ^ ((lane >> 4) & 1);
#pragma unroll
        for (int j = 0; j < W_LOADS; ++j) {
            const int trow = (j * NW + wave) * 32 + (lane >> 1);        /* row of the weight tile */
            int n = n0 + trow;
            if (EPI == 2)   /* tile rows [64w, 64w+32) = gate rows, [64w+32, 64w+64) = the matching up rows */
                n = ((trow >> 5) & 1) * (N / 2) + tn * (BN / 2) + (trow >> 6) * 32 + (trow & 31);
            if (n >= N) n = N - 1;
            wsrc[j] = packed + (int64_t)n * kb + u * 16;
        }
        /* the tile's per-row terms travel in two registers until the epilogue (a load there
         * would put a memory round trip between the last MFMA and the first store) */
        if (tid < G3_BM) {
            const int m = m0 + tid;
            row_rs = m < M ? rowsum_g[m] : 0;
            row_cf = (want_cf && m < M) ? bt * scale_g[m] : 0.0f;
        }
    };
    auto issue = [&](int kk, int buf) {
        uint8_t* st = smem + buf * G3_STAGE_BYTES;
        /* HALF, last step: units of the second half are fetched from the first (bit 2 of a lane's unit
         * is that of lane ^ wave: the swizzle's row bits above it are the piece's number) */
        static_assert(NW % 2 == 0, "the parity of a piece is that of its wave");
        const bool last = HALF && kk == steps - 1;
        const int aback = last ? (((lane >> 2) ^ wave) & 1) * 64 : 0;
        const int wback = last ? ((lane ^ (lane >> 4)) & 1) * 16 : 0;
#pragma unroll
        for (int j = 0; j < A_LOADS; ++j)
            __builtin_amdgcn_global_load_lds((bl_gptr)(asrc[j] + ((int64_t)kk * G3_BK - aback)),
                                             (bl_lptr)(st + (j * NW + wave) * 1024), 16, 0, 0);
#pragma unroll
        for (int j = 0; j < W_LOADS; ++j)
            __builtin_amdgcn_global_load_lds((bl_gptr)(wsrc[j] + ((int64_t)kk * (G3_BK / 4) - wback)),
                                             (bl_lptr)(st + G3_A_BYTES + (j * NW + wave) * 1024), 16, 0, 0);
    };

    /* per-lane LDS read offsets (bytes) inside a stage */
    const int a_row_off = (wm0 + l32) * G3_BK;
    const int a_swz = (l32 >> 1) & 7;
    const int w_off = G3_A_BYTES + ((wn0 + l32) * 2 + (h ^ ((l32 >> 3) & 1))) * 16;

    int tm, tn;
    int vb = next_tile(TABLE ? wg_start[blockIdx.x] : (int)blockIdx.x, tm, tn);
    if (vb < 0) return;
    /* measurement hook: workgroup 0 counts shader clocks and wall-clock ticks over its lifetime
     * (a wave-uniform test, so the counts stay in scalar registers) */
    const bool stamp = stamps != nullptr && blockIdx.x == 0;
    long long c_start = 0, w_start = 0;
    if (stamp) {
        c_start = clock64();
        w_start = wall_clock64();
    }
    setup(tm, tn);
    if constexpr (TABLE) {
        steps = nsteps; eN = nN; eres = nres; eacc = nacc; ey = ny;
    }
    /* STAGES - 1 k steps are in flight ahead of the matrix cores: a k step of one workgroup
     * takes far less time than a load, so the depth, not the tile, hides the latency */
    for (int s0 = 0; s0 < STAGES - 1 && s0 < steps; ++s0) issue(s0, s0);

    /* DEFER: the accumulators of the workgroup's previous tile, where that tile lies and which set
     * of per-row terms is its; cset = the set of the tile in flight */
    bl_v16i P[MI][NI];
    bool have_prev = false;
    int pm0 = 0, pn0 = 0, pset = 0, cset = 0;
    constexpr int RPG = 4;                      /* rows of a lane per store group (2: equal; 1: more groups than k steps at K = 2560, slower) */
    constexpr int GROUPS = MI * 4 * (4 / RPG);  /* store groups of a tile: RPG of the rows 8 vq + 4 h + (0..3) of row block mi */
    constexpr int SPG = RPG * NI;               /* store instructions of a group */
    /* group g of the accumulators A of the tile at (sm0, sn0) -> y; masked: the tile may cross M or N */
    auto emit_rows = [&](const bl_v16i (&A)[MI][NI], const int g, const int sm0, const int sn0, const int set,
                         const bool masked) __attribute__((always_inline)) {
        const int mi = g / 4, vq = g % 4;
        const int* rs_p = rs_base + set * 2 * G3_BM;
        const float* cf_p = (const float*)(rs_p + G3_BM);
        /* (the row is hidden from the compiler here: it would otherwise keep the 64-bit addresses of
         * all 16 * MI * NI stores of a lane in registers across the k loop) */
        int mlb = wm0 + mi * 32 + vq * 8 + h * 4;
        asm volatile("" : "+v"(mlb));
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            const int ml = mlb + v4;
            const int m = sm0 + ml;
            const int rs = rs_p[ml];
            const float c = cf_p[ml];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int n = sn0 + wn0 + ni * 32 + l32;
                if (!masked || (m < M && n < eN))
                    __builtin_nontemporal_store((float)(A[mi][ni][vq * 4 + v4] - rs) * c, ey + (int64_t)m * eN + n);
            }
        }
    };

    /* group g of the previous tile, whose finished fp32 values wait in P: one address add and one
     * store per value (32-bit byte offsets from the uniform base: the host sends outputs of 4 GiB
     * or more to the kernel without deferred stores) */
    auto emit_prev = [&](const int g) __attribute__((always_inline)) {
        constexpr int GPQ = 4 / RPG;                     /* groups per block of four rows */
        const int mi = g / (4 * GPQ), vq = (g / GPQ) % 4, v0 = (g % GPQ) * RPG;
        int mlb = wm0 + mi * 32 + vq * 8 + h * 4;
        asm volatile("" : "+v"(mlb));
        const uint32_t bo = ((uint32_t)(pm0 + mlb) * (uint32_t)eN + (uint32_t)(pn0 + wn0 + l32)) * 4u;
#pragma unroll
        for (int v4 = v0; v4 < v0 + RPG; ++v4)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                __builtin_nontemporal_store(__int_as_float(P[mi][ni][vq * 4 + v4]),
                                            (float BL_G*)((char BL_G*)ey + (size_t)(bo + ((uint32_t)v4 * (uint32_t)eN + ni * 32u) * 4u)));
    };

    while (true) {
        const int m0 = tm * G3_BM, n0 = tn * BN;
        if constexpr (DEFER) {
            rs_s = rs_base + cset * 2 * G3_BM;
            cf_s = (float*)(rs_s + G3_BM);
        }
        bl_v16i C[MI][NI];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) C[mi][ni][v] = 0;

        for (int kk = 0; kk < steps; ++kk) {
            /* stage kk must have landed; the stages issued after it may stay in flight */
            const int later = steps - 1 - kk;
            if constexpr (DEFER) {
                /* the SPG stores of the step before were issued behind this stage's loads: they may
                 * stay in flight (vector memory operations retire in order) */
                if (have_prev && kk >= 1 && kk <= GROUPS) BL_WAIT_VM(SPG);
                else BL_WAIT_VM(0);
            } else {
                bl_wait_stages<STAGES - 2, LOADS>(later < STAGES - 2 ? later : STAGES - 2);
            }
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (kk + STAGES - 1 < steps) issue(kk + STAGES - 1, (kk + STAGES - 1) % STAGES);
            const uint8_t* st = smem + (kk % STAGES) * G3_STAGE_BYTES;
            /* operands of sub-step ks+1 are fetched while ks multiplies */
            bl_v4i wq[NI], a[2][MI];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) wq[ni] = *(const bl_v4i*)(st + w_off + ni * 32 * 32);
            if (HALF && kk == steps - 1 && h == 1) {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) wq[ni] = bl_v4i{0, 0, 0, 0};
            }
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
                a[0][mi] = *(const bl_v4i*)(st + a_row_off + mi * 32 * G3_BK + (((4 * h) ^ a_swz) * 16));
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                if (ks < 3) {
                    const int unit = ((4 * h + ks + 1) ^ a_swz) * 16;
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
                        a[(ks + 1) & 1][mi] = *(const bl_v4i*)(st + a_row_off + mi * 32 * G3_BK + unit);
                }
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    const bl_v4i bop = bl_unpack16(LAYOUT == 0 ? bl_word_to_k16((uint32_t)wq[ni][ks]) : (uint32_t)wq[ni][ks]);
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
                        C[mi][ni] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks & 1][mi], bop, C[mi][ni], 0, 0, 0);
                }
            }
            /* the pending stores go out behind the step's last MFMA: the matrix core works on while
             * the wave issues them */
            if constexpr (DEFER) {
                if (have_prev && kk < GROUPS) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int g = 0; g < GROUPS; ++g)
                        if (kk == g) emit_prev(g);
                }
            }
        }

        /* Epilogue.  The per-row terms go through LDS once: a load per output row inside the
         * store loop would serialise on latency.  Every wave is past its last stage read after
         * the barrier, so the first stages of this workgroup's NEXT tile are requested here and
         * travel while this tile is stored. */
        if constexpr (DEFER) {
            if (have_prev) {
#pragma unroll
                for (int g = 0; g < GROUPS; ++g)
                    if (g >= steps) emit_prev(g);
                have_prev = false;
            }
        }
        /* EPI 1: the residual values of four row groups (32 rows) are requested ahead, a group's successor
         * when it has been stored (if there is one); clamped and unconditional.  The first ones travel while the row terms are
         * handed over.  (Fetched in front of their own stores they cost eight round trips to memory per
         * tile; all at once they spill 63 registers, this form three.  With the row maxima by DPP instead of shuffles, at M = 4096: residual
         * epilogue 82 -> 75.5 us, gate epilogue 180 -> 168 us, means of two layers.) */
        float rres[EPI == 1 ? 4 : 1][4][NI];
        auto fetch_res = [&](const int mi, const int vq) __attribute__((always_inline)) {
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                int m = m0 + wm0 + mi * 32 + vq * 8 + h * 4 + v4;
                m = m < M ? m : M - 1;
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    const int n = n0 + wn0 + ni * 32 + l32;
                    rres[vq][v4][ni] = eres[(int64_t)m * N + (n < N ? n : N - 1)];
                }
            }
        };
        if constexpr (EPI == 1) {
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) fetch_res(0, vq);
        }
        bl_mfma_fence();
        if (tid < G3_BM) {
            rs_s[tid] = row_rs;
            cf_s[tid] = row_cf;
        }
        /* these LDS writes must have been performed before any wave passes the barrier (a raw
         * s_barrier does not wait for them) */
        BL_WAIT_LGKM0();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        int tm2 = 0, tn2 = 0;
        const int vb2 = next_tile(vb + (TABLE ? 1 : (int)gridDim.x), tm2, tn2);
        if (vb2 >= 0) {
            setup(tm2, tn2);
            for (int s0 = 0; s0 < STAGES - 1 && s0 < (TABLE ? nsteps : steps); ++s0) issue(s0, s0);
        }
        if constexpr (DEFER) {
            if (vb2 >= 0 && m0 + G3_BM <= M && n0 + BN <= eN) {
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int ml = wm0 + mi * 32 + (v >> 2) * 8 + h * 4 + (v & 3);
                        const int rs = rs_s[ml];
                        const float c = cf_s[ml];
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni) P[mi][ni][v] = __float_as_int((float)(C[mi][ni][v] - rs) * c);
                    }
                pm0 = m0;
                pn0 = n0;
                pset = cset;
                have_prev = true;
            } else {
#pragma unroll
                for (int g = 0; g < MI * 4; ++g) emit_rows(C, g, m0, n0, cset, true);
            }
            cset ^= 1;
        } else if constexpr (EPI == 0) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                /* the residual values of four rows first, then their stores back to back: a load
                 * between two stores would make each store wait for the one before it */
                float rres[4][NI];
                if (eres && ey) {
#pragma unroll
                    for (int v4 = 0; v4 < 4; ++v4) {
                        const int m = m0 + wm0 + mi * 32 + vq * 8 + h * 4 + v4;
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni) {
                            const int n = n0 + wn0 + ni * 32 + l32;
                            rres[v4][ni] = (m < M && n < eN) ? eres[(int64_t)m * eN + n] : 0.0f;
                        }
                    }
                }
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    const int v = vq * 4 + v4;
                    const int ml = wm0 + mi * 32 + vq * 8 + h * 4 + v4;
                    const int m = m0 + ml;
                    if (m < M) {
                        const int rs = rs_s[ml];
                        const float c = cf_s[ml];
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni) {
                            const int n = n0 + wn0 + ni * 32 + l32;
                            if (n < eN) {
                                const int val = C[mi][ni][v] - rs;
                                if (eacc) eacc[(int64_t)m * eN + n] = val;
                                if (ey) {
                                    const float t = (float)val * c;
                                    const float out = eres ? rres[v4][ni] + t : t;
                                    __builtin_nontemporal_store(out, ey + (int64_t)m * eN + n);
                                }
                            }
                        }
                    }
                }
            }
        } else {
            /* fused producer epilogue: glue value t, its bf16 narrowing (the next BitLinear's input
             * before quantisation) and the row maximum of |bf16(t)|: over the lane's columns, then over
             * the 32 lanes of a half wave (DPP), then one atomic max per row on the float bits
             * (non-negative floats order like integers, so the result does not depend on the order) */
            constexpr int MAG0 = 0x007F0000;          /* added to a magnitude's bits: infinity is the largest int, a NaN negative */
            /* A tile inside the matrix without an int32 output stores unconditionally, so that neither a branch nor a
             * wait for memory stands between its stores; `cut`: every other one (and the residual in 128-row tiles, where both
             * forms together spill 55 registers: 4096 x 2560 -> 2560 48.9 us, 40.5 with `cut` alone).  With the
             * atomics of eight rows in one instruction (before: two rows; the epilogue waited for each), at 2560 -> 13824 with the
             * gate and the tiles of launch_fused: 128 tokens 60 -> 20 us, 512 53 -> 25, 2048 82 -> 73, 4096 151 -> 138. */
            const int NOUT = EPI == 2 ? N / 2 : N, col0 = EPI == 2 ? tn * (BN / 2) + wn0 / 2 + l32 : n0 + wn0 + l32;
            const int mlast = M - 1 - m0;
            auto finish = [&](auto cut_t) __attribute__((always_inline)) {
                constexpr bool cut = decltype(cut_t)::value;
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int vq = 0; vq < 4; ++vq) {
                        const int ml = wm0 + mi * 32 + vq * 8 + h * 4;
                        float rowmax[4];
#pragma unroll
                        for (int v4 = 0; v4 < 4; ++v4) {
                            const int v = vq * 4 + v4;
                            int mx = MAG0;
                            if (!cut || ml + v4 <= mlast) {
                                const int rs = rs_s[ml + v4];
                                const float c = cf_s[ml + v4];
                                const int64_t m = m0 + ml + v4;
#pragma unroll
                                for (int ni = 0; ni < (EPI == 2 ? 1 : NI); ++ni) {
                                    const int n = col0 + ni * 32;
                                    if (!cut || n < NOUT) {
                                        const int val = C[mi][ni][v] - rs;
                                        if (cut && acc) {
                                            acc[m * N + n] = val;
                                            if (EPI == 2) acc[m * N + NOUT + n] = C[mi][NI - 1][v] - rs;
                                        }
                                        const float t = (float)val * c;
                                        float o;
                                        if (EPI == 1) {
                                            o = rres[vq][v4][ni] + t;
                                        } else {
                                            const float u = (float)(C[mi][NI - 1][v] - rs) * c;
                                            const float r = fmaxf(t, 0.0f);
                                            const float r2 = r * r;
                                            o = r2 * u;
                                        }
                                        if (cut ? y != nullptr : EPI == 1) __builtin_nontemporal_store(o, y + m * NOUT + n);
                                        const uint32_t bits = bl_pack2_bf16(o, o);
                                        xb[m * NOUT + n] = (uint16_t)bits;
                                        mx = max(mx, (int)(((bits << 16) & 0x7FFF0000u) + (uint32_t)MAG0));
                                    }
                                }
                            }
                            rowmax[v4] = __int_as_float(mx - MAG0);
                        }
                        if constexpr (EPI == 1) {
                            if (mi + 1 < MI) fetch_res(mi + 1, vq);
                        }
#pragma unroll
                        for (int v4 = 0; v4 < 4; ++v4) rowmax[v4] = bl_half_max(rowmax[v4]);
                        /* lane v4 of a half stands for row v4: one atomic instruction for eight rows */
                        const float mine = l32 == 0 ? rowmax[0] : l32 == 1 ? rowmax[1] : l32 == 2 ? rowmax[2] : rowmax[3];
                        if (l32 < 4 && (!cut || ml + l32 <= mlast)) atomicMax(absmax + m0 + ml + l32, __float_as_int(mine));
                    }
            };
            constexpr bool both = EPI == 2 || BM < 128;
            const bool whole = mlast >= G3_BM - 1 && (EPI == 2 || n0 + BN <= N) && !acc && (y != nullptr) == (EPI == 1);
            if constexpr (both) {
                if (whole) finish(std::false_type{});
                else finish(std::true_type{});
            } else {
                finish(std::true_type{});
            }
        }
        if (vb2 < 0) {
            if (stamp && tid == 0) {
                stamps[0] = clock64() - c_start;
                stamps[1] = wall_clock64() - w_start;
            }
            break;
        }
        vb = vb2;
        tm = tm2;
        tn = tn2;
        if constexpr (TABLE) {
            steps = nsteps; eN = nN; eres = nres; eacc = nacc; ey = ny;
        }
        /* the next tile's epilogue rewrites rs_s / cf_s only after its own k loop, whose barriers
         * every wave passes after it has finished the reads above */
    }
}

/* Outputs of the fused producer epilogues (device pointers; see bl_gemm_tile256). */
struct bl_epi_args {
    uint16_t* xb;
    int* absmax;
};

/* Workgroups of a kernel that are resident at once (a multiple of 8 keeps a workgroup on its XCD's region), 0 on
 * error; asked once, together with the attribute that its LDS needs. */
template <int BM, int BN, int STAGES, int WM, int WN, int EPI, bool DEFER, bool HALF, int LAYOUT>
struct bl_tile256_launch {
    static constexpr int lds = STAGES * (BM * G3_BK + BN * G3_BK / 4) + BM * 8 * (DEFER ? 2 : 1);
    static int resident() {
        static std::atomic<int> cached{0};
        int blocks = cached.load(std::memory_order_acquire);
        if (blocks > 0) return blocks;
        const auto kern = bl_gemm_tile256<BM, BN, STAGES, WM, WN, EPI, false, DEFER, HALF, LAYOUT>;
        int dev = 0, cus = 0, per_cu = 0;
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kern, WM * WN * 64, lds) != hipSuccess ||
            cus < 1 || per_cu < 1)
            return 0;
        blocks = cus * per_cu / 8 * 8;
        if (blocks < 8) blocks = 8;
        cached.store(blocks, std::memory_order_release);
        return blocks;
    }
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

template <int BM, int BN, int STAGES, int WM, int WN, int EPI = 0, bool DEFER = false, bool HALF = false, int LAYOUT = 1>
static bl_status launch_tile256_t(const uint8_t* packed, const float* beta, const int8_t* q, const float* scale,
                                  const int32_t* rowsum, int M, int N, int K, const float* residual,
                                  int32_t* acc, float* y, hipStream_t st, bl_epi_args ep = bl_epi_args{nullptr, nullptr}) {
    constexpr int G3_BM = BM;
    using L = bl_tile256_launch<BM, BN, STAGES, WM, WN, EPI, DEFER, HALF, LAYOUT>;
    int blocks = L::resident();                          /* a persistent grid */
    if (blocks == 0) return BL_ERR_HIP;
    /* the gate epilogue's tile holds 64 gate rows and the 64 matching up rows: N/2 / 64 column tiles */
    const int tiles_m = (M + G3_BM - 1) / G3_BM, tiles_n = EPI == 2 ? (N / 2 + BN / 2 - 1) / (BN / 2) : (N + BN - 1) / BN;
    if ((int64_t)tiles_m * tiles_n > ((int64_t)1 << 30)) return BL_ERR_SHAPE;   /* (outputs beyond 2^43 values) */
    const bl_tile_order o = tile_order(tiles_m, tiles_n, BM, K);
    const int gm = o.gm, band = o.band, vgrid = o.vgrid;
    if (blocks > vgrid) blocks = vgrid;
    bl_gemm_tile256<BM, BN, STAGES, WM, WN, EPI, false, DEFER, HALF, LAYOUT><<<blocks, WM * WN * 64, L::lds, st>>>(
        packed, q, rowsum, beta, scale, M, N, K, tiles_m, tiles_n, gm, band, vgrid, residual, acc, y, ep.xb, ep.absmax, (long long*)bl_clock_stamps(), nullptr, nullptr, 0, nullptr, nullptr);
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}

/* Table walk (batched decode of a stack, more than 48 tokens): 64 x 128 tiles, one launch over
 * every tile of every product.  items / tile0: device arrays of `nitems` entries (tile0 ascending,
 * tile0[0] = 0); total_tiles = tiles of the whole table; M <= 64 tokens, the same for every
 * product.  Workgroup b takes the tiles tile_list[wg_start[b] .. wg_start[b+1]) (device arrays
 * of blocks + 1 and total_tiles entries: the host balances the k steps over the workgroups).
 * bl_gemm_table_blocks: the persistent grid (resident workgroups), 0 on error. */
static constexpr int TABLE_LDS = 2 * (64 * G3_BK + 128 * G3_BK / 4) + 64 * 8;
static std::atomic<int> g_table_blocks{0};

int bl_gemm_table_blocks(void) {
    int blocks = g_table_blocks.load(std::memory_order_acquire);
    if (blocks > 0) return blocks;
    auto kern = bl_gemm_tile256<64, 128, 2, 1, 4, 0, true>;
    int dev = 0, cus = 0, per_cu = 0;
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, TABLE_LDS) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kern, 256, TABLE_LDS) != hipSuccess ||
        cus < 1 || per_cu < 1)
        return 0;
    blocks = cus * per_cu;
    g_table_blocks.store(blocks, std::memory_order_release);
    return blocks;
}

bl_status bl_gemm_table_launch(const bl_tile_item* items, const int* tile0, int nitems, int total_tiles, int M,
                               int blocks, const int* wg_start, const int* tile_list, bl_stream s) {
    hipStream_t st = (hipStream_t)s;
    if (g_table_blocks.load(std::memory_order_acquire) == 0) return BL_ERR_VALUE;   /* no table was built in this process */
    bl_gemm_tile256<64, 128, 2, 1, 4, 0, true><<<blocks, 256, TABLE_LDS, st>>>(
        nullptr, nullptr, nullptr, nullptr, nullptr, M, 0, G3_BK, 1, 0, 1, 1, total_tiles, nullptr, nullptr, nullptr, nullptr,
        nullptr, nullptr, items, tile0, nitems, wg_start, tile_list);
    return hipGetLastError() == hipSuccess ? BL_OK : BL_ERR_HIP;
}

/* ---- few tiles: the k loop split over the waves of a workgroup -------------------------------
 * With few tokens (65 .. a few hundred) a product has fewer 64 x 128 tiles than the chip has compute
 * units, and its time is one tile's serial chain of k steps (about 720 clocks each, of which the matrix
 * cores work 256).  Here a workgroup owns a 64 x 32 tile and each of its four waves takes every fourth
 * k step of it alone: four times the workgroups, a quarter of the chain, and no barrier inside the loop (a
 * wave's stages in LDS are its own; it waits for its own loads).  The four partial tiles meet in LDS and
 * each wave finishes a quarter of the rows.  The weights cost the same bytes as before, the activations
 * are fetched by four times as many workgroups, from the L2.
 * Same LDS layout, swizzles, half last step and layout-0 words as bl_gemm_tile256 (one wave: pieces of
 * eight activation rows and one of 32 weight rows).
 * Measured (us, 64 x 128 tiles of bl_gemm_pipe / this kernel): 40 tiles 128 x 6912 -> 2560 19.8 / 11.2, 80 tiles 256 x 2560 ->
 * 2560 10.0 / 8.3, 104 tiles 800 x 7000 -> 1024 20.5 / 17.1, 160 tiles 512 x 2560 -> 2560 10.4 / 12.9: there the tiles fill the chip. */
#define KS_STAGE (64 * G3_BK + 32 * G3_BK / 4)

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
    const bool stamp = stamps != nullptr && blockIdx.x == 0;            /* measurement hook, as in bl_gemm_tile256 */
    long long c_start = 0, w_start = 0;
    if (stamp) {
        c_start = clock64();
        w_start = wall_clock64();
    }
    const int along = across ? across : tiles_m, major = at / along, minor = at - major * along;
    const int m0 = (across ? major : minor) * 64, n0 = (across ? minor : major) * 32;
    const int steps = (K + G3_BK - 1) / G3_BK;
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
            __builtin_amdgcn_global_load_lds((bl_gptr)(asrc[j] + ((int64_t)kk * G3_BK - back)), (bl_lptr)(st + j * 1024), 16, 0, 0);
        }
        __builtin_amdgcn_global_load_lds((bl_gptr)(wsrc + ((int64_t)kk * (G3_BK / 4) - (last ? wu * 16 : 0))),
                                         (bl_lptr)(st + 64 * G3_BK), 16, 0, 0);
    };
    const int a_off = l32 * G3_BK, a_swz = (l32 >> 1) & 7;
    const int w_off = 64 * G3_BK + (l32 * 2 + (h ^ ((l32 >> 3) & 1))) * 16;

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
            for (int mi = 0; mi < 2; ++mi) a[ks][mi] = *(const bl_v4i*)(st + a_off + mi * 32 * G3_BK + (((4 * h + ks) ^ a_swz) * 16));
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
    const float rounds = (float)((tiles + 511) / 512), steps = (float)((k + G3_BK - 1) / G3_BK);
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
                                             residual, acc, y, ep.xb, ep.absmax, (long long*)bl_clock_stamps());
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
        const float steps = (float)((k + G3_BK - 1) / G3_BK);
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
    if (M < 1 || M > BL_MAX_DIM || !bl_shape_ok(N, K) || K % G3_BK != 0 || N % 4 != 0) return BL_ERR_SHAPE;
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
