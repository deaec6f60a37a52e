// X' = P X for more than 32 workers, or more than 16 on rows off 16-byte boundaries, fused with the local SGD step (see mix_dense.hip).
//
// Every fp32 value is split into three bf16 values for the multiplies and the sums are fp32 (split_bf16.h has the errors).
// P (N x N, zero-padded to NPAD = 32 * MB) is tiny and lives in registers: a wavefront keeps the three planes of its 32
// rows for the whole kernel (192 of the 256 registers it can have, for N = 256).  The workgroup walks over column tiles
// of X.  A tile goes from global memory straight into LDS as it is (raw); each wavefront then splits the 1024 elements it
// fetched itself, eight rows of a column per lane and step, into the planes' fragment order [8 rows][column][8 values],
// where a lane's 16 bytes are its fragment of one matrix instruction: every LDS access is a run of consecutive 16-byte
// (raw: 4-byte) pieces.  The planes are double
// buffered, so that one of the two wavefronts of a SIMD splits and stores while the other multiplies, with one
// barrier per tile.  Gradients go through LDS too, by the same kind of load, because no registers are left to keep them in
// while the wave multiplies (requested into registers instead, they pushed P out to scratch memory: 0.95 ms).
//
// What bounds it: the memory, for N <= 128 (N = 128 x 2 M columns with gradients 0.63 ms = 4.9 TB/s, and 0.62 with
// the multiplies left out); for N = 256 x 1 M 0.82 ms, where the memory side alone takes 0.65 (128-byte pieces of rows that
// lie far apart) and the multiplies and splits alone 0.56.  The fp32 matrix instruction that this kernel used before needs
// 0.83 ms at its peak rate for the latter shape and took 1.13; N = 128 without gradients, 2.8 M columns: 0.88 -> 0.61 ms;
// N = 60 x 4 M: 0.60 -> 0.56.  Where X, the result and the gradients together are larger than the last-level cache and every row starts on
// a 128-byte line, results, and from 65 workers on loads, pass the caches by: N = 128 x 2.8 M without gradients 690 -> 678 us (a
// linear stream of as many bytes: 448), N = 256 x 1 M with them 840 -> 829, N = 128 x 1 M 318 -> 309.  Smaller matrices are still
// there when the next round reads them: rounds one after the other of N = 64 x 100 000 and x 400 000 without gradients 12.4 and 35.6 us,
// past the caches 14.0 and 42.3; the first with gradients 15.7, 16.9; N = 256 x 50 000 with gradients 47, 49.6.  A piece of a row that
// shares its lines with the next piece goes to memory twice past the caches: N = 128 x 1 M without gradients, rows of 4-byte, 16-byte
// and 64-byte boundaries 355, 337 and 265 us, past the caches 521, 478 and 263, with gradients 445, 441 and 358, 595, 639 and 410 (with
// neighbouring tiles on XCDs of their own, before TileWalk took them together: 445 -> 388).  (Loads
// past the caches cost up to 64 workers: N = 60 x 200 000 33 -> 35.)
// The stores are global ones (global_access.h): as flat ones every wait for LDS waited for them as well, N = 128 x 2.8 M
// without gradients 677 -> 662, N = 256 x 1 M 829 and 832.  The multiplies cost time although they overlap the memory side: without them the two take 631 and 565.
// The chip runs at 1.7 GHz then (2.4 in a copy), and schedules that keep the matrix cores busier are slower: the two wavefronts
// of a SIMD half a tile apart, one multiplying while the other stores and splits, 906 and 747 (881 and 768 with each fragment requested
// right behind the last multiply that reads the one before it).
// Tried without gain: two tiles of X on their way instead of one (685), one 64-column tile with a single set of
// planes (0.88), wave priorities for either phase, LDS fragments requested a step ahead.
//
// D of v_mfma_f32_32x32x16_bf16, lane l: 16 floats, d[v] = D[m = 8 * (v / 4) + 4 * (l / 32) + v % 4][n = l % 32]
#pragma once

#include <type_traits>

#include "dbw_internal.h"
#include "global_access.h"
#include "split_bf16.h"

namespace mixsplit {

using global_access::bytes;
using global_access::uniform_base;

constexpr int64_t CACHE_BYTES = (int64_t)256 << 20;    // the last-level cache

// MB: 32-row blocks of the padded P; WAVES: wavefronts of a workgroup.
template <int MB, int WAVES>
struct Cfg {
    static constexpr int NPAD = 32 * MB;              // padded number of workers
    static constexpr int KS = NPAD / 16;              // 16-wide steps of the matrix instruction
    static constexpr int CG = WAVES / MB;             // column groups of 32 among the waves
    static constexpr int TC = 32 * CG;                // tile columns
    static constexpr int RW = NPAD / WAVES < 8 ? 8 : NPAD / WAVES;   // rows and columns of the block a wave fetches and splits
    static constexpr int CW = 1024 / RW;
    static constexpr int CBLOCKS = TC / CW;
    static constexpr int GROUPS = NPAD / 8 * TC;      // 16-byte groups per plane: 128 per wave for every MB
};

// 64 x 16 (WIDE) or 64 x 4 bytes from global memory (uniform base + lane offset) to LDS at `dst` (uniform) + 16 or 4 * lane.  As inline
// assembly and not as the builtin: behind the builtin the compiler waits for the loads to land before the next LDS read,
// whichever LDS array that is from.  The kernel waits itself (vmcnt) before it reads what they bring.  (m0, the LDS
// address of such a load, has no other user in this kernel.)  STREAM: not kept in the caches.
template <bool WIDE, bool STREAM>
__device__ __forceinline__ void load_to_lds(bytes base, uint32_t lane_off, const float *dst)
{
    const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const float *)dst);
    if (WIDE && STREAM)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(lane_off), "s"(base), "s"(m0) : "memory");
    else if (WIDE)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(base), "s"(m0) : "memory");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(lane_off), "s"(base), "s"(m0) : "memory");
}

// At most N of this wave's memory operations are still under way / all its LDS operations are done.
template <int N>
__device__ __forceinline__ void wait_memory()
{
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_lds()
{
    __builtin_amdgcn_s_waitcnt(0xc07f);
    asm volatile("" ::: "memory");
}

// WIDE: every row starts on a 16-byte boundary and is padded to a multiple of four floats, so 16 bytes per lane can
// be fetched and the float4 that straddles column d lies inside its row; otherwise the same elements come 4 bytes
// per lane, in four times as many instructions (N = 254 x 730 k columns: 0.80 ms against 0.63; a
// thread per column and row that gathers its operands, as before, 30.7).
// STREAM: the matrices do not fit the last-level cache, see above.  (One store statement for both forms makes the compiler merge the
// branches of full and ragged blocks, which costs up to 10 % where a block of rows is ragged.)
template <int MB, int WAVES, int ORDER, bool HAS_G, bool WIDE, bool STREAM, class LR>
__global__ __launch_bounds__(64 * WAVES, 2) void kernel(
    int N, int64_t dcols /* = d */, int64_t ld, const float *__restrict__ Wsw, const float *__restrict__ x, const float *__restrict__ g,
    float *__restrict__ out, LR lr, int n_tiles)
{
    using C = Cfg<MB, WAVES>;
    using split_bf16::u32x4;
    constexpr bool PRO = ORDER == DBW_ORDER_ATC && HAS_G;          // x - lr g is formed before the split
    constexpr bool EPI = ORDER == DBW_ORDER_CTA && HAS_G;
    __shared__ __attribute__((aligned(16))) float raw_x[WAVES * 1024];
    __shared__ __attribute__((aligned(16))) float raw_g[HAS_G ? WAVES * 1024 : 4];
    __shared__ __attribute__((aligned(16))) u32x4 pl[2][3][C::GROUPS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave index, kept scalar
    const int rb = w % MB, cg = w / MB;                          // block of the result
    const int fr = w / C::CBLOCKS * C::RW, fc = w % C::CBLOCKS * C::CW;   // first row and column of the block it splits

    // (rows on lines, past the caches: as they come, N = 128 x 1 M with gradients 308 us, 311 otherwise)
    const TileWalk<!STREAM, int> walk(n_tiles);          // (rows of at most DBW_DENSE_MAX_LD columns)
    int tile = walk.first(), next = walk.next(tile);
    if (tile >= n_tiles) return;

    // ---- a block of ROWS x (1024 / ROWS) elements of tile t at (r0, c0) -> 4 KB of LDS, row after row, by LOADS
    // instructions.  In the place of rows and columns beyond the matrix a valid one is read (never used, never stored).
    constexpr int LOADS = WIDE ? 4 : 16, V = WIDE ? 4 : 1;                                // instructions, floats per lane
    auto fetch = [&](const float *src, int64_t t, auto rows, int r0, int c0, float *dst) {
        constexpr int COLS = 1024 / decltype(rows)::value, LANES = COLS / V, PER = COLS > 64 * V ? 1 : 64 * V / COLS;
        constexpr int PIECES = COLS > 64 * V ? COLS / (64 * V) : 1;                       // instructions per row
        const int lane_row = PIECES > 1 ? 0 : lane / LANES, lane_col = V * (PIECES > 1 ? lane : lane % LANES);
        uint32_t row_off = 4u * (uint32_t)(lane_row * (int)ld);
        asm volatile("" : "+v"(row_off));              // worked out per tile: LOADS offsets kept over the loop would spill
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int r = r0 + i / PIECES * PER;                                          // uniform
            const int64_t last = (dcols - 1) / V * V, cb = min(t * C::TC + c0 + 64 * V * (i % PIECES), last);
            const uint32_t c_off = 4u * (uint32_t)min((int64_t)lane_col, last - cb);
            load_to_lds<WIDE, STREAM && MB >= 4>(uniform_base(src + (int64_t)min(r, N - 1) * ld + cb), (lane_row < N - r ? row_off : 0u) + c_off,
                              dst + 1024 * w + 64 * V * i);
        }
    };
    auto fetch_x = [&](int64_t t) { fetch(x, t, std::integral_constant<int, C::RW>{}, fr, fc, raw_x); };
    auto fetch_g = [&](int64_t t) {
        if (PRO) fetch(g, t, std::integral_constant<int, C::RW>{}, fr, fc, raw_g);        // next to the elements of X
        if (EPI) fetch(g, t, std::integral_constant<int, 32>{}, 32 * rb, 32 * cg, raw_g); // for the wave's block of the result
    };
    // ---- the wave's block, split: two groups of eight rows per lane
    auto split = [&](int buf) {
        int half = lane >> 5;
        asm volatile("" : "+v"(half));                 // the rates of a lane's rows are picked per tile, not kept in registers
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int kg = (64 * u + lane) / C::CW, col = (64 * u + lane) % C::CW;
            const float *src = &raw_x[1024 * w + 8 * kg * C::CW + col], *gsrc = &raw_g[PRO ? 1024 * w + 8 * kg * C::CW + col : 0];
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = src[j * C::CW];
            if (PRO) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    // the rate of a row: uniform loads (of both halves' rows, where a step covers two groups)
                    const int r = fr + 8 * (64 * u / C::CW) + j;
                    float e = lr.at(min(r, N - 1));
                    if (C::CW == 32) e = half == 0 ? e : lr.at(min(r + 8, N - 1));
                    v[j] = fmaf(-e, gsrc[j * C::CW], v[j]);
                }
            }
            if (N < C::NPAD) {
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = fr + 8 * kg + j < N ? v[j] : 0.f;
            }
            const split_bf16::planes q = split_bf16::split8(v);
            const int at = (fr / 8 + kg) * C::TC + fc + col;
            pl[buf][0][at] = q.h;
            pl[buf][1][at] = q.m;
            pl[buf][2][at] = q.l;
        }
    };
    fetch_x(tile);
    fetch_g(tile);

    // ---- P, split into planes
    split_bf16::planes P[C::KS];
    constexpr int STEP = C::KS < 4 ? C::KS : 4;
#pragma unroll
    for (int s4 = 0; s4 < C::KS; s4 += STEP) {
        float v[STEP][8];
#pragma unroll
        for (int s = 0; s < STEP; ++s) {
            // Wsw: [row block][k pair][lane], lane = 32 (k & 1) + row
            const float *wp = Wsw + ((size_t)rb * (C::NPAD / 2) + 8 * (s4 + s) + 4 * (lane >> 5)) * 64 + (lane & 31);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[s][j] = wp[(j >> 1) * 64 + (j & 1) * 32];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < STEP; ++s) P[s4 + s] = split_bf16::split8_nearest(v[s]);
        __builtin_amdgcn_sched_barrier(0);
    }
    wait_memory<0>();
    split(0);
    wait_lds();
    if (next < n_tiles) {
        fetch_x(next);
        if (PRO) fetch_g(next);
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    int buf = 0;
    for (; tile < n_tiles; tile = next, next = walk.next(next)) {
        const int64_t col0 = (int64_t)tile * C::TC + 32 * cg;                              // uniform
        const bool full = 32 * rb + 32 <= N && col0 + 32 <= dcols;                // uniform: no element needs a guard
        const u32x4 *b0 = &pl[buf][0][(lane >> 5) * C::TC + 32 * cg + (lane & 31)];
        split_bf16::f32x16 acc, small;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = small[v] = 0.f;
#pragma unroll
        for (int s = 0; s < C::KS; ++s) {
            split_bf16::planes b;
            b.h = b0[2 * s * C::TC];
            b.m = b0[2 * s * C::TC + C::GROUPS];
            b.l = b0[2 * s * C::TC + 2 * C::GROUPS];
            split_bf16::mma32<false>(P[s], b, acc, small);
            __builtin_amdgcn_sched_barrier(0);
        }
        split_bf16::add_small(acc, small);

        // ---- local SGD correction and store, 32 consecutive columns per row
        if (EPI) {
            // the gradients are older than the loads of the next tile of X
            if (next < n_tiles) wait_memory<LOADS>(); else wait_memory<0>();
            int half = lane >> 5;
            asm volatile("" : "+v"(half));
            const float *gp = &raw_g[1024 * w + 128 * half + (lane & 31)];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = 8 * (v / 4) + (v & 3), row0 = 32 * rb + r;
                const float e0 = lr.at(min(row0, N - 1)), e1 = lr.at(min(row0 + 4, N - 1));
                acc[v] = fmaf(-(half == 0 ? e0 : e1), gp[32 * r], acc[v]);
            }
        }
        const uint32_t lane_off = 4u * (uint32_t)(4 * (lane >> 5) * (int)ld + (lane & 31));
        if (full) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if constexpr (STREAM)
                    global_access::store_stream(out + (int64_t)(32 * rb + 8 * (v / 4) + (v & 3)) * ld + col0, lane_off, acc[v]);
                else
                    global_access::store(out + (int64_t)(32 * rb + 8 * (v / 4) + (v & 3)) * ld + col0, lane_off, acc[v]);
            }
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row0 = 32 * rb + 8 * (v / 4) + (v & 3);
                if (row0 + 4 * (lane >> 5) < N && col0 + (lane & 31) < dcols)
                    global_access::store(out + (int64_t)row0 * ld + col0, lane_off, acc[v]);
            }
        }

        // ---- the next tile
        if (next < n_tiles) {
            if (EPI) {
                wait_lds();                            // raw_g has been read
                fetch_g(next);
            }
            // its loads are older than the stores (16 of them, if none was left out) and the gradient loads above
            if (full) wait_memory<EPI ? 16 + LOADS : 16>(); else wait_memory<EPI ? LOADS : 0>();
            split(buf ^ 1);
            wait_lds();                                // raw_x (PRO: raw_g) has been read, the planes are written
            const int after = walk.next(next);
            if (after < n_tiles) {
                fetch_x(after);
                if (PRO) fetch_g(after);
            }
        }
        // the planes of the next tile are complete, those of this one free (loads and stores stay under way)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        buf ^= 1;
    }
}

}  // namespace mixsplit
