// Dense form of the consensus update for near-complete graphs: X' = P(k) X on the matrix
// cores, fused with the local SGD step (Section 2.2, compact matrix form; rows are workers
// here, so the paper's W(k) P(k) reads P X).
//
//   CTA: out = P X - lr G            ATC: out = P (X - lr G)
//
// More than 32 workers take the kernel of mix_split.h, and so do rows off 16-byte boundaries from 17 workers on; up to 16 of
// those are mix_dense_columns' (at the end).  mix_dense_kernel does up to 32 workers on aligned rows.
//
// P (N x N, zero-padded to 32 x 32) is tiny and lives in registers: each of the 8 wavefronts of a workgroup keeps its
// A-operand fragments for the whole kernel.  The workgroup walks over column tiles of X; a tile (32 rows x 256 columns, 32
// columns for each wave) is staged once through LDS, laid out so that the B-operand fragment of v_mfma_f32_32x32x2_f32 for
// k-step kk is one conflict-free 64-lane row.  The next tile is on its way while the current one is multiplied: when no
// element needs a guard (FULL tiles) it goes from global memory straight into LDS (global_load_lds, 16 bytes per lane),
// otherwise through registers.  With the local step first (ATC) the gradient values of the
// same elements travel in registers meanwhile, and x - lr g is formed in LDS once both have
// landed, after the multiplies: forming it in registers right behind the loads made every
// wave wait for them before it could start multiplying.  In the other order the gradient
// values of the epilogue are requested before the multiply loop so that they have arrived
// when it ends.  The instruction multiplies fp32 values as they are.
//
// Fragment layout of v_mfma_f32_32x32x2_f32 (M = N = 32, K = 2), lane l in [0, 64):
//   A: a = A[m = l % 32][k = l / 32]        B: b = B[k = l / 32][n = l % 32]
//   D: 16 floats, d[v] = D[m = 8 * (v / 4) + 4 * (l / 32) + v % 4][n = l % 32]
#include <algorithm>

#include "dbw_internal.h"
#include "global_access.h"
#include "mix_split.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(1))) const void *global_cptr;
typedef __attribute__((address_space(3))) void *lds_ptr;

constexpr int DENSE_THREADS = 512;
// Flat accesses: with global ones the guarded gradient loads of the epilogue are slower, 20 workers x 4 M columns 238 us against 229 (elsewhere
// the same).
using global_access::uniform_flat;

constexpr int NPAD = 32;                              // padded number of workers
constexpr int KB = NPAD / 2;                          // k-steps of the 32x32x2 instruction
constexpr int TC = 32 * 8;                            // tile columns: 32 for each wave
constexpr int TILE = NPAD * TC;                       // floats per LDS buffer
constexpr int PASSES = TILE / 4 / DENSE_THREADS;
constexpr int DMA_PER_WAVE = TILE / 256 / 8;          // 1 KB blocks per wave and tile

// FULL: N == NPAD and every tile has all TC columns, so no access needs a guard.
template <int ORDER, bool HAS_G, bool FULL, class LR>
__global__ __launch_bounds__(DENSE_THREADS) void mix_dense_kernel(
    int N, int64_t n_vec /* float4 columns covered, the last may straddle column d */, int64_t dcols /* = d */,
    int64_t ld4, const float *__restrict__ Wsw, const float4 *__restrict__ x, const float4 *__restrict__ g,
    float *__restrict__ out, const float *__restrict__ gs, LR lr, int n_tiles)
{
    constexpr bool DMA = FULL;                                     // tiles go straight into LDS
    constexpr bool PRO = FULL && ORDER == DBW_ORDER_ATC && HAS_G;  // ... and x - lr g is formed there
    __shared__ __attribute__((aligned(16))) float lds[2 * TILE];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave index, kept scalar
    const int64_t ld = ld4 * 4;

    float wreg[KB];
#pragma unroll
    for (int kk = 0; kk < KB; ++kk) wreg[kk] = Wsw[kk * 64 + lane];

    // ---- next-tile staging through registers (guards / ATC prologue)
    float4 stage[DMA ? 1 : PASSES];
    // lane offsets are kept in bytes: uniform 64-bit base + 32-bit lane offset is an addressing mode of
    // the global memory instructions, so no 64-bit address has to live in vector registers
    const uint32_t fetch_lane_off = 16u * (uint32_t)((tid / (TC / 4)) * ld4 + tid % (TC / 4));
    auto fetch = [&](int64_t tile) {
#pragma unroll
        for (int ps = 0; ps < (DMA ? 0 : PASSES); ++ps) {
            const int k0 = ps * (DENSE_THREADS / (TC / 4));                   // uniform first row of the pass
            const int k = k0 + tid / (TC / 4);
            const int64_t col4 = tile * (TC / 4) + tid % (TC / 4);
            const float4 *xb = x + (int64_t)k0 * ld4 + tile * (TC / 4);        // uniform base
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (FULL || (k < N && col4 < n_vec)) {
                v = *(const float4 *)(uniform_flat(xb) + fetch_lane_off);
                if (ORDER == DBW_ORDER_ATC && HAS_G) {
                    const float4 gv =
                        *(const float4 *)(uniform_flat(g + (int64_t)k0 * ld4 + tile * (TC / 4)) + fetch_lane_off);
                    const float eta = lr.at(k);
                    v.x = fmaf(-eta, gv.x, v.x);
                    v.y = fmaf(-eta, gv.y, v.y);
                    v.z = fmaf(-eta, gv.z, v.z);
                    v.w = fmaf(-eta, gv.w, v.w);
                }
            }
            stage[ps] = v;
        }
    };
    // registers -> LDS buffer `buf`, in B-fragment order: [sub-tile][k-step][lane]
    auto commit = [&](int buf) {
#pragma unroll
        for (int ps = 0; ps < (DMA ? 0 : PASSES); ++ps) {
            const int f = ps * DENSE_THREADS + tid;
            const int k = f / (TC / 4), c4 = f % (TC / 4);
            const int s = c4 / 8, l = (k & 1) * 32 + (c4 & 7) * 4;
            *(float4 *)&lds[buf * TILE + ((s * KB + (k >> 1)) * 64 + l)] = stage[ps];
        }
    };
    // ---- next-tile staging straight into LDS.  One instruction fills 1 KB = the 64-lane
    // rows of four consecutive k-steps of one sub-tile; lane -> (row, 4 columns) follows.
    const uint32_t dma_lane_off = 16u * (uint32_t)((2 * (lane >> 4) + ((lane >> 3) & 1)) * ld4 + (lane & 7));
    auto dma = [&](int64_t tile, int buf) {
#pragma unroll
        for (int i = 0; i < (DMA ? DMA_PER_WAVE : 0); ++i) {
            const int q = w + 8 * i;                                             // uniform block id
            const int s = q / (KB / 4), kq = q % (KB / 4);
            const float4 *src = x + (int64_t)(8 * kq) * ld4 + tile * (TC / 4) + s * 8;   // uniform base
            __builtin_amdgcn_global_load_lds((global_cptr)(uniform_flat(src) + dma_lane_off),
                                             (lds_ptr)&lds[buf * TILE + q * 256], 16, 0, 0);
        }
    };

    // ---- local step first: the gradient values of the elements this lane's DMA requests bring in
    // (same blocks, same lane -> (row, 4 columns) map), and the update of those elements in LDS
    float4 gstage[PRO ? DMA_PER_WAVE : 1];
    auto load_gdma = [&](int64_t tile) {
#pragma unroll
        for (int i = 0; i < (PRO ? DMA_PER_WAVE : 0); ++i) {
            const int q = w + 8 * i;
            const int s = q / (KB / 4), kq = q % (KB / 4);
            const float4 *src = g + (int64_t)(8 * kq) * ld4 + tile * (TC / 4) + s * 8;   // uniform base
            gstage[i] = *(const float4 *)(uniform_flat(src) + dma_lane_off);
        }
    };
    auto apply_g = [&](int buf) {
#pragma unroll
        for (int i = 0; i < (PRO ? DMA_PER_WAVE : 0); ++i) {
            const int q = w + 8 * i;
            const int kq = q % (KB / 4);
            const float eta = lr.at(8 * kq + 2 * (lane >> 4) + ((lane >> 3) & 1));
            float4 *p = (float4 *)&lds[buf * TILE + q * 256 + 4 * lane];
            float4 v = *p;
            v.x = fmaf(-eta, gstage[i].x, v.x);
            v.y = fmaf(-eta, gstage[i].y, v.y);
            v.z = fmaf(-eta, gstage[i].z, v.z);
            v.w = fmaf(-eta, gstage[i].w, v.w);
            *p = v;
        }
    };

    int64_t tile = blockIdx.x;
    if (tile >= n_tiles) return;
    if (DMA) {
        dma(tile, 0);
        load_gdma(tile);
        __builtin_amdgcn_s_waitcnt(0);
        asm volatile("" ::: "memory");
        apply_g(0);
    } else {
        fetch(tile);
        commit(0);
    }
    __syncthreads();

    // epilogue addressing: uniform base per (tile, wave, v) + one lane offset
    const uint32_t epi_lane_off = 4u * (uint32_t)(4 * (lane >> 5) * ld + (lane & 31));

    int buf = 0;
    for (; tile < n_tiles; tile += gridDim.x) {
        const int64_t next = tile + gridDim.x;
        if (next < n_tiles) {
            if (DMA) {
                dma(next, buf ^ 1);
                load_gdma(next);
            } else {
                fetch(next);
            }
        }
        if (PRO) __builtin_amdgcn_sched_barrier(0);      // nothing that consumes those values moves up here

        // request the gradient values, multiply, correct and store; the stores come after the barrier and drain under the next
        // tile's multiplies
        const int64_t col0 = tile * TC + 32 * w;
        float gv[16];
        if (ORDER == DBW_ORDER_CTA && HAS_G) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row0 = 8 * (v / 4) + (v & 3);                           // uniform
                const float *gb = gs + (int64_t)row0 * ld + col0;
                if (FULL) {
                    gv[v] = *(const float *)(uniform_flat(gb) + epi_lane_off);
                } else {
                    const bool ok = row0 + 4 * (lane >> 5) < N && col0 + (lane & 31) < dcols;
                    gv[v] = ok ? *(const float *)(uniform_flat(gb) + epi_lane_off) : 0.f;
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        // B fragments come from LDS eight k-steps at a time, one group ahead of the multiplies
        const float *bbase = &lds[buf * TILE + w * KB * 64 + lane];
        float bq[2][8];
#pragma unroll
        for (int j = 0; j < 8; ++j) bq[0][j] = bbase[j * 64];
#pragma unroll
        for (int q = 0; q < KB / 8; ++q) {
            if (q + 1 < KB / 8) {
#pragma unroll
                for (int j = 0; j < 8; ++j) bq[(q + 1) & 1][j] = bbase[(8 * (q + 1) + j) * 64];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wreg[8 * q + j], bq[q & 1][j], acc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }

        // the next tile is complete in LDS before anybody starts on it
        if (next < n_tiles && !DMA) commit(buf ^ 1);
        if (DMA) __builtin_amdgcn_s_waitcnt(0);      // the tile written by global_load_lds has landed
        if (PRO) {
            asm volatile("" ::: "memory");               // LDS reads below stay behind the wait
            if (next < n_tiles) apply_g(buf ^ 1);
        }
        __syncthreads();
        buf ^= 1;
        // local SGD correction and store, 32 consecutive columns per row
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row0 = 8 * (v / 4) + (v & 3);
            float r = acc[v];
            if (ORDER == DBW_ORDER_CTA && HAS_G) {
                const int row = row0 + 4 * (lane >> 5);
                r = fmaf(-lr.at(FULL || row < N ? row : 0), gv[v], r);
            }
            float *ob = out + (int64_t)row0 * ld + col0;
            if (FULL || (row0 + 4 * (lane >> 5) < N && col0 + (lane & 31) < dcols))
                *(float *)(const_cast<char *>(uniform_flat(ob)) + epi_lane_off) = r;
        }
    }
}

// Up to NB workers on rows off 16-byte boundaries.  A thread keeps the sums of all workers for V columns in registers and
// takes in one worker's values after the other, with the column of P that goes with them: wave-uniform, through the scalar
// cache.  Every value is read once, nothing is staged, and rows of padding cost multiplies only.  V = 4: 16-byte accesses on
// 4-byte boundaries; the last group of a row is moved back to end with it (columns computed twice, to the same values).
typedef float vf4_any __attribute__((ext_vector_type(4), aligned(4)));

constexpr int COLUMN_THREADS = 256;
template <int NB, int V, int ORDER, bool HAS_G, class LR>
__global__ __launch_bounds__(COLUMN_THREADS) void mix_dense_columns(int N, int64_t d, int64_t ld, const float *__restrict__ Wsw,
                                                                    const float *__restrict__ x, const float *__restrict__ g,
                                                                    float *__restrict__ out, LR lr)
{
    int64_t c = V * ((int64_t)blockIdx.x * COLUMN_THREADS + threadIdx.x);
    if (c >= d) return;
    c = min(c, d - V);
    auto load = [&](const float *row, float (&v)[V]) {
        if constexpr (V == 4) {
            const vf4_any q = *(const vf4_any *)(row + c);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = q[e];
        } else {
            v[0] = row[c];
        }
    };
    constexpr bool EPI = ORDER == DBW_ORDER_CTA && HAS_G;
    float acc[NB][V], late[EPI ? NB : 1][V];                         // (gradients of the epilogue: under way during the sums)
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if (EPI) load(g + (int64_t)min(i, N - 1) * ld, late[EPI ? i : 0]);
#pragma unroll
        for (int e = 0; e < V; ++e) acc[i][e] = 0.f;
    }
#pragma unroll 2
    for (int j = 0; j < N; ++j) {
        float v[V], gv[V];
        load(x + (int64_t)j * ld, v);
        if (ORDER == DBW_ORDER_ATC && HAS_G) {
            load(g + (int64_t)j * ld, gv);
            const float eta = lr.at(j);
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = fmaf(-eta, gv[e], v[e]);
        }
        const float *p = Wsw + (j >> 1) * 64 + 32 * (j & 1);       // column j of P, rows 0 .. 31
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int e = 0; e < V; ++e) acc[i][e] = fmaf(p[i], v[e], acc[i][e]);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if (i < N) {
            if (EPI) {
                const float eta = lr.at(i);
#pragma unroll
                for (int e = 0; e < V; ++e) acc[i][e] = fmaf(-eta, late[EPI ? i : 0][e], acc[i][e]);
            }
            float *o = out + (int64_t)i * ld + c;
            if constexpr (V == 4) *(vf4_any *)o = vf4_any{acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
            else o[0] = acc[i][0];
        }
    }
}

template <int NB, int V, int ORDER, bool HAS_G, class LR>
int launch_columns(dbw_ctx *c, const float *W, const float *x, const float *g, float *out, LR lr, hipStream_t s)
{
    const int64_t per = (int64_t)V * COLUMN_THREADS, blocks = (c->d + per - 1) / per;
    if (blocks > INT32_MAX) return DBW_ERR_UNSUPPORTED;
    dbw_timer tm(c, "mix_dense_columns", s);
    hipLaunchKernelGGL((mix_dense_columns<NB, V, ORDER, HAS_G, LR>), dim3((unsigned)blocks), dim3(COLUMN_THREADS), 0, s, c->N, c->d, c->ld, W,
                       x, g, out, lr);
    DBW_HIP(hipGetLastError());
    return DBW_OK;
}

template <int V, int ORDER, bool HAS_G, class LR>
int launch_columns_n(dbw_ctx *c, const float *W, const float *x, const float *g, float *out, LR lr, hipStream_t s)
{
    if (c->N <= 4) return launch_columns<4, V, ORDER, HAS_G, LR>(c, W, x, g, out, lr, s);
    if (c->N <= 8) return launch_columns<8, V, ORDER, HAS_G, LR>(c, W, x, g, out, lr, s);
    return launch_columns<16, V, ORDER, HAS_G, LR>(c, W, x, g, out, lr, s);
}

template <int ORDER, bool HAS_G, class LR>
int launch_fp32(dbw_ctx *c, const float *W, const float *x, const float *g, float *out, LR lr, hipStream_t s)
{
    // rows are padded to a multiple of four floats: the float4 that straddles column d is read whole and stored up to d
    const int64_t n_vec = (c->d + 3) / 4, n_tiles = (n_vec * 4 + TC - 1) / TC;
    if (n_tiles > INT32_MAX) return DBW_ERR_UNSUPPORTED;
    const int64_t grid = std::min<int64_t>(n_tiles, 256 * 2);     // two workgroups' tiles fill a compute unit's LDS
    const bool full = c->N == NPAD && c->d % TC == 0;
    dbw_timer tm(c, "mix_dense_kernel", s);
    if (full)
        hipLaunchKernelGGL((mix_dense_kernel<ORDER, HAS_G, true, LR>), dim3((unsigned)grid), dim3(DENSE_THREADS), 0, s,
                           c->N, n_vec, c->d, c->ld / 4, W, (const float4 *)x, (const float4 *)g, out, g, lr,
                           (int)n_tiles);
    else
        hipLaunchKernelGGL((mix_dense_kernel<ORDER, HAS_G, false, LR>), dim3((unsigned)grid), dim3(DENSE_THREADS), 0,
                           s, c->N, n_vec, c->d, c->ld / 4, W, (const float4 *)x, (const float4 *)g, out, g, lr,
                           (int)n_tiles);
    DBW_HIP(hipGetLastError());
    return DBW_OK;
}

template <int MB, int WAVES, int ORDER, bool HAS_G, bool WIDE, class LR>
int launch_split(dbw_ctx *c, const float *W, const float *x, const float *g, float *out, LR lr, hipStream_t s)
{
    using C = mixsplit::Cfg<MB, WAVES>;
    const int64_t n_tiles = (c->d + C::TC - 1) / C::TC;
    if (n_tiles > INT32_MAX) return DBW_ERR_UNSUPPORTED;
    dbw_timer tm(c, "mix_dense_split", s);
    const bool lines = c->ld % 32 == 0 && ((uintptr_t)x | (uintptr_t)out | (HAS_G ? (uintptr_t)g : 0)) % 128 == 0;
    const bool stream = lines && (HAS_G ? 12 : 8) * c->N * c->ld > mixsplit::CACHE_BYTES;
    // persistent: as many workgroups as the compute units' LDS holds
    const dim3 grid((unsigned)std::min<int64_t>(n_tiles, 256 * 8 / WAVES)), block(64 * WAVES);
    if (stream)
        hipLaunchKernelGGL((mixsplit::kernel<MB, WAVES, ORDER, HAS_G, WIDE, true, LR>), grid, block, 0, s, c->N, c->d, c->ld, W, x, g, out, lr, (int)n_tiles);
    else
        hipLaunchKernelGGL((mixsplit::kernel<MB, WAVES, ORDER, HAS_G, WIDE, false, LR>), grid, block, 0, s, c->N, c->d, c->ld, W, x, g, out, lr, (int)n_tiles);
    DBW_HIP(hipGetLastError());
    return DBW_OK;
}

template <int MB, int ORDER, bool HAS_G, bool WIDE, class LR>
int launch_mb(dbw_ctx *c, const float *W, const float *x, const float *g, float *out, LR lr, hipStream_t s)
{
    // Up to 64 workers two workgroups of four wavefronts per compute unit, with tiles of half the width, give shorter
    // vectors more even rounds of tiles; longer vectors want the longer pieces of a row (N = 60, four / eight waves:
    // 134 154 columns 23.0 / 25.7 us, 600 000 93 / 96, 1.2 M 180 / 176, 4 M 600 / 555).  The line, 24 tiles for each of 256
    // workgroups, is 786 432 columns there and where N = 60 crosses; N = 40, with more padding, would rather have four waves to
    // 1.5 M (114 / 119), and N = 24 off 16-byte boundaries, with tiles twice as wide, takes the same either way (1.5 M 82 / 78).
    if constexpr (MB <= 2)
        if (c->d <= 24 * 256 * (int64_t)mixsplit::Cfg<MB, 8>::TC) return launch_split<MB, 4, ORDER, HAS_G, WIDE, LR>(c, W, x, g, out, lr, s);
    return launch_split<MB, 8, ORDER, HAS_G, WIDE, LR>(c, W, x, g, out, lr, s);
}

template <int ORDER, bool HAS_G, class LR>
int launch(dbw_ctx *c, const float *W, const float *x, const float *g, float *out, LR lr, hipStream_t s)
{
    if (c->ld > DBW_DENSE_MAX_LD) return DBW_ERR_UNSUPPORTED;
    const bool wide = c->ld % 4 == 0 && (uintptr_t)x % 16 == 0 && (!HAS_G || (uintptr_t)g % 16 == 0);
    if (!wide) {
        // Up to 16 workers the 32 rows of the matrix instruction are mostly padding, of which the copies and splits below cost as
        // much as of the rest (d = 2 000 003 with gradients: N = 2 143 us, here 9.6; N = 8 143, 31.5; N = 16 144, 82; with N = 32 the
        // two come out even, and rows of 50 000 columns 10.3, 15).  Four columns per thread once that fills the chip (N = 16 x
        // 357 003 17.7 us with one, 15.5 with four; x 700 001 27.7, 22.9; x 5 001 7.2, 7.9).
        if (c->N <= 16) {
            if (c->d >= (int64_t)1 << 19) return launch_columns_n<4, ORDER, HAS_G, LR>(c, W, x, g, out, lr, s);
            return launch_columns_n<1, ORDER, HAS_G, LR>(c, W, x, g, out, lr, s);
        }
        switch (c->Npad) {
        case 32: return launch_mb<1, ORDER, HAS_G, false, LR>(c, W, x, g, out, lr, s);
        case 64: return launch_mb<2, ORDER, HAS_G, false, LR>(c, W, x, g, out, lr, s);
        case 128: return launch_mb<4, ORDER, HAS_G, false, LR>(c, W, x, g, out, lr, s);
        case 256: return launch_mb<8, ORDER, HAS_G, false, LR>(c, W, x, g, out, lr, s);
        default: return DBW_ERR_UNSUPPORTED;
        }
    }
    switch (c->Npad) {
    // Up to 32 workers the fp32 matrix instructions are far from being the bound and the rows of padding would only be
    // fetched and split: N = 10 x 134 154 columns 10.4 us against 13.3, x 4 M 116 against 184; N = 30 x 4 M 286 against 279.
    case 32: return launch_fp32<ORDER, HAS_G, LR>(c, W, x, g, out, lr, s);
    case 64: return launch_mb<2, ORDER, HAS_G, true, LR>(c, W, x, g, out, lr, s);
    case 128: return launch_mb<4, ORDER, HAS_G, true, LR>(c, W, x, g, out, lr, s);
    case 256: return launch_mb<8, ORDER, HAS_G, true, LR>(c, W, x, g, out, lr, s);
    default: return DBW_ERR_UNSUPPORTED;
    }
}

}  // namespace

int dbw_launch_mix_dense(dbw_ctx *c, const float *x, const float *g, float *out, float lr, const float *lr_vec,
                         hipStream_t s, const float *W)
{
    if (!W) W = c->Wdense;
    if (!W) return DBW_ERR_STATE;
    if (!g) return launch<DBW_ORDER_CTA, false>(c, W, x, g, out, dbw_lr_scalar{0.f}, s);
    if (lr_vec && c->order == DBW_ORDER_ATC) return launch<DBW_ORDER_ATC, true>(c, W, x, g, out, dbw_lr_vector{lr_vec}, s);
    if (lr_vec) return launch<DBW_ORDER_CTA, true>(c, W, x, g, out, dbw_lr_vector{lr_vec}, s);
    if (c->order == DBW_ORDER_ATC) return launch<DBW_ORDER_ATC, true>(c, W, x, g, out, dbw_lr_scalar{lr}, s);
    return launch<DBW_ORDER_CTA, true>(c, W, x, g, out, dbw_lr_scalar{lr}, s);
}
