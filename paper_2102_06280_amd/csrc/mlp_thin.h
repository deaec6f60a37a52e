// Fully connected layers on short batches (up to 255 samples per worker), all workers in one launch
// (Section 2.1, stochastic gradient of the local loss):
//   forward_kernel         a_l[s][n] = act(sum_k a_{l-1}[s][k] W_l[n][k] + b_l[n])
//   forward_kernel (BACK)  dz_{l-1}[s][n] = sum_k dz_l[s][k] W_l[k][n] where a_{l-1}[s][n] > 0 (the gradient of the input: everywhere)
//   wgrad_kernel           dW_l[m][n] = sum_s dz_l[s][m] a_{l-1}[s][n],   db_l[m] = sum_s dz_l[s][m]
// With so few samples the tiled GEMM kernel (bgemm.h) spends its time on LDS round trips and
// barriers: a 64 x 784 x 200 product per worker reached a fifth of the matrix rate.  Here every
// operand goes from global memory straight into matrix-instruction fragments
// (v_mfma_f32_16x16x4_f32; A: lane l holds A[m = l % 16][k = l / 16], B: B[k = l / 16][n = l % 16],
// D: d[v] = D[m = 4 (l / 16) + v][n = l % 16]) with 128-bit loads on any 4-byte boundary, so that widths need not divide by anything.
//
// forward: both operands are contiguous along k.  The instruction does not care which four k a
// step stands for, so lane (l16, lq) loads k = 16 c + 4 lq .. + 3 of its row with one load, and
// element t of that load feeds step t of chunk c (that step then covers k = 16 c + 4 lq' + t for
// lq' = 0..3).  A workgroup owns up to 64 samples x 32 or 16 outputs of one worker; its eight wavefronts
// take every eighth chunk of 16 k, and their accumulators are added through LDS in a fixed order.  What bounds it are the matrix
// instructions of the compute unit with most workgroups, hence the tiles and the parts of the reduction that thin_plan picks: 1568 -> 128
// on 16 workers x 50 samples, 64 tiles of 32 outputs, 24 us, in two parts of tiles of 16 12.
// BACK: the weights are contiguous along the outputs; a lane loads the CB consecutive outputs of each of its four k, and its
// values go to CB different accumulators.
//
// wgrad: both operands are contiguous along their output index; the layout trick of mlp_wgrad.h
// (a lane's four consecutive outputs go to four different tiles) applies, but with at most 16 groups
// of four samples a tile is too little work to share: every wavefront owns a 32 x 64 tile, fetches
// all its samples at once (of more than 64: 36 or 32 at a time, summed apart), multiplies and stores, with no LDS and no barrier.
//
// Widths or rows that are no multiple of four floats, and batches of 65 to 255 samples, took bgemm.h (and several launches for what
// is one here); rounds, before and now: 617-301-75-10 on 20 workers x 101 samples 96 / 75 us, 783-200-10 on 32 x 50 69 / 47,
// 333-77-55-10 on 12 x 17 47 / 35, 100-99-98-97-10 on 8 x 50 73 / 42, 784-200-10 on 32 x 128 85 / 73, 784-300-10 on 4 x 129 52 / 34.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fc_head.h"
#include "mlp_thin_plan.h"
#include "mlp_wgrad.h"

namespace mlpthin {

using fchead::f32x4;
using fchead::pick;
constexpr int XCDS = 8;
constexpr int FWD_THREADS = 64 * FWD_WAVES;

struct FwdArgs {
    int B, K, N, workers, relu;          // samples, inputs (four or more) and outputs
    int splits, kper;                    // parts of the reduction, of kper chunks of 16 k
    const float *a;                      // a_{l-1} [B][a_ld] at a + w * a_stride
    int64_t a_ld, a_stride;
    const float *params;                 // worker rows of stride p_stride; W [N][K] at w_off, b [N] at b_off
    int64_t p_stride, w_off, b_off;
    float *out;                          // a_l [B][out_ld] at out + w * out_stride; splits > 1: sums [split][B][out_ld], without bias and ReLU
    int64_t out_ld, out_stride;
    const float *mask;                   // BACK: a_{l-1}, laid out like out: the result is kept where it is positive (null: everywhere)
};

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2_any __attribute__((ext_vector_type(2), aligned(4)));

// grid = (tiles of 16 CB outputs x workers, rounded up to a multiple of XCDS and renumbered so that one XCD receives consecutive
// tiles: the tiles of a worker read the same samples through the same L2; blocks of samples; splits).
template <int RB, int CB, bool BACK = false>
__global__ __launch_bounds__(FWD_THREADS) void forward_kernel(FwdArgs g)
{
    constexpr int WAVES = FWD_WAVES;
    constexpr int TM = 16 * RB, TN = 16 * CB, TP = TN + 4;
    __shared__ __attribute__((aligned(16))) float red[WAVES / 2][TM * TP];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles = (g.N + TN - 1) / TN;
    const int per = gridDim.x / XCDS, id = (blockIdx.x % XCDS) * per + blockIdx.x / XCDS;
    if (id >= tiles * g.workers) return;
    const int t = id % tiles, w = id / tiles, split = blockIdx.z;
    const int m0 = TM * blockIdx.y, n0 = TN * t;

    // rows beyond the batch and outputs beyond the layer: any valid row instead, never stored
    const float *pa[RB], *pb[BACK ? 1 : CB];
#pragma unroll
    for (int i = 0; i < RB; ++i) pa[i] = g.a + w * g.a_stride + (int64_t)min(m0 + 16 * i + l16, g.B - 1) * g.a_ld + 4 * lq;
    const int col = n0 + CB * l16;                   // BACK: the lane's first output
    const float *wp = g.params + w * g.p_stride + g.w_off;
    if constexpr (BACK) {
        pb[0] = wp + (int64_t)(4 * lq) * g.N + min(col, g.N - CB);
    } else {
#pragma unroll
        for (int j = 0; j < CB; ++j) pb[j] = wp + (int64_t)min(n0 + 16 * j + l16, g.N - 1) * g.K + 4 * lq;
    }
    // the weights of the lane's four k from k on, of which `left` exist (the rest: zero)
    auto weights = [&](int k, int left, f32x4 (&y)[CB]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float *p = pb[0] + (int64_t)(k + (e < left ? e : left > 0 ? 0 : -4 * lq)) * g.N;
            if constexpr (CB == 2) {
                const f32x2_any v = *(const f32x2_any *)p;
                y[0][e] = e < left ? (col > g.N - 2 ? v[1] : v[0]) : 0.f;         // the pair was moved back to end with the row
                y[1][e] = e < left ? v[1] : 0.f;
            } else {
                y[0][e] = e < left ? *p : 0.f;
            }
        }
    };

    f32x4 acc[RB][CB];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const f32x4 (&x)[RB], const f32x4 (&y)[CB]) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
                for (int j = 0; j < CB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i][e], y[j][e], acc[i][j], 0, 0, 0);
    };

    // whole chunks of 16 k: of the split's, number wave, wave + WAVES, ... are this wavefront's, the next one in flight
    // while one is multiplied (deeper prefetch was slower: 24 loads per wavefront queued before the first multiply took
    // 6 us to issue, and the products then ran behind the transfers instead of under them)
    const int all = g.K / 16, c0 = split * g.kper, c1 = min(all, c0 + g.kper);
    const int mine = c1 - c0 > wave ? (c1 - c0 - wave + WAVES - 1) / WAVES : 0;
    f32x4 ra[RB], rb[CB];
    auto fetch = [&](int n) {                 // this wavefront's n-th chunk
        const int k = 16 * (c0 + wave + WAVES * n);
#pragma unroll
        for (int i = 0; i < RB; ++i) ra[i] = *(const f32x4_any *)(pa[i] + k);
        if constexpr (BACK) {
            weights(k, 4, rb);
        } else {
#pragma unroll
            for (int j = 0; j < CB; ++j) rb[j] = *(const f32x4_any *)(pb[j] + k);
        }
    };
    if (mine > 0) fetch(0);
    for (int n = 0; n < mine; ++n) {
        f32x4 x[RB], y[CB];
#pragma unroll
        for (int i = 0; i < RB; ++i) x[i] = ra[i];
#pragma unroll
        for (int j = 0; j < CB; ++j) y[j] = rb[j];
        if (n + 1 < mine) fetch(n + 1);
        multiply(x, y);
    }
    // the last, partial chunk: a lane's four k are read where the row still has four, and those beyond the row are zero
    if (g.K % 16 != 0 && split == g.splits - 1 && (c1 - c0) % WAVES == wave) {
        const int left = g.K - 16 * all - 4 * lq;                // of the lane's four k, the first `left` exist
        const int back = left >= 4 ? 0 : 4 - left;               // read that many earlier (lanes without any: the row's last four)
        auto tail = [&](const float *p) {
            const f32x4 v = *(const f32x4_any *)(p + 16 * all - back);
            f32x4 r;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float q = 0.f;
#pragma unroll
                for (int b = 0; b + e < 4; ++b) q = back == b ? v[e + b] : q;
                r[e] = q;
            }
            return r;
        };
        f32x4 x[RB], y[CB];
#pragma unroll
        for (int i = 0; i < RB; ++i) x[i] = tail(pa[i]);
        if constexpr (BACK) {
            weights(16 * all, left, y);
        } else {
#pragma unroll
            for (int j = 0; j < CB; ++j) y[j] = tail(pb[j]);
        }
        multiply(x, y);
    }

    // the four results that this thread stores; their bias, or what masks them, arrives during the sums below (of the last, partial group of a
    // row the row's last four: no condition stands in the way of the load)
    static_assert(TM * (TN / 4) <= FWD_THREADS, "four results to a thread");
    const int er = tid / (TN / 4), ec = n0 + 4 * (tid % (TN / 4)), left = g.N - ec;
    const int64_t row_at = (int64_t)min(m0 + er, g.B - 1) * g.out_ld;
    const bool masked = BACK && g.mask;
    const float *late_at = masked ? g.mask + w * g.out_stride + row_at : wp + (BACK ? 0 : g.b_off - g.w_off);
    f32x4 late = {0.f, 0.f, 0.f, 0.f};
    if (g.N >= 4) late = *(const f32x4_any *)(late_at + min(ec, g.N - 4));

    // ---- the eight partial tiles: wavefronts 4..7 hand theirs to 0..3 through LDS, which add them and put
    // the sums back; then all threads add the four sums in order, bias, ReLU, 128-bit stores.
    // Register v of accumulator (i, j), lane (l16, lq): row 16 i + 4 lq + v, column 16 j + l16.
    auto slot = [&](int i, int j, int v) { return (16 * i + 4 * lq + v) * TP + (BACK ? CB * l16 + j : 16 * j + l16); };
    if (wave >= WAVES / 2) {
        float *dst = red[wave - WAVES / 2];
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) dst[slot(i, j, v)] = acc[i][j][v];
    }
    __syncthreads();
    if (wave < WAVES / 2) {          // reads and writes the same words of its own slot: no other wavefront touches them
        float *dst = red[wave];
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) dst[slot(i, j, v)] += acc[i][j][v];
    }
    __syncthreads();
    if (er >= TM || m0 + er >= g.B || left <= 0) return;
    f32x4 v = *(const f32x4 *)&red[0][er * TP + ec - n0];
#pragma unroll
    for (int q = 1; q < WAVES / 2; ++q) v += *(const f32x4 *)&red[q][er * TP + ec - n0];
    if (left < 4) {                  // (one group of a row)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (c < left) late[c] = late_at[ec + c];
    }
    if (BACK) {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = !masked || late[c] > 0.f ? v[c] : 0.f;
    } else if (g.splits == 1) {
        v += late;
        if (g.relu) {
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = fmaxf(v[c], 0.f);
        }
    }
    float *__restrict__ out = g.out + w * g.out_stride + (int64_t)split * g.B * g.out_ld + row_at + ec;
    if (left >= 4) {
        *(f32x4_any *)out = v;
    } else {
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (c < left) out[c] = v[c];
    }
}

// Weight (and bias) gradients for batches of at most 4 GROUPS <= 64 samples: mlpwgrad::Args with splits = 1 and
// tiles of 32 rows x 64 columns, one tile per wavefront (a lane loads two consecutive outputs of dz and four of a:
// narrow layers lose less to padding on the row side than with mlp_wgrad.h's 64 x 32, and a lane's four columns
// leave as one 128-bit store).  grid = head_blocks x workers + ceil(tiles x workers / 4) workgroups of four
// wavefronts, each part rounded up to a multiple of XCDS; the workgroups in front of the tiles add the head's
// per-chunk sums as in mlp_wgrad.h.
// Sums of at most 32 samples start from zero and are added afterwards: less rounding than in one long sum.  LONG: more than 64 samples, 4 GROUPS at a
// time, in sums of half of that.  Error of dW and db against 64 bits in 1e-7, bgemm.h / sums of whole steps / here: 64-33 on 200 samples 1.38 1.41 /
// 1.29 1.48 / 1.17 1.15, 617-301 on 101 1.91 1.24 / 1.83 1.12 / 1.80 1.06, 333-77 on 60 (one sum) 1.77 1.24 / 1.79 1.14 / 1.67 1.12.  (A third level of
// sums and steps of 12 samples: 784-300 on 200 2.97 -> 2.94.)  With 36 or 32 samples in flight instead of 64 three wavefronts to a SIMD have
// registers for LONG (784-512 on 32 workers x 128 samples 66 us, 76 with 52 or 64 and sums apart).  The bound on the wavefronts keeps the sums out
// of accumulation registers, which they would need besides the others: 784-200-10 on 32 x 64 samples 46.8 -> 46.3 us a round.
constexpr int WG_TM = 32, WG_TN = 64;
template <int GROUPS, bool LONG>
__global__ __launch_bounds__(mlpwgrad::THREADS, GROUPS == 4 ? 1 : 3) void wgrad_kernel(mlpwgrad::Args g, fchead::Args h, int chunks, int head_blocks)
{
    constexpr int TM = WG_TM, TN = WG_TN, WAVES = mlpwgrad::WAVES;
    typedef float vec2 __attribute__((ext_vector_type(2)));
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles = pick(g.tile_begin, g.layers + 1);
    const int wave_tiles = tiles * g.workers, tile_wgs = (wave_tiles + WAVES - 1) / WAVES;
    const int head_grid = gridDim.x - (tile_wgs + XCDS - 1) / XCDS * XCDS;
    if ((int)blockIdx.x < head_grid) {                          // the whole workgroup
        const int hid = blockIdx.x;
        if (hid < head_blocks * g.workers) fchead::reduce_body(h, chunks, hid % head_blocks, hid / head_blocks);
        return;
    }
    const int b = blockIdx.x - head_grid, per = (gridDim.x - head_grid) / XCDS, id = (b % XCDS) * per + b / XCDS;
    if (id >= tile_wgs) return;
    const int wt = id * WAVES + wave;
    if (wt >= wave_tiles) return;                               // no barrier below
    // With the average on the way the workers of a tile run next to each other, on one XCD, whose L2 then holds the rows that they read of
    // one another: 64 workers, 784-500-10, batch 16, the round 116 us with the tiles of a worker together, 86 so, 784-200-10, batch 64,
    // 6 neighbours 83, 79; 20 on a ring, whose rows fit anywhere, 37.7, 39.5.
    const bool mix = g.avg.x != nullptr;
    const int bx = mix ? wt / g.workers : wt % tiles, w = mix ? wt % g.workers : wt / tiles;
    int l = 1;
    while (l < g.layers && bx >= pick(g.tile_begin, l + 1)) ++l;
    const int N = pick(g.n_cols, l), H = pick(g.n_rows, l), ntn = (N + TN - 1) / TN;
    const int t = bx - pick(g.tile_begin, l), m0 = TM * (t / ntn), n0 = TN * (t % ntn);
    const bool bias = pick(g.want_db, l) && n0 == 0;
    // A pair of rows or group of columns that sticks out over the matrix is moved back to end with it (what it shares with the one before
    // is computed twice, to the same values); one that lies beyond it is the last one, never stored.
    const bool rows_ok = m0 + 2 * l16 < H, cols_ok = n0 + 4 * l16 < N;
    const int ncol = min(n0 + 4 * l16, N - 4);
    const float *__restrict__ dz = g.dz + w * g.dz_stride + pick(g.dz_off, l) + min(m0 + 2 * l16, H - 2);
    const float *__restrict__ av = pick(g.a, l) + w * pick(g.a_stride, l) + ncol;
    const int64_t a_ld = pick(g.a_ld, l);

    // group u = samples 4 u .. 4 u + 3, lane group lq takes sample 4 u + lq; a sample beyond the batch: a valid
    // row, zeroed (every load unconditional: loads under a condition each cost a register move per element)
    average::Row nb{};
    if (mix) nb = average::row(g.avg, w);
    // row block i, column block j: tile row 2 m + i, tile column 4 n + j for the instruction's indices m, n
    constexpr int APART = LONG ? (GROUPS + 1) / 2 : 8;          // groups whose sum is formed from zero
    f32x4 acc[2][4], sum[2][4];
    vec2 dacc = {0.f, 0.f}, dsum = dacc;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto add = [&] {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                sum[i][j] += acc[i][j];
                acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        dsum += dacc;
        dacc = vec2{0.f, 0.f};
    };
    int s0 = 0;
    do {
        vec2 x[GROUPS];
        f32x4 y[GROUPS];
#pragma unroll
        for (int u = 0; u < GROUPS; ++u) {
            const int sm = s0 + 4 * u + lq, sl = sm < g.B ? sm : 0;
            x[u] = *(const f32x2_any *)(dz + (int64_t)sl * H);
            y[u] = *(const f32x4_any *)(av + (int64_t)sl * a_ld);
        }
        __builtin_amdgcn_sched_barrier(0); // every load in flight before the first multiply (left alone, the compiler
                                           // saves registers by fetching a few groups at a time: 18.1 against 17.6 us)
#pragma unroll
        for (int u = 0; u < GROUPS; ++u) {
            const bool first = !LONG && u < APART;
            vec2 xv = x[u];
            f32x4 yv = y[u];
            if (s0 + 4 * u + lq >= g.B) {
                xv = vec2{0.f, 0.f};
                yv = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            (first ? dsum : dacc) += xv;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    f32x4 &to = first ? sum[i][j] : acc[i][j];
                    to = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[i], yv[j], to, 0, 0, 0);
                }
            if (LONG ? (u + 1) % APART == 0 || u + 1 == GROUPS : GROUPS > APART && u + 1 == GROUPS) add();
        }
        s0 += 4 * GROUPS;
    } while (LONG && s0 < g.B);
    // register r of (i, j), lane (l16, lq): tile row 2 (4 lq + r) + i, tile column 4 l16 + j
    float *__restrict__ out = g.grads + w * g.g_stride + pick(g.w_off, l);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        f32x4 v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = f32x4{sum[i][0][r], sum[i][1][r], sum[i][2][r], sum[i][3][r]};
        if (mix) {
            uint32_t off[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) off[r] = 4u * (uint32_t)((min(m0 + 2 * (4 * lq + r), H - 2) + i) * N + ncol);
            average::apply<f32x4, 4>(g.avg, nb, w, pick(g.w_off, l), off, v);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int first = m0 + 2 * (4 * lq + r);
            if (cols_ok && first < H) *(f32x4_any *)(out + (int64_t)(min(first, H - 2) + i) * N + ncol) = v[r];
        }
    }
    if (bias) {
        vec2 v[1];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            dsum[i] += __shfl_xor(dsum[i], 16, 64);
            dsum[i] += __shfl_xor(dsum[i], 32, 64);
        }
        v[0] = dsum;
        if (lq == 0 && rows_ok) {
            const int64_t at = (int64_t)H * N + min(m0 + 2 * l16, H - 2);
            if (mix) {
                const uint32_t off[1] = {(uint32_t)(4 * at)};
                average::apply<vec2, 1>(g.avg, nb, w, pick(g.w_off, l), off, v);
            }
            *(f32x2_any *)(out + at) = v[0];
        }
    }
}

}  // namespace mlpthin
