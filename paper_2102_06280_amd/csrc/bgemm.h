// Batched fp32 GEMM on the matrix cores, one independent problem per worker:
//   C_w[m][n] = epilogue( sum_k A_w(m, k) * B_w(k, n) ),   w = blockIdx.z / splits
// Every worker has its own operands (its own parameters, its own mini-batch), which is
// what the per-worker gradient of Section 2.1 needs.
//
// Operands are described by small loader structs.  A loader splits the address of element
// (row, k) into a part that depends on the row only (`row_ctx`), a part that depends on k
// only (`k_ctx`) and a cheap combination (`load`), all in 32-bit arithmetic relative to
// the worker's base pointer, and states whether its elements are contiguous along k (KC)
// or along the row index.
// A dense operand that is contiguous along k (WIDE) is fetched eight k of a row per thread, two 16-byte loads on whatever
// 4-byte boundary the row starts.  For the others the global -> LDS copy assigns work so that one of the two indices is
// the same for a whole wavefront and the other runs with the lane: for a KC operand a wavefront reads 64
// consecutive k of one row, otherwise 64 consecutive rows of one k.  Loads are therefore
// coalesced; the context of the wave-uniform index is computed on the scalar unit, the
// per-lane context once per k-step (KC) or once per kernel (otherwise).
// The tile keeps the operand's natural layout in LDS.
//
// Workgroup: 256 threads = 4 wavefronts, tile BM x BN (64 x 64 or 32 x 128), k-step 64.  Each wavefront owns a 32 x 32
// part.  Two kernels:
//
// backward_kernel, split_kernel (weight and data gradients of dense layers): every value is split into
// three bf16 values (split_bf16.h) when the tile is written to LDS, as [plane][8 k][row][8 values], where a lane's
// fragment of v_mfma_f32_32x32x16_bf16 is one 128-bit read.  A thread therefore fetches eight consecutive k of a row
// at a time, of a row-contiguous operand with eight loads whose lanes run along the rows.  20 workers, batch 101,
// 617-301-75-26 on rows without padding: three weight gradients 42 us (fp32 matrix instructions and 4-byte loads 46), two
// data gradients 26 (26); 11 workers, batch 1 024, 161-185-185-24: 52 (61), 38 (44).  Small and large partial products
// are summed apart.
//
// kernel (forward products of dense layers, most data gradients that have a launch to themselves, convolution operands):
// 2 x 2 fragments of v_mfma_f32_16x16x4_f32 per wavefront (true fp32).  The sign of a forward product decides whole samples'
// gradients where it is next to zero, so its rounding is that of the chain and head kernels that compute the same layer;
// the split form gained nothing, since the fetches bound both.  The three forward products of the first example: 46 us
// (with 4-byte loads 113), of the second 59 (123).
//   A fragment: lane l holds A[m = l % 16][slot l / 16], B fragment: B[slot l / 16][n = l % 16]
//   D: 4 floats, d[v] = D[m = 4 * (l / 16) + v][n = l % 16]
// The four k-slots of instruction j (0..3) of a 16-wide k group are k = 4 * slot + j for
// both operands, which lets a k-contiguous operand fetch four instructions' worth of
// values with one 128-bit LDS read.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "split_bf16.h"

namespace bgemm {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 64, THREADS = 256;
constexpr int LDS_KC = BK + 4;                       // row stride of a k-contiguous tile [rows][68]
constexpr int lds_rc(int rows) { return rows + 4; }  // row stride of a row-contiguous tile [64][rows + 4]
constexpr int lds_floats(bool kc, int rows) { return kc ? rows * LDS_KC : BK * lds_rc(rows); }

// Dense operand.  KC: element (r, k) at p[w * stride + r * ld + k]; otherwise at
// p[w * stride + k * ld + r].  Offsets inside one worker's block fit 32 bits.
// ALIGNED (see aligned): the tile is fetched 16 bytes at a time without a guard.
template <bool KC_, bool ALIGNED_ = false>
struct Dense {
    static constexpr bool KC = KC_, ALIGNED = ALIGNED_, WIDE = KC_ && !ALIGNED_;
    const float *p;
    int64_t ld, stride;
    struct RowCtx { int off; bool ok; };
    struct KCtx { int off; bool ok; };
    __device__ __forceinline__ RowCtx row_ctx(int r, bool ok) const { return {KC ? r * (int)ld : r, ok}; }
    __device__ __forceinline__ KCtx k_ctx(int k, bool ok) const { return {KC ? k : k * (int)ld, ok}; }
    __device__ __forceinline__ float load(int w, const RowCtx &r, const KCtx &k) const
    {
        const bool ok = r.ok && k.ok;
        const float v = (p + w * stride)[ok ? r.off + k.off : 0];
        return ok ? v : 0.f;
    }
};

// Epilogue: optional per-column bias, ReLU, or masking by the sign of another matrix.
struct Epilogue {
    float *C;
    int64_t ldc, strideC;
    const float *bias;      // [n], per worker stride strideBias; nullptr = none
    int64_t strideBias;
    const float *mask;      // keep C[m][n] only where mask[m][n] > 0; nullptr = none
    int64_t ldmask, strideMask;
    int relu;
    __device__ __forceinline__ void store(int w, int /*split*/, int m, int n, float v) const
    {
        if (bias) v += bias[w * strideBias + n];
        if (relu) v = v > 0.f ? v : 0.f;
        if (mask) v = mask[w * strideMask + (int64_t)m * ldmask + n] > 0.f ? v : 0.f;
        C[w * strideC + (int64_t)m * ldc + n] = v;
    }
};

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// Eight consecutive floats, on any 4-byte boundary, of which the first `left` exist; the rest are zero.
__device__ __forceinline__ void load8(const float *src, int left, float *v)
{
    if (left >= 8) {
        const f32x4_any a = *(const f32x4_any *)src, b = *(const f32x4_any *)(src + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = a[j];
            v[4 + j] = b[j];
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = j < left ? src[j] : 0.f;
    }
}

// Whether every row of an operand starts on a 16-byte boundary and its contiguous extent divides by four.
template <bool KC>
inline bool aligned(const Dense<KC> &op, int rows, int K)
{
    return (uintptr_t)op.p % 16 == 0 && op.ld % 4 == 0 && op.stride % 4 == 0 && (KC ? K : rows) % 4 == 0;
}

// How a loader's operand is fetched: dense ones 16 bytes at a time (ALIGNED), dense ones that are contiguous along k eight
// elements at a time (WIDE), all others element by element.
template <class L>
struct fetch_kind {
    template <class T> static constexpr int test(decltype(T::WIDE) *) { return T::ALIGNED ? 2 : T::WIDE ? 1 : 0; }
    template <class T> static constexpr int test(...) { return 0; }
    static constexpr int value = test<L>(nullptr);
};
template <class L>
struct wide {
    static constexpr bool value = fetch_kind<L>::value == 1;
};
template <class L>
struct vectors {
    static constexpr bool value = fetch_kind<L>::value == 2;
};

// Global -> registers for a ROWS x 64 operand tile (ROWS / 4 elements per thread).
//   ALIGNED: elements 4 j .. 4 j + 3 are, with f = tid + 256 j, (row = f / 16, k = 4 (f % 16) ..) of a KC operand, otherwise
//   (row = 4 (f % (ROWS / 4)) .., k = f / (ROWS / 4)); in the place of a group outside the operand the first one is read and
//   replaced by zero when the tile is written to LDS (replaced at once, it would have to arrive before the multiplies)
//   WIDE: elements 8 u .. 8 u + 7 are (row = tid / 8 + 32 u, k = 8 (tid % 8) ..): eight lanes read 256 contiguous bytes
//   KC: element j of the thread is (row = wave + 4 j, k = lane)
//   RC: ROWS >= 64; element j is (row = lane + 64 (j % (ROWS / 64)), k = wave + 4 (j / (ROWS / 64)))
// `rows` holds the per-lane row contexts of an RC operand (computed once per kernel).
template <class L, int ROWS>
struct RowCache {
    typename L::RowCtx c[L::KC ? 1 : ROWS / 64];
};

template <class L, int ROWS>
__device__ __forceinline__ void make_rows(const L &op, int r0, int R, int lane, RowCache<L, ROWS> &rows)
{
    if (!L::KC) {
#pragma unroll
        for (int g = 0; g < ROWS / 64; ++g) {
            const int r = r0 + lane + 64 * g;
            rows.c[g] = op.row_ctx(r < R ? r : 0, r < R);
        }
    }
}

template <class L, int ROWS>
__device__ __forceinline__ void fetch_tile(const L &op, int w, int r0, int R, int k0, int K, int wave, int lane,
                                           const RowCache<L, ROWS> &rows, float (&v)[ROWS / 4], uint32_t &inside)
{
    static_assert(L::KC || ROWS >= 64, "a row-contiguous operand needs at least 64 tile rows");
    if constexpr (vectors<L>::value) {
        const float *base = op.p + w * op.stride;
        inside = 0;
#pragma unroll
        for (int j = 0; j < ROWS / 16; ++j) {
            const int f = 64 * wave + lane + 256 * j;
            const int r = r0 + (L::KC ? f / 16 : 4 * (f % (ROWS / 4))), k = k0 + (L::KC ? 4 * (f % 16) : f / (ROWS / 4));
            const bool ok = r < R && k < K;
            const f32x4 q = *(const f32x4 *)(base + (ok ? (L::KC ? r * (int)op.ld + k : k * (int)op.ld + r) : 0));
            inside |= (ok ? 1u : 0u) << j;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * j + e] = q[e];
        }
    } else if constexpr (wide<L>::value) {
        const float *base = op.p + w * op.stride;
        const int tid = 64 * wave + lane;
#pragma unroll
        for (int u = 0; u < ROWS / 32; ++u) {
            const int r = r0 + tid / 8 + 32 * u, k = k0 + 8 * (tid % 8), left = r < R ? K - k : 0;
            load8(base + (left > 0 ? r * (int)op.ld + k : 0), left, v + 8 * u);
        }
    } else if (L::KC) {
        const int k = k0 + lane;
        const typename L::KCtx kc = op.k_ctx(k < K ? k : 0, k < K);      // per lane, shared by all rows
#pragma unroll
        for (int j = 0; j < ROWS / 4; ++j) {
            const int r = r0 + wave + 4 * j;                                 // wave-uniform
            v[j] = op.load(w, op.row_ctx(r < R ? r : 0, r < R), kc);
        }
    } else {
        constexpr int RG = ROWS / 64;
#pragma unroll
        for (int j = 0; j < ROWS / 4; ++j) {
            const int k = k0 + wave + 4 * (j / RG);                          // wave-uniform
            v[j] = op.load(w, rows.c[j % RG], op.k_ctx(k < K ? k : 0, k < K));
        }
    }
}

template <class L, int ROWS>
__device__ __forceinline__ void commit_tile(float *lds, int wave, int lane, const float (&v)[ROWS / 4], uint32_t inside)
{
    if constexpr (vectors<L>::value) {
#pragma unroll
        for (int j = 0; j < ROWS / 16; ++j) {
            const int f = 64 * wave + lane + 256 * j;
            const bool ok = inside >> j & 1u;
            float *d = &lds[L::KC ? f / 16 * LDS_KC + 4 * (f % 16) : f / (ROWS / 4) * lds_rc(ROWS) + 4 * (f % (ROWS / 4))];
            *(f32x4 *)d = f32x4{ok ? v[4 * j] : 0.f, ok ? v[4 * j + 1] : 0.f, ok ? v[4 * j + 2] : 0.f, ok ? v[4 * j + 3] : 0.f};
        }
        return;
    }
    if constexpr (wide<L>::value) {
        const int tid = 64 * wave + lane;
#pragma unroll
        for (int q = 0; q < ROWS / 16; ++q)
            *(f32x4 *)&lds[(tid / 8 + 32 * (q / 2)) * LDS_KC + 8 * (tid % 8) + 4 * (q % 2)] =
                f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        return;
    }
#pragma unroll
    for (int j = 0; j < ROWS / 4; ++j) {
        if (L::KC)
            lds[(wave + 4 * j) * LDS_KC + lane] = v[j];
        else
            lds[(wave + 4 * (j / (ROWS / 64))) * lds_rc(ROWS) + lane + 64 * (j % (ROWS / 64))] = v[j];
    }
}

// Values of the four instructions of k group `kg` for the 16-row fragment at row `rbase`.
template <class L, int ROWS>
__device__ __forceinline__ f32x4 frag(const float *lds, int rbase, int kg, int lane)
{
    f32x4 f;
    if (L::KC) {
        f = *(const f32x4 *)&lds[(rbase + (lane & 15)) * LDS_KC + kg * 16 + 4 * (lane >> 4)];
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) f[j] = lds[(kg * 16 + 4 * (lane >> 4) + j) * lds_rc(ROWS) + rbase + (lane & 15)];
    }
    return f;
}

// blockIdx.z = worker * splits + split; a split covers k in [split * kper, (split + 1) * kper)
// (kper a multiple of BK) and hands its partial sum to the epilogue, which decides where it
// goes; with splits == 1 the result is final.
template <class LA, class LB, class EP, int BM, int BN>
__global__ __launch_bounds__(THREADS) void kernel(LA A, LB B, EP E, int M, int N, int K, int splits, int kper)
{
    static_assert((BM == 64 && BN == 64) || (BM == 32 && BN == 128), "supported tiles: 64 x 64, 32 x 128");
    static_assert(BM == 64 || LA::KC, "the 32-row tile needs a k-contiguous A operand");
    __shared__ __attribute__((aligned(16))) float As[lds_floats(LA::KC, BM)];
    __shared__ __attribute__((aligned(16))) float Bs[lds_floats(LB::KC, BN)];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = blockIdx.z / splits, split = blockIdx.z % splits;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    const int kbeg = split * kper, kend = min(K, kbeg + kper);
    constexpr int WM = BM / 32;                          // waves along m
    const int wm = (wave % WM) * 32, wn = (wave / WM) * 32;

    f32x4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    RowCache<LA, BM> arows;
    RowCache<LB, BN> brows;
    make_rows<LA, BM>(A, m0, M, lane, arows);
    make_rows<LB, BN>(B, n0, N, lane, brows);
    float ra[BM / 4], rb[BN / 4];
    uint32_t ina = 0, inb = 0;
    auto fetch = [&](int k0) {
        fetch_tile<LA, BM>(A, w, m0, M, k0, kend, wave, lane, arows, ra, ina);
        fetch_tile<LB, BN>(B, w, n0, N, k0, kend, wave, lane, brows, rb, inb);
    };
    fetch(kbeg);
    for (int k0 = kbeg; k0 < kend; k0 += BK) {
        __syncthreads();                       // previous tile fully consumed
        commit_tile<LA, BM>(As, wave, lane, ra, ina);
        commit_tile<LB, BN>(Bs, wave, lane, rb, inb);
        __syncthreads();
        if (k0 + BK < kend) fetch(k0 + BK);    // next tile's loads fly during the MFMAs
        if constexpr (fetch_kind<LA>::value || fetch_kind<LB>::value) __builtin_amdgcn_sched_barrier(0);   // nothing that consumes them moves up here
#pragma unroll
        for (int kg = 0; kg < BK / 16; ++kg) {
            f32x4 fa[2], fb[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) fa[a] = frag<LA, BM>(As, wm + 16 * a, kg, lane);
#pragma unroll
            for (int b = 0; b < 2; ++b) fb[b] = frag<LB, BN>(Bs, wn + 16 * b, kg, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[a][j], fb[b][j], acc[a][b], 0, 0, 0);
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int n = n0 + wn + 16 * b + (lane & 15);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + wm + 16 * a + 4 * (lane >> 4) + v;
                if (m < M && n < N) E.store(w, split, m, n, acc[a][b][v]);
            }
        }
}

// ---- the split kernel

// A 64 x 64 operand tile as units of (eight consecutive k, row), two of them per thread.
//   KC: unit u is (row tid / 8 + 32 u, k 8 (tid % 8)): eight lanes read 256 contiguous bytes of a row
//   otherwise unit u of wave `wave` is k group wave + 4 u of the rows, one per lane
template <bool KC>
struct SplitTile {
    static constexpr int ROWS = 64, UNITS = 2;
    static constexpr int PITCH = ROWS + 1;               // 16-byte groups between k groups: the lanes of a unit column differ in bank
    static constexpr int GROUPS = 8 * PITCH;

    float v[UNITS][8];

    __device__ __forceinline__ void fetch(const Dense<KC> &op, int w, int r0, int R, int k0, int K, int tid)
    {
        const float *base = op.p + w * op.stride;
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            if constexpr (KC) {
                const int r = r0 + tid / 8 + 32 * u, k = k0 + 8 * (tid % 8), left = r < R ? K - k : 0;
                load8(base + (left > 0 ? r * (int)op.ld + k : 0), left, v[u]);
            } else {
                // rows and k beyond the operand: any valid element; commit replaces those of k, those of a row reach
                // only results that are not stored
                const int kg = __builtin_amdgcn_readfirstlane(tid >> 6) + 4 * u;
                const uint32_t lane_off = (uint32_t)min(r0 + (tid & 63), R - 1);
#pragma unroll
                for (int j = 0; j < 8; ++j) v[u][j] = (base + (int64_t)min(k0 + 8 * kg + j, K - 1) * op.ld)[lane_off];
            }
        }
    }
    // k_left: k of the tile that exist (64 or more: all)
    __device__ __forceinline__ void commit(split_bf16::u32x4 *lds, int tid, int k_left)
    {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int kg = KC ? tid % 8 : (tid >> 6) + 4 * u, r = KC ? tid / 8 + 32 * u : tid & 63;
            if (!KC && k_left < 64) {
#pragma unroll
                for (int j = 0; j < 8; ++j) v[u][j] = 8 * kg + j < k_left ? v[u][j] : 0.f;
            }
            const split_bf16::planes p = split_bf16::split8(v[u]);
            split_bf16::u32x4 *d = lds + kg * PITCH + r;
            d[0] = p.h;
            d[GROUPS] = p.m;
            d[2 * GROUPS] = p.l;
        }
    }
    // fragment of the 32 rows from rbase on, step s (k 16 s .. + 15) of the tile
    static __device__ __forceinline__ split_bf16::planes frag(const split_bf16::u32x4 *lds, int rbase, int s, int lane)
    {
        const split_bf16::u32x4 *d = lds + (2 * s + (lane >> 5)) * PITCH + rbase + (lane & 31);
        return {d[0], d[GROUPS], d[2 * GROUPS]};
    }
};

constexpr int SPLIT_GROUPS = 3 * SplitTile<true>::GROUPS;     // LDS of one operand, in 16-byte groups

template <bool KCA, bool KCB, class EP>
__device__ __forceinline__ void split_tile(const Dense<KCA> &A, const Dense<KCB> &B, const EP &E, int M, int N, int K, int splits,
                                           int kper, int tile_n, int tile_m, int z, split_bf16::u32x4 *As, split_bf16::u32x4 *Bs)
{
    typedef SplitTile<KCA> TA;
    typedef SplitTile<KCB> TB;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = z / splits, split = z % splits;
    const int m0 = tile_m * 64, n0 = tile_n * 64;
    const int kbeg = split * kper, kend = min(K, kbeg + kper);
    const int wm = (wave % 2) * 32, wn = (wave / 2) * 32;

    split_bf16::f32x16 acc, small;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = small[v] = 0.f;
    TA ta;
    TB tb;
    if (kbeg < kend) {
        ta.fetch(A, w, m0, M, kbeg, kend, tid);
        tb.fetch(B, w, n0, N, kbeg, kend, tid);
    }
    for (int k0 = kbeg; k0 < kend; k0 += BK) {
        __syncthreads();                       // previous tile fully consumed
        ta.commit(As, tid, kend - k0);
        tb.commit(Bs, tid, kend - k0);
        __syncthreads();
        if (k0 + BK < kend) {                  // next tile's loads fly during the MFMAs
            ta.fetch(A, w, m0, M, k0 + BK, kend, tid);
            tb.fetch(B, w, n0, N, k0 + BK, kend, tid);
        }
        __builtin_amdgcn_sched_barrier(0);     // nothing that consumes them moves up here
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) split_bf16::mma32<true>(TA::frag(As, wm, s, lane), TB::frag(Bs, wn, s, lane), acc, small);
    }
    split_bf16::add_small(acc, small);
    const int n = n0 + wn + (lane & 31);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int m = m0 + wm + 8 * (v / 4) + 4 * (lane >> 5) + v % 4;
        if (m < M && n < N) E.store(w, split, m, n, acc[v]);
    }
}

// One problem set of split_tile: grid of tiles x workers x splits, flat.
template <bool KCA, bool KCB, class EP>
struct SplitProblem {
    Dense<KCA> A;
    Dense<KCB> B;
    EP E;
    int M, N, K, splits, kper;
    __host__ __device__ int tiles() const { return ((M + 63) / 64) * ((N + 63) / 64); }
    __device__ __forceinline__ void run(int id, split_bf16::u32x4 *As, split_bf16::u32x4 *Bs) const
    {
        const int tn = (N + 63) / 64, t = id % tiles();
        split_tile(A, B, E, M, N, K, splits, kper, t % tn, t / tn, id / tiles(), As, Bs);
    }
};
template <bool KCA, bool KCB, class EP>
inline SplitProblem<KCA, KCB, EP> split_problem(const Dense<KCA> &A, const Dense<KCB> &B, const EP &E, int M, int N, int K, int splits = 1)
{
    const int kper = (K + splits - 1) / splits;
    return {A, B, E, M, N, K, splits, (kper + BK - 1) / BK * BK};
}

// Column sums of the deltas dz [B][C] (the bias gradient): RG groups of rows, each with four independent partial sums,
// combined in a fixed order; a workgroup of RG * COLS threads takes COLS columns.
template <int RG, int COLS>
__device__ __forceinline__ void column_sums(int B, int C, const float *__restrict__ d, float *__restrict__ db, int c0, float *part)
{
    const int cl = threadIdx.x % COLS, rg = threadIdx.x / COLS, o = c0 + cl;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    if (o < C) {
        int b = rg;
        for (; b + 3 * RG < B; b += 4 * RG) {
            s0 += d[(int64_t)b * C + o];
            s1 += d[(int64_t)(b + RG) * C + o];
            s2 += d[(int64_t)(b + 2 * RG) * C + o];
            s3 += d[(int64_t)(b + 3 * RG) * C + o];
        }
        for (; b < B; b += RG) s0 += d[(int64_t)b * C + o];
    }
    part[rg * COLS + cl] = (s0 + s1) + (s2 + s3);
    __syncthreads();
    if (rg == 0 && o < C) {
        float s = part[cl];
        for (int r = 1; r < RG; ++r) s += part[r * COLS + cl];
        db[o] = s;
    }
}

// The backward pass of one dense layer, whose three parts all wait for the same deltas and for nothing else: data gradient
// (workgroups 0 .. nd - 1; none: nd = 0), weight gradient (the next nw) and bias gradient (the rest, `chunks` per worker; none:
// db = nullptr).  As launches of their own the parts of the narrow layers leave most of the chip idle one after the
// other: for 617-301-75-26 on 20 workers x 101 samples eight launches took 87 us, three take 50 (round 145 -> 122 us); for
// 161-185-185-24 on 11 x 1 024 111 -> 75, for 784-256-256-10 on 40 x 100 79 -> 60.
struct BiasSums {
    const float *dz;
    int64_t stride;
    float *db;
    int64_t stride_db;
    int B, C, chunks;           // chunks of 8 columns (batches of 512 and more: 32 groups of rows) or of 32 (8 groups)
};
constexpr int LONG_BATCH = 512;
template <class EP, class EPD>
__global__ __launch_bounds__(THREADS, 3) void backward_kernel(SplitProblem<false, false, EP> wg, SplitProblem<true, false, EPD> dg, BiasSums bs,
                                                              int nd, int nw)
{
    __shared__ __attribute__((aligned(16))) split_bf16::u32x4 As[SPLIT_GROUPS];
    __shared__ __attribute__((aligned(16))) split_bf16::u32x4 Bs[SPLIT_GROUPS];
    const int id = blockIdx.x;
    if (id < nd) {
        dg.run(id, As, Bs);
    } else if (id < nd + nw) {
        wg.run(id - nd, As, Bs);
    } else {
        const int c = (id - nd - nw) % bs.chunks, w = (id - nd - nw) / bs.chunks;
        const float *d = bs.dz + w * bs.stride;
        float *db = bs.db + w * bs.stride_db;
        if (bs.B >= LONG_BATCH) column_sums<32, 8>(bs.B, bs.C, d, db, 8 * c, (float *)As);
        else column_sums<8, 32>(bs.B, bs.C, d, db, 32 * c, (float *)As);
    }
}

template <class EP, class EPD>
inline hipError_t launch_backward(const SplitProblem<false, false, EP> &wg, const SplitProblem<true, false, EPD> *dg, const BiasSums &bs,
                                  int workers, hipStream_t s)
{
    const int nd = dg ? dg->tiles() * workers * dg->splits : 0, nw = wg.tiles() * workers * wg.splits, nb = bs.db ? bs.chunks * workers : 0;
    hipLaunchKernelGGL((backward_kernel<EP, EPD>), dim3(nd + nw + nb), dim3(THREADS), 0, s, wg, dg ? *dg : SplitProblem<true, false, EPD>{},
                       bs, nd, nw);
    return hipGetLastError();
}

// BM = 32 uses 32 x 128 tiles (for problems with at most 32 rows), otherwise 64 x 64.
template <int BM, class LA, class LB, class EP>
inline hipError_t launch(const LA &A, const LB &B, const EP &E, int M, int N, int K, int batch, hipStream_t s,
                         int splits = 1)
{
    constexpr int BN = BM == 32 ? 128 : 64;
    int kper = (K + splits - 1) / splits;
    kper = (kper + BK - 1) / BK * BK;
    const dim3 grid((N + BN - 1) / BN, (M + BM - 1) / BM, batch * splits);
    hipLaunchKernelGGL((kernel<LA, LB, EP, BM, BN>), grid, dim3(THREADS), 0, s, A, B, E, M, N, K, splits, kper);
    return hipGetLastError();
}

// The data gradient alone (its layer's weight gradient has another kernel).
template <class EP>
__global__ __launch_bounds__(THREADS, 3) void split_kernel(SplitProblem<true, false, EP> p)
{
    __shared__ __attribute__((aligned(16))) split_bf16::u32x4 As[SPLIT_GROUPS];
    __shared__ __attribute__((aligned(16))) split_bf16::u32x4 Bs[SPLIT_GROUPS];
    p.run(blockIdx.x, As, Bs);
}
template <class EP>
inline hipError_t launch_split(const SplitProblem<true, false, EP> &p, int workers, hipStream_t s)
{
    hipLaunchKernelGGL(split_kernel<EP>, dim3(p.tiles() * workers * p.splits), dim3(THREADS), 0, s, p);
    return hipGetLastError();
}

}  // namespace bgemm
