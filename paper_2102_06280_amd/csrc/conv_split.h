// Stride-1 'same' convolutions and their weight gradients on the bf16 matrix instructions, every fp32 value split into three
// bf16 values (split_bf16.h), for any number of channels and image size that fits LDS (forward_lds, wgrad_lds below).
//
// Forward (and, with flipped filters, the data gradient): one workgroup takes 64 pooling windows = 256 output pixels,
// of one sample or of several small ones, and all output channels (up to 64; more in further workgroups).
//   out[co][p] = sum over taps t and channels c of  Wt[co][t][c] * in[p + t][c]
// The reduction runs over channels inside a tap, 16 at a time, so that the eight values of a lane's fragment are
// eight channels of ONE pixel: the image lies in LDS as [plane][8 channels][position][8 values], split once when
// it is copied there, and the fragment of any pixel shifted by any tap is one aligned 128-bit read, with no bounds
// check (zero halo) and no patch matrix.  The filters are brought into the same order, split, once per round
// (prepare_kernel) and stream through LDS, two taps (or four) at a time, by loads that bypass the registers.
//
// The 32 columns of a fragment are eight 2 x 2 pooling windows, four lanes each: ReLU, pooling and the window
// codes need moves inside a quad of lanes only.
//
// What bounds it, at 64 workers x 32 samples, 32 -> 64 channels, 16 x 16 pixels (53.7 GFLOP, six times that in bf16):
// forward 239 us = 1.35 PFLOP/s of bf16 (a register-resident loop reaches 1.87); the data gradient, with 32 output rows per
// wave, reads 9 KB of LDS per 12 matrix instructions and comes to 232.  The fp32 kernels they replace took 433 and 447 us
// (122 TFLOP/s).  Of a workgroup's 64 us 50 are the products, which run at about 80 % of that loop, 4 the first copy of the image
// and the rest the epilogue, which two workgroups of a compute unit tend to reach together: with the four pixels of a window brought into
// one lane per channel (quad_transpose) a maximum is taken once instead of in all four lanes, and rows are stored in pairs of
// pixels (248 and 246 us before; 32 x 32, 16 -> 32 channels on 16 x 16, 3 x 3: 28 -> 26.5 and 38 -> 35).
//
// Up to sixteen output channels (of the forward pass, or the first layer's in the data gradient) would leave half of a 32-row block
// empty: there a wave multiplies 16 x 16 outputs over 32 values, which are the sixteen channels of two taps.  It reads 15 KB of
// LDS per 24 instructions of half the time, which then bounds it.  Data gradient, 32-row blocks / this: 16 x 50, 16 <- 32 channels on
// 14 x 14, 5 x 5: 65 / 50 us; 32 x 32, 16 <- 32 on 16 x 16, 3 x 3: 35 / 31; 32 x 32, 12 <- 24 on 10 x 10, 3 x 3: 19.7 / 18.4;
// a round of 64 x 64, 32 -> 16 on 16 x 16, 5 x 5 (the forward pass): 1075 / 981.  From seventeen rows on half of a block is used at least.
//
// Where a sum is not finite, a workgroup (a wave of first_kernel) multiplies a second time: the small partial products, what is not
// finite of them dropped, then the large ones; in the weight gradient both of them dense, after a sparse first time.  With one infinite weight of
// conv2 in every one of those 64 workers a round takes 2.29 ms, with nothing but NaN 2.07, with an infinite pixel in one sample of
// each worker 2.17 (1.58 with finite values).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "split_bf16.h"

namespace convsplit {

using split_bf16::f32x16;
using split_bf16::planes;
using split_bf16::u32x4;

constexpr int THREADS = 256, WINDOWS = 64;            // of the forward kernel: 4 waves x 2 blocks x 8 windows

struct Shape {
    int Cin, Cout, H, W, KS, B;
};

// Row pitch of the image in LDS (positions): an odd multiple of 4, so that the two rows of eight lanes' windows fall
// into different banks.
__host__ __device__ inline int pitch(const Shape &s)
{
    int p = s.W + s.KS - 1;
    while (p % 8 != 4) ++p;
    return p;
}
__host__ __device__ inline int samples_per_group(const Shape &s)
{
    const int t = s.H * s.W / 4;
    return t >= WINDOWS ? 1 : WINDOWS / t;
}
__host__ __device__ inline int positions(const Shape &s) { return (s.H + s.KS - 1) * pitch(s); }
// MB: 32-row blocks of output channels per workgroup, 0 where sixteen rows are all there are.  A step of the reduction is one tap of
// sixteen channels, with sixteen rows two of them (the last tap meets zeros); a chunk is the steps whose filters are in LDS at a time.
__host__ __device__ constexpr int step_taps(int Cout) { return Cout <= 16 ? 2 : 1; }
inline int forward_blocks(int Cout) { return Cout <= 16 ? 0 : (Cout <= 32 ? 1 : 2); }
constexpr int chunk_steps(int MB) { return MB == 1 ? 4 : 2; }
inline size_t forward_lds(const Shape &s, int MB)
{
    return 16 * ((size_t)6 * samples_per_group(s) * positions(s) + (size_t)2 * chunk_steps(MB) * (MB ? MB : 1) * 192);
}

// Filters in fragment order: [worker][16-channel group][step][32-row block][plane][lane][8 values].
__host__ __device__ inline int group_steps(int Cout, int KK) { return (KK + step_taps(Cout) - 1) / step_taps(Cout); }
__host__ __device__ inline int row_blocks(int Cout) { return Cout <= 32 ? 1 : (Cout + 63) / 64 * 2; }
inline int64_t filter_floats(int Cin, int Cout, int KS) { return (int64_t)((Cin + 15) / 16) * group_steps(Cout, KS * KS) * row_blocks(Cout) * 768; }

// src: filters [C2][C1][KK] of a convolution C1 -> C2, in its forward order (rows = C2, reduction over C1), or in that
// of its data gradient (rows = C1, reduction over C2, taps reversed).  A workgroup brings the filters of 32 rows x 16
// reduction channels into LDS as they lie in memory (runs of 16 KK or 32 KK floats) and writes all their taps.  64
// workers x 32 -> 64 channels, 5 x 5: 15 us; a thread per group of eight that gathers them from memory itself 38.
// grid = (16-channel groups x row blocks of both directions, workers).
__host__ __device__ inline int prepare_blocks(int Cin, int Cout) { return (Cin + 15) / 16 * row_blocks(Cout); }

constexpr int PREPARE_THREADS = 1024;

template <int KK, bool FLIP>
__device__ __forceinline__ void prepare(float *tile /* LDS [16 channels][32 rows][KK] */, const float *__restrict__ s, u32x4 *__restrict__ d,
                                        int C1, int C2, int blk)
{
    static_assert(KK % 2 == 1, "the row length keeps lanes' rows in different banks");
    constexpr int INNER = (FLIP ? 32 : 16) * KK, OUTER = FLIP ? 16 : 32;     // the outer index in memory is C2
    const int mbt = row_blocks(FLIP ? C1 : C2), mb = blk % mbt, g = blk / mbt, tid = threadIdx.x;
    const int i0 = (FLIP ? 32 * mb : 16 * g) * KK, o0 = FLIP ? 16 * g : 32 * mb;
    constexpr int PER = (512 * KK + PREPARE_THREADS - 1) / PREPARE_THREADS;
    static_assert(INNER * OUTER == 512 * KK, "the loops cover the block");
    float f[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {                  // all of a thread's loads in flight
        const int e = tid + PREPARE_THREADS * u, o = e / INNER, i = e % INNER;
        const bool ok = e < 512 * KK && o0 + o < C2 && i0 + i < C1 * KK;
        const float v = s[ok ? (int64_t)(o0 + o) * C1 * KK + i0 + i : 0];
        f[u] = ok ? v : 0.f;
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int e = tid + PREPARE_THREADS * u, o = e / INNER, i = e % INNER, ch = FLIP ? o : i / KK, row = FLIP ? i / KK : o;
        if (e < 512 * KK) tile[(ch * 32 + row) * KK + i % KK] = f[u];
    }
    __syncthreads();
    const int rows = FLIP ? C1 : C2, steps = group_steps(rows, KK);
    const bool two = step_taps(rows) == 2;
    for (int e = tid; e < steps * 64; e += PREPARE_THREADS) {
        const int lane = e % 64, step = e / 64;
        const int tap = two ? 2 * step + lane / 32 : step, ch = two ? lane / 16 % 2 : lane / 32, row = two ? lane % 16 : lane % 32;
        const int t = min(tap, KK - 1);
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float f = tile[((8 * ch + j) * 32 + row) * KK + (FLIP ? KK - 1 - t : t)];
            v[j] = tap < KK ? f : 0.f;
        }
        const planes p = split_bf16::split8_nearest(v);
        u32x4 *at = d + ((int64_t)(g * steps + step) * mbt + mb) * 192 + lane;
        at[0] = p.h;
        at[64] = p.m;
        at[128] = p.l;
    }
}

template <int KK>
__global__ __launch_bounds__(PREPARE_THREADS) void prepare_kernel(const float *__restrict__ src, int64_t src_stride, u32x4 *__restrict__ fwd,
                                                      u32x4 *__restrict__ bwd, int64_t dst_stride, int C1, int C2)
{
    __shared__ float tile[512 * KK];
    const int nf = prepare_blocks(C1, C2), blk = blockIdx.x;
    const float *s = src + blockIdx.y * src_stride;
    if (blk < nf) prepare<KK, false>(tile, s, fwd + blockIdx.y * dst_stride, C1, C2, blk);
    else prepare<KK, true>(tile, s, bwd + blockIdx.y * dst_stride, C1, C2, blk - nf);
}

struct FwdArgs {
    Shape s;
    const float *in;            // [worker][B][Cin][H][W]; EXPAND: the pooled gradients [B][Cin][H/2][W/2] with in_code
    int64_t in_stride;
    const uint8_t *in_code;
    int64_t in_code_stride;
    const u32x4 *filters;       // prepare_kernel
    int64_t filters_stride;
    const float *bias;          // or null
    int64_t bias_stride;
    float *out;                 // [worker][B][Cout][H][W]; POOL: [B][Cout][H/2][W/2] after ReLU and pooling, with code
    int64_t out_stride;
    uint8_t *code;
    int64_t code_stride;
    const float *wgt;           // first_kernel: the filters themselves
    int64_t wgt_stride;
};

template <int CTRL>
__device__ __forceinline__ float quad(float v)        // v of the quad's lanes in the order that CTRL gives
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// v[i] of lane j of a quad <-> v[j] of lane i
__device__ __forceinline__ void quad_transpose(float (&v)[4], int lane)
{
    auto exchange = [](float &x, float &y, bool upper, auto ctrl) {       // (the moves with all lanes, outside of the selects)
        const float px = quad<decltype(ctrl)::value>(x), py = quad<decltype(ctrl)::value>(y);
        x = upper ? py : x;
        y = upper ? y : px;
    };
    const std::integral_constant<int, 0xB1> xor1;
    const std::integral_constant<int, 0x4E> xor2;
    exchange(v[0], v[1], lane & 1, xor1);
    exchange(v[2], v[3], lane & 1, xor1);
    exchange(v[0], v[2], lane & 2, xor2);
    exchange(v[1], v[3], lane & 2, xor2);
}

// 64 x 16 bytes from global memory to LDS; the caller waits for them (see mix_split.h).
__device__ __forceinline__ void load_to_lds(const u32x4 *src, const u32x4 *dst)
{
    const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const u32x4 *)dst);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(m0) : "memory");
}

// grid = (ceil(B / samples_per_group) x ceil(windows of a sample / 64 if there is one sample), workers, row blocks / MB or 1);
// dynamic LDS = forward_lds.
template <int MB, bool POOL, bool EXPAND>
__global__ __launch_bounds__(THREADS, 2) void forward_kernel(FwdArgs a)
{
    extern __shared__ __attribute__((aligned(16))) u32x4 sm[];
    constexpr bool SIXTEEN = MB == 0;                 // rows: matrix instructions of 16 x 16 outputs over two taps
    constexpr int TCH = chunk_steps(MB), RB = SIXTEEN ? 1 : MB, COLS = SIXTEEN ? 16 : 32, NB = 64 / COLS;
    using Acc = std::conditional_t<SIXTEEN, split_bf16::f32x4, f32x16>;
    constexpr int REGS = sizeof(Acc) / 4;
    const int H = a.s.H, W = a.s.W, KS = a.s.KS, KK = KS * KS, HW = H * W, T = HW / 4, WP = pitch(a.s), POS = positions(a.s);
    const int spg = samples_per_group(a.s), xt = spg > 1 ? 1 : (T + WINDOWS - 1) / WINDOWS;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = blockIdx.y, b0 = blockIdx.x / xt * spg, q0 = blockIdx.x % xt * WINDOWS, nb_s = min(spg, a.s.B - b0);
    const int half = spg * POS, plane = 2 * half;     // 16-byte groups of eight channels / of a plane
    u32x4 *img = sm, *wb = sm + 3 * plane;

    const int groups = (a.s.Cin + 15) / 16, mbt = row_blocks(a.s.Cout), gs = group_steps(a.s.Cout, KK), cpg = (gs + TCH - 1) / TCH, chunks = groups * cpg;
    const u32x4 *fl = a.filters + w * a.filters_stride + blockIdx.z * RB * 192 + lane;
    auto fetch = [&](int c) {                          // chunk c of the filters, a quarter of it by each wave
        const int t0 = c % cpg * TCH, n = min(TCH, gs - t0) * RB * 3;
        const int64_t first = (int64_t)(c / cpg * gs + t0) * mbt * 192;
#pragma unroll
        for (int u = 0; u < (TCH * RB * 3 + 3) / 4; ++u) {
            const int i = wave + 4 * u;
            if (i < n) load_to_lds(fl + first + (int64_t)(i / (RB * 3)) * mbt * 192 + i % (RB * 3) * 64, wb + (c & 1) * TCH * RB * 192 + i * 64);
        }
    };
    fetch(0);
    for (int e = tid; e < 3 * plane; e += THREADS) img[e] = u32x4{0u, 0u, 0u, 0u};       // the halo stays zero

    // this lane's pixel in each of the blocks of columns: four lanes per window
    int pos[NB], smp[NB], win[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int q = q0 + COLS / 4 * (NB * wave + nb) + lane % COLS / 4;
        smp[nb] = spg > 1 ? q / T : 0;
        win[nb] = spg > 1 ? q % T : q;
        if (smp[nb] >= nb_s || win[nb] >= T) smp[nb] = -1;                                // beyond the samples: never stored
        const int wy = win[nb] / (W / 2), wx = win[nb] % (W / 2);
        pos[nb] = (smp[nb] < 0 ? 0 : smp[nb] * POS + (2 * wy + (lane >> 1 & 1)) * WP + 2 * wx + (lane & 1)) + lane / COLS % 2 * half;
    }
    Acc acc[RB][NB];
    auto zero = [&] {
#pragma unroll
        for (int mb = 0; mb < RB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < REGS; ++v) acc[mb][nb][v] = 0.f;
    };
    zero();

    // the partial products of the whole reduction, all of them or those of one kind; chunk 0 is on its way
    auto products = [&](auto small, auto large) {
        for (int c = 0; c < chunks; ++c) {
            if (c % cpg == 0) {                            // the next 16 channels of the image
                __syncthreads();
                const int pad = KS / 2, g = c / cpg;
                if (EXPAND) {
                    // a window of eight channels: split once, then masked by the codes into its four positions
                    for (int e = tid; e < 2 * spg * T; e += THREADS) {
                        const int hh = e / (spg * T), r = e % (spg * T), s = r / T, q = r % T, wy = q / (W / 2), wx = q % (W / 2);
                        float v[8];
                        int cd[8];
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const int ch = 16 * g + 8 * hh + j;
                            const bool ok = s < nb_s && ch < a.s.Cin;
                            const int64_t at = ok ? ((int64_t)(b0 + s) * a.s.Cin + ch) * T + q : 0;
                            const float f = a.in[w * a.in_stride + at];
                            const int code = a.in_code[w * a.in_code_stride + at];
                            v[j] = ok ? f : 0.f;
                            cd[j] = ok ? code : 4;
                        }
                        const planes p = split_bf16::split8_nearest(v);
                        u32x4 *d = img + hh * half + s * POS + (2 * wy + pad) * WP + 2 * wx + pad;
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            u32x4 mask;
#pragma unroll
                            for (int j = 0; j < 4; ++j) mask[j] = (cd[2 * j] == k ? 0xffffu : 0u) | (cd[2 * j + 1] == k ? 0xffff0000u : 0u);
                            u32x4 *dk = d + (k >> 1) * WP + (k & 1);
                            dk[0] = p.h & mask;
                            dk[plane] = p.m & mask;
                            dk[2 * plane] = p.l & mask;
                        }
                    }
                } else {
                    for (int e = tid; e < 2 * spg * HW; e += THREADS) {
                        const int hh = e / (spg * HW), r = e % (spg * HW), s = r / HW, px = r % HW, y = px / W, x = px % W;
                        float v[8];
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const int ch = 16 * g + 8 * hh + j;
                            const bool ok = s < nb_s && ch < a.s.Cin;
                            const float f = a.in[w * a.in_stride + (ok ? ((int64_t)(b0 + s) * a.s.Cin + ch) * HW + px : 0)];
                            v[j] = ok ? f : 0.f;
                        }
                        const planes p = split_bf16::split8_nearest(v);
                        u32x4 *d = img + hh * half + s * POS + (y + pad) * WP + x + pad;
                        d[0] = p.h;
                        d[plane] = p.m;
                        d[2 * plane] = p.l;
                    }
                }
            }
            // chunk c has landed and everybody is done with chunk c - 1, whose place chunk c + 1 takes
            __builtin_amdgcn_s_waitcnt(0);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (c + 1 < chunks) fetch(c + 1);
            const int t0 = c % cpg * TCH, nt = min(TCH, gs - t0);
            const u32x4 *wc = wb + (c & 1) * TCH * RB * 192 + lane;
#pragma unroll
            for (int t = 0; t < TCH; ++t) {
                if (t < nt) {
                    auto offset = [&](int tap) { return tap / KS * WP + tap % KS; };
                    int off = offset(step_taps(SIXTEEN ? 16 : 32) * (t0 + t));
                    bool none = false;                 // behind the last tap: the first position, which is halo
                    if (SIXTEEN) {
                        const int second = 2 * (t0 + t) + 1;
                        none = lane >= 32 && second == KK;
                        off = lane >= 32 ? offset(second) : off;
                    }
                    planes fa[RB], fb[NB];
#pragma unroll
                    for (int mb = 0; mb < RB; ++mb) {
                        const u32x4 *p = wc + (t * RB + mb) * 192;
                        fa[mb] = planes{p[0], p[64], p[128]};
                    }
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const u32x4 *p = img + (none ? 0 : pos[nb] + off);
                        fb[nb] = planes{p[0], p[plane], p[2 * plane]};
                    }
                    split_bf16::mma_block<decltype(small)::value, decltype(large)::value>(fa, fb, acc);
                }
            }
        }
    };
    products(std::true_type{}, std::true_type{});
    // ---- some sum of the workgroup is not finite: again, in the order that tells infinities from NaN (see split_bf16.h)
    bool bad = false;
#pragma unroll
    for (int mb = 0; mb < RB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) bad |= smp[nb] >= 0 && split_bf16::any_not_finite(acc[mb][nb]);
    int *votes = (int *)(wb + (chunks & 1) * TCH * RB * 192);     // in the half of the filters that nobody reads any more
    const int vote = __any(bad);
    if (lane == 0) votes[wave] = vote;
    __syncthreads();
    if (votes[0] | votes[1] | votes[2] | votes[3]) {
        __syncthreads();                               // the votes have been read
        fetch(0);
        zero();
        products(std::true_type{}, std::false_type{});
#pragma unroll
        for (int mb = 0; mb < RB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) split_bf16::drop_not_finite(acc[mb][nb]);
        __syncthreads();                               // the filters have been used
        fetch(0);
        products(std::false_type{}, std::true_type{});
    }

    // ---- epilogue.  Register v of a lane: output channel 32 mb + 8 (v / 4) + 4 (lane / 32) + v % 4 (SIXTEEN: 4 (lane / 16) + v), the lane's pixel.
    const int m0 = 32 * MB * blockIdx.z, PP = T;
    float *ob = a.out + w * a.out_stride;
#pragma unroll
    for (int mb = 0; mb < RB; ++mb)
#pragma unroll
        for (int k = 0; k < REGS / 4; ++k) {
            const int c0 = m0 + 32 * mb + 8 * k + 4 * (lane / COLS);
            const int co = c0 + (lane & 3);
            const float bv = a.bias && co < a.s.Cout ? a.bias[w * a.bias_stride + co] : 0.f;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                // a pixel of four channels in every lane of a quad -> the four pixels of channel `co` in each
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = acc[mb][nb][4 * k + i];
                quad_transpose(v, lane);
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] += bv;
                const int64_t row = (int64_t)(b0 + smp[nb]) * a.s.Cout + co;
                if (POOL) {
                    const float mx = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
                    int arg = v[2] == mx ? 2 : 3;
                    arg = v[1] == mx ? 1 : arg;
                    arg = v[0] == mx ? 0 : arg;
                    arg = mx > 0.f ? arg : 4;
                    if (smp[nb] >= 0 && co < a.s.Cout) {
                        ob[row * PP + win[nb]] = fmaxf(mx, 0.f);
                        a.code[w * a.code_stride + row * PP + win[nb]] = (uint8_t)arg;
                    }
                } else if (smp[nb] >= 0 && co < a.s.Cout) {
                    typedef float f32x2_any __attribute__((ext_vector_type(2), aligned(4)));
                    float *o = ob + row * HW + 2 * (win[nb] / (W / 2)) * W + 2 * (win[nb] % (W / 2));
                    *(f32x2_any *)o = f32x2_any{v[0], v[1]};
                    *(f32x2_any *)(o + W) = f32x2_any{v[2], v[3]};
                }
            }
        }
}

// ---- forward pass, ReLU and pooling of a layer with few input channels (the network's first).
//
// With one or three channels the reduction of forward_kernel would be mostly padding.  Here it runs over taps (c, kh, kw) in their order in
// memory, eight to a lane and sixteen to a step: the lower half of a wavefront takes the first half of the filter rows (c, kh), the upper
// half the other, so that the pattern of rows and taps in a lane's eight values is the same for all lanes, repeats after
// eight rows, and is known to the compiler.  A lane's values for the output pixels 8 m .. 8 m + 7 come from the sixteen pixels from 8 m on of two
// to four rows, read as aligned 16-byte groups: two taps side by side are one register or a shift of two, the last tap of a row and the
// first of the next one permutation.  A wave takes 32 positions (y, m) = 256 output pixels at a time, even and odd y in
// neighbouring lanes for the pooling; the filters stay in LDS, split, over all samples of the workgroup.
//
// The matrix instructions bound it (75 of 80 values of a 3-channel 5 x 5 filter's reduction are used, 27 of 32 with 3 x 3).  Then the
// copies of the images and the epilogue.  us, before with the taps of one row in a lane's eight values (5 or 3 of 8 used) / now:
// 64 workers x 32 samples, 3 -> 32 channels on 32 x 32 pixels, 5 x 5: 101 / 87; 32 x 32, 3 -> 16 on 32 x 32, 3 x 3: 38 / 29; 16 x 50, 1 -> 16
// on 28 x 28, 5 x 5: 29 / 26.  A lane finishing one channel only in the epilogue (half the operations, its row of the other
// channel handed over by selects) was slower: 98, 35, 32.
struct FirstPlan {
    int spg, iters;             // samples in LDS at a time, and how often
    size_t lds;
};
__host__ __device__ inline int first_groups(const Shape &s) { return (s.W + 7) / 8; }            // m
__host__ __device__ inline int first_rows(const Shape &s) { return (s.Cin * s.KS + 1) / 2; }     // filter rows of a half
__host__ __device__ inline int first_steps(const Shape &s) { return (first_rows(s) * s.KS + 7) / 8; }
// 16-byte groups of one plane of one sample's image: rows of 8 m + 8 values
__host__ __device__ inline int first_image(const Shape &s) { return s.Cin * (s.H + s.KS - 1) * (first_groups(s) + 1); }
inline bool first_plan(const Shape &s, int workers, FirstPlan &p)
{
    const int per = s.H * first_groups(s);              // positions of a sample; four waves x 32 of them
    p.spg = per >= 128 ? 1 : 128 / per;
    if (p.spg > s.B) p.spg = s.B;
    p.lds = 48 * ((size_t)p.spg * first_image(s) + (size_t)first_steps(s) * 64);
    if (p.lds > 160 * 1024) {
        p.spg = 1;
        p.lds = 48 * ((size_t)first_image(s) + (size_t)first_steps(s) * 64);
    }
    const int64_t groups = (int64_t)((s.B + p.spg - 1) / p.spg) * workers;
    // Several turns, for which the filters are split once, where the chip is full all the same.  One / two / four turns, us:
    // 8 192 groups (128 workers x 64 samples, 3 x 3) 252, 251, 244; 4 000 (100 x 40, 5 x 5) 205, 197, 197; 2 048 108, 105, 102;
    // 1 024 58, 56, 72.  Several samples to a group end less evenly (100 x 100 samples of 16 x 16, 2 500 groups: 106, 115, 146).
    p.iters = groups >= 4096 ? 4 : (groups >= 2048 ? 2 : 1);
    return p.lds <= 160 * 1024;
}

// grid = (ceil(B / (spg iters)), workers, 32-row blocks of the output channels); dynamic LDS = plan.lds.  Of FwdArgs: s, in, wgt
// (not split), bias, out, code.
template <int KS>
__global__ __launch_bounds__(THREADS, 2) void first_kernel(FwdArgs a, FirstPlan plan)
{
    extern __shared__ __attribute__((aligned(16))) u32x4 sm[];
    const int H = a.s.H, W = a.s.W, Cin = a.s.Cin, Cout = a.s.Cout, pad = KS / 2, HP = H + KS - 1, M = first_groups(a.s), IPG = M + 1;
    const int spg = plan.spg, image = first_image(a.s), iplane = spg * image, steps = first_steps(a.s), wplane = steps * 64;
    const int pairs = Cin * KS, rows = first_rows(a.s), PP = H * W / 4, m0 = 32 * blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = blockIdx.y;
    u32x4 *img = sm, *wl = sm + 3 * iplane;
    const float *inw = a.in + w * a.in_stride, *wg = a.wgt + w * a.wgt_stride;

    for (int e = tid; e < wplane; e += THREADS) {        // filters: lane (channel, half) of step e / 64 holds taps 8 step .. of its half
        const int ln = e % 64, t0 = e / 64 * 8, half = ln / 32, co = m0 + ln % 32;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int t = t0 + j;
            const bool ok = t < rows * KS && half * rows + t / KS < pairs && co < Cout;
            const float f = wg[ok ? (co * pairs + half * rows) * KS + t : 0];
            v[j] = ok ? f : 0.f;
        }
        const planes p = split_bf16::split8_nearest(v);
        wl[e] = p.h;
        wl[e + wplane] = p.m;
        wl[e + 2 * wplane] = p.l;
    }
    for (int e = tid; e < 3 * iplane; e += THREADS) img[e] = u32x4{0u, 0u, 0u, 0u};      // the halo stays zero

    for (int it = 0; it < plan.iters; ++it) {
        const int b0 = (blockIdx.x * plan.iters + it) * spg, ns = min(spg, a.s.B - b0);
        if (ns <= 0) break;                              // uniform
        __syncthreads();                                 // the images before have been used
        for (int e = tid; e < ns * Cin * H * IPG; e += THREADS) {
            const int g = e % IPG, y = e / IPG % H, sc = e / IPG / H;                     // sc = sample Cin + channel
            const float *src = inw + (((int64_t)b0 * Cin + sc) * H + y) * W;
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int x = 8 * g + j - pad;
                const float f = src[min(max(x, 0), W - 1)];
                v[j] = (unsigned)x < (unsigned)W ? f : 0.f;
            }
            const planes p = split_bf16::split8_nearest(v);
            u32x4 *d = img + (sc * HP + y + pad) * IPG + g;
            d[0] = p.h;
            d[iplane] = p.m;
            d[2 * iplane] = p.l;
        }
        __syncthreads();
        const int total = ns * H * M;
        for (int blk = wave; blk * 32 < total; blk += 4) {
            // position n of the block: y parity innermost, then m, then pairs of rows, then samples
            const int n = 32 * blk + (lane & 31), nn = n < total ? n : 0, q = nn >> 1;
            const int m = q % M, yh = q / M % (H / 2), smp = q / M / (H / 2), dy = nn & 1;
            const u32x4 *base = img + smp * image + (2 * yh + dy) * IPG + m;
            f32x16 acc[8];
            auto zero = [&] {
#pragma unroll
                for (int x = 0; x < 8; ++x)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[x][v] = 0.f;
            };
            zero();
            // the partial products of the whole reduction, all of them or those of one kind.  MASK: nothing but the filter's taps
            // is multiplied (otherwise zero weights take up the rest of a step, which is the same for finite values)
            auto products = [&](auto small, auto large, auto mask) {
                constexpr bool SMALL = decltype(small)::value, LARGE = decltype(large)::value, MASK = decltype(mask)::value;
#pragma unroll 1
                for (int s0 = 0; s0 < steps; s0 += KS) {            // eight rows of either half
#pragma unroll
                    for (int g = 0; g < KS; ++g) {
                        if (s0 + g >= steps) break;
                        const int r0 = 8 * g / KS, NR = (8 * g + 7) / KS - r0 + 1;        // rows of the step; constants once unrolled
                        const u32x4 *src[4];
#pragma unroll
                        for (int r = 0; r < NR; ++r) {
                            const int row = s0 / KS * 8 + r0 + r, p0 = min(row, pairs - 1), p1 = min(row + rows, pairs - 1);     // (beyond: zero weights)
                            src[r] = base + (lane < 32 ? (p0 / KS) * HP + p0 % KS : (p1 / KS) * HP + p1 % KS) * IPG;
                        }
                        const u32x4 *ws = wl + (s0 + g) * 64 + lane;
                        const u32x4 fh = ws[0], fm = ws[wplane], fl = ws[2 * wplane];
                        uint32_t d[4][8];
                        auto read = [&](int plane) {
#pragma unroll
                            for (int r = 0; r < NR; ++r) {
                                const u32x4 lo = src[r][plane * iplane], hi = src[r][plane * iplane + 1];
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    d[r][i] = lo[i];
                                    d[r][4 + i] = hi[i];
                                }
                            }
                        };
                        auto shifted = [&](int x) {      // the eight taps' values for output pixel 8 m + x
                            u32x4 f;
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int t = 8 * g + 2 * i, ra = t / KS - r0, rb = (t + 1) / KS - r0, pa = x + t % KS, pb = x + (t + 1) % KS;
                                if (ra == rb)
                                    f[i] = pa % 2 == 0 ? d[ra][pa / 2] : __builtin_amdgcn_alignbit(d[ra][pa / 2 + 1], d[ra][pa / 2], 16);
                                else
                                    f[i] = __builtin_amdgcn_perm(d[rb][pb / 2], d[ra][pa / 2], (pb % 2 ? 0x07060000u : 0x05040000u) | (pa % 2 ? 0x0302u : 0x0100u));
                                if (MASK) {
                                    const int tap = s0 * 8 + t, left = min(rows, lane < 32 ? rows : pairs - rows) * KS - tap;     // taps of the half from this one on
                                    f[i] = left >= 2 ? f[i] : (left == 1 ? f[i] & 0xffffu : 0u);
                                }
                            }
                            return split_bf16::frag(f);
                        };
                        auto mma = [&](const u32x4 &f, split_bf16::bf16x8 b, int x) {
                            acc[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(split_bf16::frag(f), b, acc[x], 0, 0, 0);
                        };
                        if (SMALL) {
                            read(2);
#pragma unroll
                            for (int x = 0; x < 8; ++x) mma(fh, shifted(x), x);
                            read(1);
#pragma unroll
                            for (int x = 0; x < 8; ++x) {
                                const auto b = shifted(x);
                                mma(fm, b, x);
                                mma(fh, b, x);
                            }
                        }
                        read(0);
#pragma unroll
                        for (int x = 0; x < 8; ++x) {
                            const auto b = shifted(x);
                            if (SMALL) {
                                mma(fl, b, x);
                                mma(fm, b, x);
                            }
                            if (LARGE) mma(fh, b, x);
                        }
                        __builtin_amdgcn_sched_barrier(0);       // (with the reads of several steps ahead the registers run out)
                    }
                }
            };
            products(std::true_type{}, std::true_type{}, std::false_type{});
            bool bad = false;
#pragma unroll
            for (int x = 0; x < 8; ++x) bad |= n < total && split_bf16::any_not_finite(acc[x]);
            if (__any(bad)) {      // again, in the order that tells infinities from NaN (see split_bf16.h)
                zero();
                products(std::true_type{}, std::false_type{}, std::true_type{});
#pragma unroll
                for (int x = 0; x < 8; ++x) split_bf16::drop_not_finite(acc[x]);
                products(std::false_type{}, std::true_type{}, std::true_type{});
            }
            // ---- the two lanes of a position pair hold the same four windows; each stores every other output channel
            const int64_t wbase = yh * (W / 2) + 4 * m;
            const int left = W / 2 - 4 * m;              // windows that exist
#pragma unroll
            for (int v2 = 0; v2 < 16; v2 += 2) {
                const int co = m0 + 8 * (v2 / 4) + 4 * (lane >> 5) + v2 % 4 + dy;
                float mx[4];
                uint32_t code = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float r[2];
                    uint32_t cd[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int cv = co - dy + i;      // the bias of the register's channel
                        const float bias = a.bias[w * a.bias_stride + min(cv, Cout - 1)];
                        const float x0 = acc[2 * j][v2 + i] + bias, x1 = acc[2 * j + 1][v2 + i] + bias;
                        const float y0 = quad<0xB1>(x0), y1 = quad<0xB1>(x1);             // the other row
                        const float t0 = dy ? y0 : x0, t1 = dy ? y1 : x1, u0 = dy ? x0 : y0, u1 = dy ? x1 : y1;
                        const float top = fmaxf(fmaxf(t0, t1), fmaxf(u0, u1));
                        uint32_t k = u0 == top ? 2 : 3;
                        k = t1 == top ? 1 : k;
                        k = t0 == top ? 0 : k;
                        cd[i] = top > 0.f ? k : 4;
                        r[i] = fmaxf(top, 0.f);
                    }
                    mx[j] = dy ? r[1] : r[0];
                    code |= (dy ? cd[1] : cd[0]) << (8 * j);
                }
                if (n < total && co < Cout) {
                    const int64_t at = ((int64_t)(b0 + smp) * Cout + co) * PP + wbase;
                    float *o = a.out + w * a.out_stride + at;
                    uint8_t *c = a.code + w * a.code_stride + at;
                    if (left >= 4) {
                        typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
                        *(f32x4_any *)o = f32x4_any{mx[0], mx[1], mx[2], mx[3]};
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (j < left) {
                            if (left < 4) o[j] = mx[j];
                            c[j] = (uint8_t)(code >> (8 * j));
                        }
                }
            }
        }
    }
}

// ---- weight gradient: dW[co][c][kh][kw] = sum over samples and pixels of dz[co][y][x] in[c][y + kh - pad][x + kw - pad],
// with dz given as pooled gradients and window codes.
//
// The reduction runs over the pixels of a pair of rows, 16 of each at a time (rows padded with zeros to a multiple of 16).  The deltas are
// pooled, so that of two neighbouring pixels at most one is not zero: v_smfmac_f32_32x32x32_bf16, whose first operand has two values
// for every four terms and four bits that say which, multiplies both rows' pixels in the time of one's.  Of the image a lane's
// fragment is sixteen consecutive pixels, which would start at any one, depending on kw, and LDS
// reads want aligned ones: the 32 columns of a fragment are therefore pairs (c, kh), a lane reads the twenty pixels from x
// on once, and the KS fragments of its kw are shifts of those inside the registers (none for an even kw, eight
// v_alignbit for an odd one).  A wave owns 32 output channels x 32 pairs x all kw; image and deltas are split when they
// are copied into LDS.  Where there are few such blocks, several waves share one, take turns with the steps
// and add their sums through LDS in wave order.  Every workgroup writes a partial result:
// part[worker][split][co][c][kh][kw], summed in split order by a separate pass.
//
// 64 workers x 32 samples, 32 -> 64 channels, 16 x 16 pixels: 170 us, with a dense instruction of 16 pixels 246, an fp32 kernel 427; 145 of
// them without the copies into LDS, 80 the copies alone.  Ten blocks on the four SIMDs of a compute unit are three rounds of 2.5, and
// LDS holds one workgroup.  16 workers x 50 samples, 16 -> 32 channels on 14 x 14: 34 us, 45 (implicit fp32 GEMM: 231).  Error of
// dW against 64 bits, dense / sparse: 2.34e-7 / 2.31e-7 for the first, 1.52e-7 / 1.46e-7 for the second, 1.62e-7 / 1.43e-7 for 16 -> 64 on 12 x 12.
//
// What a sparse instruction leaves out is not multiplied, so where a pixel, and not only where a sum, is not finite the workgroup goes
// through its products again with every delta written out (two dense steps of 16 pixels; LDS is laid out for these).
struct WgradPlan {
    int mb, nb, units;          // 32-row and 32-column blocks
    int kw, waves, groups;      // waves that share a block, waves of a workgroup, workgroups along the blocks
    int rows, sb;               // image rows per delta tile, samples per workgroup
    int splits;                 // partial results per worker
    bool paired;                // two workgroups have to fit on a compute unit that would not with 5 x 5 filters' registers
    size_t lds;
};
constexpr int WGRAD_MAX_WAVES = 12;

__host__ __device__ inline int row_elems(const Shape &s) { return (s.W + 15) / 16 * 16; }        // of a delta row
__host__ __device__ inline int image_pitch(const Shape &s) { return row_elems(s) + 8; }          // of an image row
inline size_t wgrad_image_lds(const Shape &s) { return (size_t)6 * s.Cin * (s.H + s.KS - 1) * image_pitch(s); }
inline size_t wgrad_delta_lds(const Shape &s, int mb, int rows) { return (size_t)6 * 32 * mb * (rows * row_elems(s) + 8); }

inline bool wgrad_plan(const Shape &s, int workers, WgradPlan &p)
{
    p.mb = (s.Cout + 31) / 32;
    p.nb = (s.Cin * s.KS + 31) / 32;
    p.units = p.mb * p.nb;
    // Eight wavefronts for few blocks: more of them hide the copies and splits, which a workgroup does between barriers, but
    // their sums meet in LDS.  No number is the best everywhere (four / eight / twelve waves, us): 64 workers x 64 samples, 3 x 3, 32 -> 32 channels
    // on 8 x 8 72, 60, 69, 16 -> 16 on 16 x 16 73, 69, 91; 50 x 20, 3 x 3, 32 -> 24 on 14 x 14 49, 37, 34; 40 x 40, 5 x 5, 16 -> 32 on 14 x 14 62,
    // 56, 68.
    p.kw = p.units >= 5 ? 1 : 8 / p.units;
    p.groups = (p.units + WGRAD_MAX_WAVES - 1) / WGRAD_MAX_WAVES;
    p.waves = (p.units + p.groups - 1) / p.groups * p.kw;
    // two workgroups per compute unit if a tile of at least four rows leaves room for that
    const size_t img = wgrad_image_lds(s), most = 160 * 1024;
    int per_cu = 2;
    p.rows = 0;
    for (; per_cu >= 1 && p.rows == 0; --per_cu)
        for (int r = s.H; r >= (per_cu == 2 ? 4 : 2); r -= 2)
            if (img + wgrad_delta_lds(s, p.mb, r) <= most / per_cu) {
                p.rows = r;
                break;
            }
    ++per_cu;
    if (p.rows == 0) return false;
    // even tiles: as many as the rows found make necessary
    const int tiles = (s.H + p.rows - 1) / p.rows;
    p.rows = ((s.H + tiles - 1) / tiles + 1) / 2 * 2;
    p.lds = img + wgrad_delta_lds(s, p.mb, p.rows);
    const size_t sums = p.kw > 1 ? sizeof(float) * 64 * 16 * s.KS * (p.waves / p.kw) : 0;
    if (p.lds < sums) p.lds = sums;
    // enough workgroups for the chip, and no more partial results than that needs: samples are given out by the ceiling, so that one turn
    // holds all workgroups (by the floor, 16 x 50, 16 -> 32 channels on 14 x 14 46.0 us and 14.9 for the sums, 36.8 and 12.1 now; 50 x 20,
    // 32 -> 24 on 14 x 14, 3 x 3: the round 242, 225).  A workgroup of up to eight samples: with four, 64 x 32, 5 x 5, 32 -> 64 on
    // 16 x 16 takes 193 us and 43 for the sums (181 and 38), 64 x 64, 3 x 3, 32 -> 32 on 8 x 8 78 (60); with sixteen the sums of a workgroup are
    // twice as long, and only some sizes are faster (64 x 64, 5 x 5, 32 -> 16 on 16 x 16 247 against 256, the others the same)
    p.sb = (int)(((int64_t)s.B * workers * p.groups + 256 * per_cu - 1) / (256 * per_cu));
    p.sb = p.sb < 1 ? 1 : (p.sb > 8 ? 8 : p.sb);
    p.splits = (s.B + p.sb - 1) / p.sb;
    // The 5 x 5 kernel takes 161 registers, three wavefronts to a SIMD: of two workgroups of five to eight the second finds no place.
    // Limited to 128 (44 bytes per lane go to scratch) both run: 16 x 50, 16 -> 32 on 14 x 14 44.0 -> 35.5 us, 20 x 13, 32 -> 32 on 10 x 10
    // 35.6 -> 26.2, 64 x 64, 8 -> 32 on 10 x 10 71.2 -> 53.2, 32 x 32, 16 -> 64 on 12 x 12 59.8 -> 51.2.  Where one workgroup is all that a compute
    // unit gets, the limit changes little: 64 x 32, 32 -> 64 on 16 x 16 179 and 177 (the round 1556 either way), 16 x 16, 8 -> 16 on 12 x 12 13.7
    // and 14.2.  (Of nine to twelve wavefronts the second workgroup finds no place either way: 16 x 32, 20 -> 96 on 8 x 8 48.8 us with it and
    // without, 16 x 64, 32 -> 64 on 6 x 6 56.9 and 57.5.  Their samples given out as for one workgroup were faster with the dense instruction, 48.6
    // against 57.3 and 62.7 against 71.5, but the sums of a workgroup twice as long and up to 15 % less exact.)
    p.paired = per_cu == 2 && p.waves > 4 && (int64_t)p.splits * workers * p.groups > 256;
    return true;
}

struct WgradArgs {
    Shape s;
    WgradPlan p;
    const float *in;            // [worker][B][Cin][H][W]
    int64_t in_stride;
    const float *dp;            // pooled gradients [worker][B][Cout][H/2][W/2], with code
    int64_t dp_stride;
    const uint8_t *code;
    int64_t code_stride;
    float *part;
    int64_t part_stride;
};

// grid = (ceil(B / sb), workers, groups), block = 64 waves; dynamic LDS = plan.lds.
template <int KS, int PER_SIMD>
__global__ __launch_bounds__(64 * WGRAD_MAX_WAVES, PER_SIMD) void wgrad_kernel(WgradArgs a)
{
    extern __shared__ __attribute__((aligned(16))) u32x4 sm[];
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const int H = a.s.H, W = a.s.W, Cin = a.s.Cin, Cout = a.s.Cout, pad = KS / 2, HP = H + KS - 1, TAPS = Cin * KS * KS;
    const int RE = row_elems(a.s), segs = RE / 16, IP = image_pitch(a.s), DP = a.p.rows * RE + 8;    // elements; all multiples of 8
    const int iplane = Cin * HP * IP / 8, dplane = 32 * a.p.mb * DP / 8;                             // 16-byte groups
    u32x4 *img = sm, *dz = sm + 3 * iplane;
    const int tid = threadIdx.x, lane = tid & 63, threads = 64 * a.p.waves;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int upg = a.p.waves / a.p.kw, unit = blockIdx.z * upg + wave % upg, kwave = wave / upg;
    const bool idle = unit >= a.p.units;               // uniform: a wave of the last group without a block
    const int mb = unit % a.p.mb, nb = unit / a.p.mb;
    const int w = blockIdx.y, b0 = blockIdx.x * a.p.sb, b1 = min(a.s.B, b0 + a.p.sb);

    const float *inw = a.in + w * a.in_stride, *dpw = a.dp + w * a.dp_stride;
    const uint8_t *cdw = a.code + w * a.code_stride;
    for (int e = tid; e < 3 * (iplane + dplane); e += threads) sm[e] = u32x4{0u, 0u, 0u, 0u};        // halo and padding stay zero

    const int n = 32 * nb + (lane & 31), nc = n < Cin * KS ? n : 0;                                  // pair (c, kh) of the lane
    const int boff = (((nc / KS) * HP + nc % KS) * IP + 8 * (lane >> 5)) / 8;
    const int aoff = ((32 * mb + (lane & 31)) * DP + 8 * (lane >> 5)) / 8;

    f32x16 acc[KS];
    auto zero = [&] {
#pragma unroll
        for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[k][v] = 0.f;
    };
    zero();

    // The image of a sample, split, into LDS; whether this thread has seen a pixel that is not finite.
    auto copy_image = [&](int b) {
        const int per = IP / 8;
        float t = 0.f;
        for (int e = tid; e < Cin * H * per; e += threads) {
            const int m = e % per, y = e / per % H, c = e / per / H;
            const float *src = inw + (((int64_t)b * Cin + c) * H + y) * W;
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int x = 8 * m + j - pad;
                const float f = src[min(max(x, 0), W - 1)];
                v[j] = (unsigned)x < (unsigned)W ? f : 0.f;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) t = fmaf(v[j], 0.f, t);
            const planes p = split_bf16::split8_nearest(v);
            u32x4 *d = img + (c * HP + y + pad) * per + m;
            d[0] = p.h;
            d[iplane] = p.m;
            d[2 * iplane] = p.l;
        }
        return t != t;
    };
    // the partial products of one kind of the whole reduction, every delta written out.  Pixels that meet only the padding of the delta
    // rows are left out
    auto products = [&](auto small, auto large) {
        constexpr bool SMALL = decltype(small)::value, LARGE = decltype(large)::value;
        for (int b = b0; b < b1; ++b)
            for (int r0 = 0; r0 < H; r0 += a.p.rows) {
                const int rows = min(a.p.rows, H - r0);
                __syncthreads();                           // the previous tile has been used
                if (r0 == 0) copy_image(b);
                const int per = RE / 8;
                for (int e = tid; e < Cout * (rows / 2) * per; e += threads) {       // four windows: eight pixels of two rows
                    const int m = e % per, yh = e / per % (rows / 2), co = e / per / (rows / 2);
                    const int64_t o = ((int64_t)b * Cout + co) * (H * W / 4) + (r0 / 2 + yh) * (W >> 1);
                    float g[8];                                  // (each window's value twice)
                    int cd[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int xw = 4 * m + j;
                        const bool ok = xw < W / 2;
                        g[2 * j] = g[2 * j + 1] = dpw[o + (ok ? xw : 0)];
                        const int code = cdw[o + (ok ? xw : 0)];
                        cd[j] = ok ? code : 4;
                    }
                    const planes p = split_bf16::split8_nearest(g);      // both halves of a word: the window's value
                    u32x4 *d = dz + (co * DP + 2 * yh * RE) / 8 + m;
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        u32x4 mask;
#pragma unroll
                        for (int j = 0; j < 4; ++j) mask[j] = cd[j] == 2 * r ? 0xffffu : (cd[j] == 2 * r + 1 ? 0xffff0000u : 0u);
                        u32x4 *dr = d + r * (RE / 8);
                        dr[0] = p.h & mask;
                        dr[dplane] = p.m & mask;
                        dr[2 * dplane] = p.l & mask;
                    }
                }
                __syncthreads();
                if (idle) continue;
                const int steps = rows * segs;
                for (int st = kwave; st < steps; st += a.p.kw) {
                    const int yr = st / segs, x8 = 2 * (st % segs);
                    const u32x4 *ap = dz + aoff + yr * (RE / 8) + x8;
                    const u32x4 *bp = img + boff + (r0 + yr) * (IP / 8) + x8;
                    planes fa;
                    fa.h = ap[0];
                    fa.m = ap[dplane];
                    fa.l = ap[2 * dplane];
                    // fragment kw of one plane of the image: elements kw .. kw + 7 of the twelve read
                    u32x4 fb[KS];
                    auto read = [&](int plane) {
                        const u32x4 q = bp[plane * iplane];
                        const u32x2 r = *(const u32x2 *)&bp[plane * iplane + 1];
                        const uint32_t d[6] = {q[0], q[1], q[2], q[3], r[0], r[1]};
#pragma unroll
                        for (int k = 0; k < KS; ++k)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                fb[k][i] = k % 2 == 0 ? d[k / 2 + i] : __builtin_amdgcn_alignbit(d[k / 2 + i + 1], d[k / 2 + i], 16);
                                fb[k][i] = 8 * x8 + 8 * (lane >> 5) + 2 * i < W ? fb[k][i] : 0u;
                            }
                    };
                    auto step = [&](const u32x4 &x) {
#pragma unroll
                        for (int k = 0; k < KS; ++k)
                            acc[k] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(split_bf16::frag(x), split_bf16::frag(fb[k]), acc[k], 0, 0, 0);
                    };
                    if (SMALL) {
                        read(2);
                        step(fa.h);
                        read(1);
                        step(fa.m);
                        step(fa.h);
                    }
                    read(0);
                    if (SMALL) {
                        step(fa.l);
                        step(fa.m);
                    }
                    if (LARGE) step(fa.h);
                }
            }
    };
    // The deltas are pooled: of the two pixels of a window in an image row at most one is not zero.  So the first time through a sparse
    // instruction multiplies 32 pixels, sixteen of a pair of rows, in the time of sixteen.  LDS holds of four windows, for each plane, the values that lie
    // in the upper row and those in the lower one (zero where the other row has it), and for all planes which pixel of the window
    // they stand for: [plane][channel][row pair][four windows][8 values], [channel][row pair][four windows] of 16 bits.
    const int per = RE / 8, dgroups = a.p.rows / 2 * per + 1, splane = 32 * a.p.mb * dgroups;
    uint16_t *places = (uint16_t *)(dz + 3 * splane);
    const int half = lane >> 5;
    const int arow = (32 * mb + (lane & 31)) * dgroups + half, brow = (((nc / KS) * HP + nc % KS + half) * IP) / 8;
    bool bad = false;                                  // a pixel is not finite (those that meet no delta are not multiplied)
    for (int b = b0; b < b1; ++b)
        for (int r0 = 0; r0 < H; r0 += a.p.rows) {
            const int rows = min(a.p.rows, H - r0);
            __syncthreads();                           // the previous tile has been used
            if (r0 == 0) bad |= copy_image(b);
            for (int e = tid; e < Cout * (rows / 2) * per; e += threads) {
                const int m = e % per, yh = e / per % (rows / 2), co = e / per / (rows / 2);
                const int64_t o = ((int64_t)b * Cout + co) * (H * W / 4) + (r0 / 2 + yh) * (W >> 1);
                float g[4];
                int cd[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int xw = 4 * m + j;
                    const bool ok = xw < W / 2;
                    g[j] = dpw[o + (ok ? xw : 0)];
                    const int code = cdw[o + (ok ? xw : 0)];
                    cd[j] = ok ? code : 4;
                }
                uint32_t h[2], mi[2], lo[2], up[2], down[2], place = 0;
                split_bf16::split_nearest<4>(g, h, mi, lo);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int c0 = cd[2 * q], c1 = cd[2 * q + 1];
                    up[q] = (c0 < 2 ? 0xffffu : 0u) | (c1 < 2 ? 0xffff0000u : 0u);
                    down[q] = (c0 >> 1 == 1 ? 0xffffu : 0u) | (c1 >> 1 == 1 ? 0xffff0000u : 0u);
                    place |= (uint32_t)((c0 & 1) | (2 | (c1 & 1)) << 2) << (4 * q);
                }
                const int at = co * dgroups + yh * per + m;
                dz[at] = u32x4{h[0] & up[0], h[1] & up[1], h[0] & down[0], h[1] & down[1]};
                dz[at + splane] = u32x4{mi[0] & up[0], mi[1] & up[1], mi[0] & down[0], mi[1] & down[1]};
                dz[at + 2 * splane] = u32x4{lo[0] & up[0], lo[1] & up[1], lo[0] & down[0], lo[1] & down[1]};
                places[at] = (uint16_t)(place | place << 8);
            }
            __syncthreads();
            if (idle) continue;
            const int steps = rows / 2 * segs;
            for (int st = kwave; st < steps; st += a.p.kw) {
                const int yh = st / segs, sg = st % segs, at = arow + yh * per + 2 * sg;
                planes fa;
                fa.h = dz[at];
                fa.m = dz[at + splane];
                fa.l = dz[at + 2 * splane];
                const int place = places[at] | 0x8888;   // (channels beyond the last: two different places as well)
                const u32x4 *bp = img + brow + (r0 + 2 * yh) * (IP / 8) + 2 * sg;
                // fragment kw of one plane of the image: elements kw .. kw + 15 of the twenty read
                split_bf16::u32x8 fb[KS];
                auto read = [&](int plane) {
                    const u32x4 q0 = bp[plane * iplane], q1 = bp[plane * iplane + 1];
                    const u32x2 r = *(const u32x2 *)&bp[plane * iplane + 2];
                    const uint32_t d[10] = {q0[0], q0[1], q0[2], q0[3], q1[0], q1[1], q1[2], q1[3], r[0], r[1]};
#pragma unroll
                    for (int k = 0; k < KS; ++k)
#pragma unroll
                        for (int i = 0; i < 8; ++i) fb[k][i] = k % 2 == 0 ? d[k / 2 + i] : __builtin_amdgcn_alignbit(d[k / 2 + i + 1], d[k / 2 + i], 16);
                };
                auto step = [&](const u32x4 &x) {
#pragma unroll
                    for (int k = 0; k < KS; ++k) split_bf16::mma_sparse(x, fb[k], place, acc[k]);
                };
                read(2);
                step(fa.h);
                read(1);
                step(fa.m);
                step(fa.h);
                read(0);
                step(fa.l);
                step(fa.m);
                step(fa.h);
            }
        }
    // ---- some sum of the workgroup is not finite: again, in the order that tells infinities from NaN (see split_bf16.h).  The
    // look at the sums and the vote take 2 us of 38 (489 samples of 16 x 16, 12 -> 24 channels); looking at the middle filter column
    // alone would take 1, but miss partial products beyond the range of fp32 whose sum is an infinity
#pragma unroll
    for (int k = 0; k < KS; ++k) bad |= n < Cin * KS && split_bf16::any_not_finite(acc[k]);
    uint8_t *votes = (uint8_t *)(dz + dgroups - 1);    // behind the first channel's deltas: 16 bytes that nobody else uses, zero so far
    if (__any(bad) && lane == 0) votes[wave] = 1;
    __syncthreads();
    const u32x4 vote = *(const u32x4 *)votes;
    if (vote[0] | vote[1] | vote[2]) {                 // (12 waves at most)
        zero();
        __syncthreads();                               // the votes have been read
        for (int e = tid; e < 3 * dplane; e += threads) dz[e] = u32x4{0u, 0u, 0u, 0u};
        products(std::true_type{}, std::false_type{});
#pragma unroll
        for (int k = 0; k < KS; ++k) split_bf16::drop_not_finite(acc[k]);
        products(std::false_type{}, std::true_type{});
    }
    // ---- the waves that share a block: their sums through LDS, added to the first one's in wave order
    float *sums = (float *)sm + (wave % upg) * 1024 * KS + lane;
    for (int q = 1; q < a.p.kw; ++q) {
        __syncthreads();                               // the tiles and the votes, or the sums before, have been read
        if (kwave == q)
#pragma unroll
            for (int k = 0; k < KS; ++k)
#pragma unroll
                for (int v = 0; v < 16; ++v) sums[64 * (16 * k + v)] = acc[k][v];
        __syncthreads();
        if (kwave == 0)
#pragma unroll
            for (int k = 0; k < KS; ++k)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[k][v] += sums[64 * (16 * k + v)];
    }
    if (idle || kwave != 0) return;

    float *pb = a.part + w * a.part_stride + (int64_t)blockIdx.x * Cout * TAPS;
    if (n < Cin * KS) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int co = 32 * mb + 8 * (v / 4) + 4 * (lane >> 5) + v % 4;
            if (co < Cout) {
#pragma unroll
                for (int k = 0; k < KS; ++k) pb[(int64_t)co * TAPS + n * KS + k] = acc[k][v];
            }
        }
    }
}

}  // namespace convsplit
