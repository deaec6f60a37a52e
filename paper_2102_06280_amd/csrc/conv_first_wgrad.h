// Weight gradient of a convolution with few input channels (the network's first): dW[co][t] = sum over samples and pixels of
// dz[co][y][x] in[c][y + kh - pad][x + kw - pad], t = (c, kh, kw), with dz given as pooled gradients and window codes.
//
// conv_split.h's kernel takes 32 rows (c, kh) as a fragment's columns, of which one channel fills three or five and three
// channels nine or fifteen.  Here the columns are the taps themselves, sixteen to a block (v_mfma_f32_16x16x32_bf16: rows
// lane % 16, reduction values 8 (lane / 16) .. + 7), so that 25 taps fill 32 and 75 fill 80, and the output channels come in blocks of
// sixteen.  The reduction runs over pixels, eight consecutive ones of a row to a lane; which row and which eight is the lane
// group's own affair, so a row need only be padded to a multiple of eight.
//
// The image lies in LDS once for every kw, shifted by it, as [plane][c][kw][row][8 pixels]: a lane's fragment of any tap is one aligned
// 16-byte read and nothing has to be shifted afterwards.  With one to three channels that is 30 to 40 KB for a tile of the image, and
// four workgroups share a compute unit.  The deltas are nobody else's: a wavefront has all taps of its rows, so it fetches the pooled
// gradients and codes of its own pixels into registers, splits them once and masks them into the two pixel rows of the windows.
// The four wavefronts of a workgroup take turns with the pixels; their sums meet in LDS at the end.  Every workgroup writes a
// partial result: part[worker][split][co][taps], summed in split order by a separate pass.
//
// Six of the nine partial products are kept, like in the other convolutions.  A wavefront's six instructions of one step start from
// zero and their result is added to the sum, so that the sum is rounded once in 32 pixels and not six times.  The bf16 instructions cut off
// what does not fit towards minus infinity, which adds up; the deltas of odd rows therefore enter negated and
// their steps are subtracted.  Error of dW against 64 bits (2-norm; normal pixels and deltas), fp32 instruction / products added
// to the sum directly / now: 64 workers x 32 samples, 3 -> 32 channels, 32 x 32 pixels, 5 x 5 2.3e-7 / 3.7e-7 / 1.2e-7; 4 x 8 1.9e-7 / 2.1e-7 /
// 0.9e-7; conv_split.h's kernel for the first: 16 x 50, 1 -> 16, 28 x 28, 5 x 5 2.5e-7 / 2.5e-7 / 1.5e-7.
//
// us, before (conv_split.h's kernel; an fp32 one for the third) / now: 16 workers x 50 samples, 1 -> 16 channels, 28 x 28 pixels, 5 x 5:
// 73 / 15; 32 x 32, 3 -> 16, 32 x 32, 3 x 3: 39 / 21; 64 x 32, 3 -> 32, 32 x 32, 5 x 5: 114 / 99 (the products added directly: 14, 21,
// 98).  The last has matrix instructions for 28 us; three wavefronts to a SIMD (registers) wait two thirds of their time, for the copies, the
// deltas and each other.  Not faster: the next tile's pixels and deltas requested ahead (113, the deltas alone 106), four
// wavefronts (206, registers spill), larger tiles (101).
#pragma once

#include "conv_split.h"

namespace convsplit {

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct FirstWgradPlan {
    int mb, nb;                 // 16-row blocks of a workgroup (one or two), 16-column blocks
    int rows, sb, splits;       // image rows of a tile, samples per workgroup, partial results per worker
    size_t lds;
};

// 16-byte groups of the version of a channel for one kw, and of a plane.  LDS serves sixteen lanes at a time (0-3, 12-15, 20-27 and 4-11, 16-19,
// 28-31 of either half of a wavefront), whose groups should differ mod 16.  Without the padding the taps of a filter row would all
// meet: 5.6 cycles for sixteen lanes instead of 2.0 with three channels of 32 x 32 and 5 x 5, tiles of eight rows.
__host__ __device__ inline int first_wgrad_version(const Shape &s, int rows)
{
    const int g = first_groups(s), want = g % 4 == 0 ? 6 : (g % 2 == 0 ? 10 : 11), n = (rows + s.KS - 1) * g;
    return n + (want - n % 16 + 16) % 16;
}
__host__ __device__ inline int first_wgrad_plane(const Shape &s, int rows) { return s.Cin * s.KS * first_wgrad_version(s, rows); }

// Left to conv_split.h's kernel, this one / that (us): tiles of two rows, two thirds of whose pixels are halo (16 workers x 32 samples, 3 -> 32
// channels, 48 x 48 pixels, 5 x 5 125 / 76; 64 x 64 177 / 133; 7 -> 32, 48 x 48, 3 x 3 113 / 78; tiles of four: 2 -> 32, 64 x 64, 5 x 5 0.8 times as
// long here), and 3 x 3 filters of six to eight channels with more than sixteen output channels, where that kernel's column blocks are more
// than half full and this one's tiles leave wavefronts idle (6 -> 64, 32 x 32 59 / 51; 7 -> 64, 16 x 16 20.5 / 17.5; 8 -> 32, 24 x 24
// even; 6 -> 64 on 24 x 24 0.85 times as long here; up to sixteen output channels 6 -> 8, 32 x 32 0.84, five channels 5 -> 64 0.92).
inline bool first_wgrad_plan(const Shape &s, int workers, FirstWgradPlan &p)
{
    if (s.KS != 3 && s.KS != 5) return false;
    p.nb = (s.Cin * s.KS * s.KS + 15) / 16;
    if (p.nb > 5) return false;                          // (registers: a wavefront has all taps)
    p.mb = s.Cout <= 16 ? 1 : 2;
    if (s.KS == 3 && p.nb > 3 && p.mb == 2) return false;
    const size_t sums = sizeof(float) * 4 * p.mb * p.nb * 256;
    int tiles = 1;
    for (;; ++tiles) {                                   // the fewest tiles of which four workgroups fit a compute unit; a thread per group
        p.rows = ((s.H + tiles - 1) / tiles + 1) / 2 * 2;
        if (p.rows == 2) return false;
        p.lds = (size_t)48 * first_wgrad_plane(s, p.rows);
        if (p.lds <= 39 * 1024 && s.Cin * (p.rows + s.KS - 1) * first_groups(s) <= THREADS) break;
    }
    if (p.lds < sums) p.lds = sums;
    const int64_t blocks = (int64_t)workers * ((s.Cout + 16 * p.mb - 1) / (16 * p.mb));
    const int64_t slots = 256 * (p.mb == 1 ? 4 : 3);     // workgroups that run at a time (registers): as few turns as that takes
    p.sb = (int)((s.B * blocks + slots - 1) / slots);
    p.sb = p.sb < 1 ? 1 : (p.sb > 8 ? 8 : p.sb);
    p.splits = (s.B + p.sb - 1) / p.sb;
    return true;
}

struct FirstWgradArgs {
    Shape s;
    FirstWgradPlan p;
    const float *in;            // [worker][B][Cin][H][W]
    int64_t in_stride;
    const float *dp;            // pooled gradients [worker][B][Cout][H/2][W/2], with code
    int64_t dp_stride;
    const uint8_t *code;
    int64_t code_stride;
    float *part;
    int64_t part_stride;
};

__device__ __forceinline__ bool not_finite4(const f32x4 &a)
{
    float t = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) t = fmaf(a[v], 0.f, t);
    return t != t;
}

// grid = (splits, workers, blocks of 16 MB output channels); dynamic LDS = plan.lds.
template <int KS, int MB, int NB>
__global__ __launch_bounds__(THREADS, 3) void first_wgrad_kernel(FirstWgradArgs a)
{
    extern __shared__ __attribute__((aligned(16))) u32x4 sm[];
    __shared__ int votes[4];
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    constexpr int PAD = KS / 2, PX = 8 + KS - 1;         // pixels behind the KS versions of a group
    const int H = a.s.H, W = a.s.W, Cin = a.s.Cin, Cout = a.s.Cout, TAPS = Cin * KS * KS, G = first_groups(a.s);
    const int TR = a.p.rows, RT = TR + KS - 1, version = first_wgrad_version(a.s, TR), plane = first_wgrad_plane(a.s, TR);
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = blockIdx.y, b0 = blockIdx.x * a.p.sb, b1 = min(a.s.B, b0 + a.p.sb), m0 = 16 * MB * blockIdx.z;
    const float *inw = a.in + w * a.in_stride, *dpw = a.dp + w * a.dp_stride;
    const uint8_t *cdw = a.code + w * a.code_stride;

    int tap[NB];                                         // the lane's column of each block (beyond the taps: the first, never stored)
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int t = 16 * n + l16 < TAPS ? 16 * n + l16 : 0, c = t / (KS * KS), kh = t / KS % KS, kw = t % KS;
        tap[n] = (c * KS + kw) * version + kh * G;
    }
    f32x4 acc[MB][NB];
    auto zero = [&] {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int n = 0; n < NB; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    zero();

    // the partial products of the whole reduction, all of them or those of one kind.  MASK: pixels that meet only padding are left
    // out (otherwise they meet zeros there, which is the same for finite values)
    auto products = [&](auto small, auto large, auto mask) {
        constexpr bool SMALL = decltype(small)::value, LARGE = decltype(large)::value, MASK = decltype(mask)::value;
        for (int b = b0; b < b1; ++b)
            for (int r0 = 0; r0 < H; r0 += TR) {
                const int rows = min(TR, H - r0), units = rows / 2 * G;
                __syncthreads();                           // the tile before has been used
                if (tid < Cin * RT * G) {
                    const int m = tid % G, r = tid / G % RT, c = tid / G / RT, y = r0 + r - PAD;
                    const float *src = inw + (((int64_t)b * Cin + c) * H + min(max(y, 0), H - 1)) * W;
                    float v[PX];
#pragma unroll
                    for (int j = 0; j < PX; ++j) {
                        const int x = 8 * m + j - PAD;
                        const float f = src[min(max(x, 0), W - 1)];
                        v[j] = (unsigned)x < (unsigned)W && (unsigned)y < (unsigned)H ? f : 0.f;
                    }
                    uint32_t q[3][PX / 2];
                    split_bf16::split_nearest(v, q[0], q[1], q[2]);
                    u32x4 *d = sm + c * KS * version + r * G + m;
#pragma unroll
                    for (int kw = 0; kw < KS; ++kw)
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            u32x4 f;
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                f[i] = kw % 2 == 0 ? q[k][kw / 2 + i] : __builtin_amdgcn_alignbit(q[k][kw / 2 + i + 1], q[k][kw / 2 + i], 16);
                            d[k * plane + kw * version] = f;
                        }
                }
                __syncthreads();
                for (int u0 = 4 * wave; u0 < units; u0 += 16) {
                    const bool real = u0 + lq < units;
                    const int u = real ? u0 + lq : 0, yp = u / G, m = u % G;
                    const bool whole = real && 8 * m + 4 < W;                // (the width divides by four)
                    uint32_t q[MB][3][2], cd[MB][4];                         // pooled gradients as planes of pairs, window codes
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) {
                        const int co = m0 + 16 * mb + l16;
                        const int64_t o = (((int64_t)b * Cout + min(co, Cout - 1)) * (H / 2) + r0 / 2 + yp) * (W / 2) + 4 * m;
                        const int second = whole ? 2 : 0;
                        const f32x2 d0 = *(const f32x2 *)(dpw + o), d1 = *(const f32x2 *)(dpw + o + second);
                        const uint32_t e0 = *(const uint16_t *)(cdw + o), e1 = *(const uint16_t *)(cdw + o + second);
                        const bool ok0 = real && co < Cout, ok1 = whole && co < Cout;
                        const float g[4] = {ok0 ? d0[0] : 0.f, ok0 ? d0[1] : 0.f, ok1 ? d1[0] : 0.f, ok1 ? d1[1] : 0.f};
                        const uint32_t c0 = ok0 ? e0 : 0x0404u, c1 = ok1 ? e1 : 0x0404u;
                        cd[mb][0] = c0 & 0xffu;
                        cd[mb][1] = c0 >> 8;
                        cd[mb][2] = c1 & 0xffu;
                        cd[mb][3] = c1 >> 8;
                        split_bf16::split_nearest(g, q[mb][0], q[mb][1], q[mb][2]);
                    }
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        if (r == 1) {                                        // the signs of the second row's, see above
#pragma unroll
                            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                                for (int k = 0; k < 3; ++k)
#pragma unroll
                                    for (int j = 0; j < 2; ++j) q[mb][k][j] ^= 0x80008000u;
                        }
                        u32x4 fa[MB][3];                                     // row r: of each window's four pixels one has its value
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                const uint32_t keep = cd[mb][j] == 2u * r ? 0xffffu : (cd[mb][j] == 2u * r + 1 ? 0xffff0000u : 0u);
#pragma unroll
                                for (int k = 0; k < 3; ++k)
                                    fa[mb][k][j] = __builtin_amdgcn_perm(q[mb][k][j / 2], q[mb][k][j / 2], j % 2 ? 0x03020302u : 0x01000100u) & keep;
                            }
                        const u32x4 *img = sm + (2 * yp + r) * G + m;
                        constexpr int NG = MB == 1 ? 2 : 1;                  // column blocks at a time: two sums under way at least
#pragma unroll
                        for (int n0 = 0; n0 < NB; n0 += NG) {
                            u32x4 fb[NG][3];
#pragma unroll
                            for (int g = 0; g < NG; ++g)
                                if (n0 + g < NB)
#pragma unroll
                                    for (int k = 0; k < 3; ++k) {
                                        fb[g][k] = img[tap[n0 + g] + k * plane];
                                        if (MASK) {
                                            fb[g][k][0] = real ? fb[g][k][0] : 0u;
                                            fb[g][k][1] = real ? fb[g][k][1] : 0u;
                                            fb[g][k][2] = whole ? fb[g][k][2] : 0u;
                                            fb[g][k][3] = whole ? fb[g][k][3] : 0u;
                                        }
                                    }
                            f32x4 t[MB][NG];
#pragma unroll
                            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                                for (int g = 0; g < NG; ++g) t[mb][g] = f32x4{0.f, 0.f, 0.f, 0.f};
                            auto step = [&](int ka, int kb) {
#pragma unroll
                                for (int g = 0; g < NG; ++g)
                                    if (n0 + g < NB)
#pragma unroll
                                        for (int mb = 0; mb < MB; ++mb)
                                            t[mb][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(split_bf16::frag(fa[mb][ka]), split_bf16::frag(fb[g][kb]),
                                                                                               t[mb][g], 0, 0, 0);
                            };
                            if (SMALL) {
                                step(0, 2);
                                step(1, 1);
                                step(0, 1);
                                step(2, 0);
                                step(1, 0);
                            }
                            if (LARGE) step(0, 0);
#pragma unroll
                            for (int g = 0; g < NG; ++g)
                                if (n0 + g < NB)
#pragma unroll
                                    for (int mb = 0; mb < MB; ++mb) acc[mb][n0 + g] = r == 0 ? acc[mb][n0 + g] + t[mb][g] : acc[mb][n0 + g] - t[mb][g];

                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
    };
    products(std::true_type{}, std::true_type{}, std::false_type{});
    // ---- some sum of the workgroup is not finite: again, in the order that tells infinities from NaN (see split_bf16.h)
    bool bad = false;
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) bad |= not_finite4(acc[m][n]);
    const int vote = __any(bad);
    if (lane == 0) votes[wave] = vote;
    __syncthreads();
    if (votes[0] | votes[1] | votes[2] | votes[3]) {
        zero();
        products(std::true_type{}, std::false_type{}, std::true_type{});
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[m][n][v] = split_bf16::not_finite(acc[m][n][v]) ? 0.f : acc[m][n][v];
        products(std::false_type{}, std::true_type{}, std::true_type{});
        __syncthreads();
    }

    // ---- the wavefronts' sums through LDS, added in wavefront order.  Register v of a lane: channel 4 lq + v, column l16 of the block.
    f32x4 *sums = (f32x4 *)sm;
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) sums[((wave * MB + m) * NB + n) * 64 + lane] = acc[m][n];
    __syncthreads();
    float *pb = a.part + w * a.part_stride + (int64_t)blockIdx.x * Cout * TAPS;
    for (int q = wave; q < MB * NB; q += 4) {
        const int m = q / NB, n = q % NB, t = 16 * n + l16;
        f32x4 s = sums[q * 64 + lane];
#pragma unroll
        for (int k = 1; k < 4; ++k) s += sums[(k * MB * NB + q) * 64 + lane];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int co = m0 + 16 * m + 4 * lq + v;
            if (co < Cout && t < TAPS) pb[(int64_t)co * TAPS + t] = s[v];
        }
    }
}

}  // namespace convsplit
