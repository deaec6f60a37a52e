// Weight gradient of a stride-1 'same' convolution with fp32 matrix instructions, input image and deltas resident in LDS:
// the first layer of the 3 -> 32 channel network on 32 x 32 inputs (5 x 5 filters), where half of a column block of
// conv_split.h's kernel is padding (64 workers x 32 samples: 115 us here, 151 there).
//
// Fragment layout of v_mfma_f32_16x16x4_f32, lane l: A[m = l % 16][slot l / 16],
// B[slot l / 16][n = l % 16], D: d[v] = D[m = 4 (l / 16) + v][n = l % 16]; instruction j of a
// 16-wide k group uses k = 4 slot + j.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace convlds {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Four horizontally adjacent pixels (x = 4 x4 .. 4 x4 + 3 of image row y) of a map that is stored
// as its 2 x 2 max-pooled gradient plus the window codes of the forward pass: a pixel
// holds the pooled gradient of its window if it was the window's first maximum, else zero.
// `pooled` / `code` point at the plane [H/2][W/2] of one (sample, channel).
__device__ __forceinline__ float4 expand_pooled(const float *pooled, const uint8_t *code, int y, int x4, int W)
{
    const int o = (y >> 1) * (W >> 1) + 2 * x4;
    const float2 g = *(const float2 *)&pooled[o];
    const uint32_t c = *(const uint16_t *)&code[o];
    const uint32_t c0 = c & 0xffu, c1 = c >> 8, pos = (uint32_t)(y & 1) * 2u;
    return make_float4(c0 == pos ? g.x : 0.f, c0 == pos + 1 ? g.x : 0.f, c1 == pos ? g.y : 0.f, c1 == pos + 1 ? g.y : 0.f);
}

// dW[co][t] = sum over samples b and pixels p of
// dz[b][co][p] * in[b][tap t shifted by p], as the GEMM with M = output channels, N = filter
// taps t = (c, kh, kw), K = pixels.  The sample's input (all CIN channels, zero halo) and a
// chunk of PC pixels of its deltas sit in LDS.  The A fragment (deltas, k = pixel) is a
// 128-bit LDS read; the B fragment is img[tap_offset(lane's tap) + pixel_offset(k)], where
// the pixel offset of k = 16 kg + 4 slot + j is a per-lane constant plus a compile-time
// immediate, so the reads need no address arithmetic at all.
// Waves are arranged WM (channels) x WN (taps) x WK (pixels); every (workgroup, wk) pair
// writes its own partial result  part[worker][split = blockIdx.x * WK + wk][co][t], which a
// separate pass sums in split order (deterministic).  grid = (ceil(B / SB), workers).
template <int CIN, int MT, int NT, int WM, int WN, int WK, int H, int W, int KS, int PC>
struct WCfg {
    static constexpr int PAD = KS / 2, HP = H + 2 * PAD, WP = W + 2 * PAD;
    static constexpr int COUT = 16 * MT * WM, PIX = H * W, KK = KS * KS, TAPS = CIN * KK;
    static constexpr int WAVES = WM * WN * WK, THREADS = 64 * WAVES;
    static constexpr int IMG = CIN * HP * WP;
    static constexpr int LDD = PC + 4;                   // row stride of the delta tile [COUT][PC]
    static constexpr int KG_CHUNK = PC / 16, KG_WAVE = KG_CHUNK / WK;
    static_assert(16 * NT * WN >= TAPS, "tap fragments must cover all taps");
    static_assert(PIX % PC == 0 && KG_CHUNK % WK == 0 && W % 16 == 0, "shape not supported");
    static constexpr size_t lds_bytes = sizeof(float) * (IMG + COUT * LDD);
};

// The deltas are given as the pooled gradients [worker][B][COUT][H/2][W/2] with dz_code of the same shape
// and are expanded while the tile is copied into LDS (see expand_pooled).
template <int CIN, int MT, int NT, int WM, int WN, int WK, int H, int W, int KS, int PC>
__global__ __launch_bounds__(64 * WM * WN * WK) void conv_wgrad_kernel(
    const float *__restrict__ in, int64_t in_stride, const float *__restrict__ dz, int64_t dz_stride,
    float *__restrict__ part, int64_t part_stride, int B, int SB, const uint8_t *__restrict__ dz_code,
    int64_t dz_code_stride)
{
    using C = WCfg<CIN, MT, NT, WM, WN, WK, H, W, KS, PC>;
    __shared__ __attribute__((aligned(16))) float img[C::IMG];
    __shared__ __attribute__((aligned(16))) float dzs[C::COUT * C::LDD];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = (wave / WM) % WN, wk = wave / (WM * WN);
    const int w = blockIdx.y, b0 = blockIdx.x * SB, b1 = min(B, b0 + SB);

    for (int e = tid; e < C::IMG; e += C::THREADS) img[e] = 0.f;     // the halo stays zero

    // per-lane LDS element index of this lane's tap (plus its k-slot) for each tap fragment
    int bbase[NT];
#pragma unroll
    for (int nf = 0; nf < NT; ++nf) {
        const int t = 16 * (wn * NT + nf) + (lane & 15);
        const int c = t / C::KK, rr = t % C::KK, kh = rr / KS, kw = rr % KS;
        bbase[nf] = (t < C::TAPS ? c * C::HP * C::WP + kh * C::WP + kw : 0) + 4 * (lane >> 4);
    }
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nf = 0; nf < NT; ++nf) acc[mt][nf] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int b = b0; b < b1; ++b) {
        const float *inb = in + w * in_stride + (int64_t)b * CIN * C::PIX;
        const float *dzb = dz + w * dz_stride + (int64_t)b * C::COUT * (C::PIX / 4);
        const uint8_t *dcb = dz_code + w * dz_code_stride + (int64_t)b * C::COUT * (C::PIX / 4);
        for (int chunk = 0; chunk < C::PIX / PC; ++chunk) {
            __syncthreads();                   // previous tile fully consumed
            if (chunk == 0) {
                for (int e = tid; e < CIN * H * (W / 4); e += C::THREADS) {
                    const int c = e / (H * (W / 4)), rem = e % (H * (W / 4)), y = rem / (W / 4), x4 = rem % (W / 4);
                    const float4 v = *(const float4 *)&inb[(c * H + y) * W + 4 * x4];
                    float *dst = &img[c * C::HP * C::WP + (y + C::PAD) * C::WP + C::PAD + 4 * x4];
                    dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
                }
            }
            for (int e = tid; e < C::COUT * (PC / 4); e += C::THREADS) {
                const int co = e / (PC / 4), p4 = e % (PC / 4), p = chunk * PC + 4 * p4;
                *(float4 *)&dzs[co * C::LDD + 4 * p4] =
                    expand_pooled(dzb + co * (C::PIX / 4), dcb + co * (C::PIX / 4), p / W, (p % W) / 4, W);
            }
            __syncthreads();
            const int chunk_row = chunk * (PC / W);                  // first image row of the chunk
            // k runs over the wave's pixel groups i (16 pixels each) and the four k-slots j of a
            // group; the B values of step (i, j) + 1 are requested before the multiplies of step
            // (i, j), and scheduling barriers keep the compiler from requesting more than that
            // ahead (hundreds of values otherwise, which spill)
            auto pixel_offset = [&](int i) {
                const int kgl = wk * C::KG_WAVE + i;                 // k group inside the chunk (wave-uniform)
                // W % 16 == 0 keeps a group inside one image row
                return (chunk_row + (16 * kgl) / W) * C::WP + (16 * kgl) % W;
            };
            float fb[2][NT];
            {
                const int poff = pixel_offset(0);
#pragma unroll
                for (int nf = 0; nf < NT; ++nf) fb[0][nf] = img[bbase[nf] + poff];
            }
#pragma unroll
            for (int i = 0; i < C::KG_WAVE; ++i) {
                const int kgl = wk * C::KG_WAVE + i;
                f32x4 fa[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    fa[mt] = *(const f32x4 *)&dzs[(16 * (wm * MT + mt) + (lane & 15)) * C::LDD + 16 * kgl + 4 * (lane >> 4)];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int step = 4 * i + j;
                    if (step + 1 < 4 * C::KG_WAVE) {
                        const int poff = pixel_offset((step + 1) / 4) + (step + 1) % 4;
#pragma unroll
                        for (int nf = 0; nf < NT; ++nf) fb[(step + 1) & 1][nf] = img[bbase[nf] + poff];
                    }
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int nf = 0; nf < NT; ++nf)
                            acc[mt][nf] =
                                __builtin_amdgcn_mfma_f32_16x16x4f32(fa[mt][j], fb[step & 1][nf], acc[mt][nf], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }

    float *pb = part + w * part_stride + (int64_t)(blockIdx.x * WK + wk) * C::COUT * C::TAPS;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nf = 0; nf < NT; ++nf) {
            const int t = 16 * (wn * NT + nf) + (lane & 15);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int co = 16 * (wm * MT + mt) + 4 * (lane >> 4) + v;
                if (t < C::TAPS) pb[co * C::TAPS + t] = acc[mt][nf][v];
            }
        }
}

}  // namespace convlds
