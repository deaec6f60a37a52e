// Mini-batch gradients of the convolutional model for all workers at once (Section 2.1,
// stochastic gradient of the local loss).  Network per worker, input [B][C0][H][W]:
//   conv KxK (C0->C1, same padding) -> ReLU -> maxpool 2x2 -> conv KxK (C1->C2, same) ->
//   ReLU -> maxpool 2x2 -> flatten [C2][H/4][W/4] -> FC F -> ReLU -> FC classes -> softmax
//   cross-entropy, mean over the batch.
// Parameter row layout: conv1 W [C1][C0][K][K], b [C1]; conv2 W [C2][C1][K][K], b [C2];
// fc1 W [F][flat], b [F]; fc2 W [classes][F], b [classes].
//
// Convolutions with 3 x 3 and 5 x 5 filters take the LDS-resident kernels of conv_split.h and conv_first_wgrad.h; the rest are implicit GEMMs on the
// batched fp32 MFMA kernel: the patch matrix is never materialised, the operand loaders compute the input address of each element.
//   forward   z[co][pix]      = sum_k  W[co][k] * patch[k][pix]        k = (ci, kh, kw)
//   wgrad     dW[co][k]       = sum_pix dz[co][pix] * patch[k][pix]
//   dgrad     din[ci][pix_in] = sum_k' W[co][ci][kh][kw] * dz[co][pix_in shifted]   k' = (co, kh, kw)
// Output channels are the GEMM's M and pixels its N, so stores run along consecutive pixels.
// Max pooling keeps a code per window (the first maximum in window order (0,0),(0,1),(1,0),(1,1)) where the backward
// kernels read codes; otherwise the backward pass re-derives it from the stored pre-activations.
#include <algorithm>

#include "bgemm.h"
#include "conv_first_wgrad.h"
#include "conv_split.h"
#include "dbw_internal.h"

namespace {

using bgemm::Dense;

struct ConvShape {
    int Cin, Cout, H, W, KS, pad;   // stride-1 'same' convolution
};

// Filter size as a compile-time constant where it is a common one (KS_ = 0: run time), so
// that splitting k into (channel, tap) needs no division.
template <int KS_>
__device__ __forceinline__ int filter_size(const ConvShape &s) { return KS_ > 0 ? KS_ : s.KS; }

// Contexts shared by the convolution loaders.  A pixel context addresses tensor element
// (b, channel 0, y, x) of a [B][C][H][W] tensor; a tap context adds the channel plane and
// the (dy, dx) shift of one filter tap.  Element = base + off, valid iff the shifted
// position is inside the image.
struct PixelCtx { int base, y, x; bool ok; };
struct TapCtx { int off, dy, dx; bool ok; };

__device__ __forceinline__ PixelCtx pixel_ctx(const ConvShape &s, int C, int pix, bool ok)
{
    const int HW = s.H * s.W;
    const int b = pix / HW, hw = pix - b * HW, y = hw / s.W, x = hw - y * s.W;
    return {b * C * HW + hw, y, x, ok};
}

// k = (channel, kh, kw); sign = +1 reads the input of a forward tap (y + kh - pad),
// sign = -1 the output position that used this input with that tap (y - kh + pad).
template <int KS_>
__device__ __forceinline__ TapCtx tap_ctx(const ConvShape &s, int k, int sign, bool ok)
{
    const int KS = filter_size<KS_>(s), KK = KS * KS;
    const int ch = k / KK, rr = k - ch * KK, kh = rr / KS, kw = rr - kh * KS;
    const int dy = sign * (kh - s.pad), dx = sign * (kw - s.pad);
    return {ch * s.H * s.W + dy * s.W + dx, dy, dx, ok};
}

__device__ __forceinline__ float conv_load(const float *t, const ConvShape &s, const PixelCtx &p, const TapCtx &k)
{
    const bool ok = p.ok && k.ok && (unsigned)(p.y + k.dy) < (unsigned)s.H && (unsigned)(p.x + k.dx) < (unsigned)s.W;
    const float v = t[ok ? p.base + k.off : 0];
    return ok ? v : 0.f;
}

// B operand of the forward GEMM: (k = tap, row = output pixel), contiguous along pixels.
template <int KS_>
struct PatchRC {
    static constexpr bool KC = false;
    const float *in;
    int64_t stride;
    ConvShape s;
    typedef PixelCtx RowCtx;
    typedef TapCtx KCtx;
    __device__ __forceinline__ RowCtx row_ctx(int pix, bool ok) const { return pixel_ctx(s, s.Cin, pix, ok); }
    __device__ __forceinline__ KCtx k_ctx(int k, bool ok) const { return tap_ctx<KS_>(s, k, 1, ok); }
    __device__ __forceinline__ float load(int w, const RowCtx &r, const KCtx &k) const
    {
        return conv_load(in + w * stride, s, r, k);
    }
};

// B operand of the weight-gradient GEMM: row = filter tap, reduction index = output pixel.
template <int KS_>
struct PatchKC {
    static constexpr bool KC = true;
    const float *in;
    int64_t stride;
    ConvShape s;
    typedef TapCtx RowCtx;
    typedef PixelCtx KCtx;
    __device__ __forceinline__ RowCtx row_ctx(int kf, bool ok) const { return tap_ctx<KS_>(s, kf, 1, ok); }
    __device__ __forceinline__ KCtx k_ctx(int pix, bool ok) const { return pixel_ctx(s, s.Cin, pix, ok); }
    __device__ __forceinline__ float load(int w, const RowCtx &r, const KCtx &k) const
    {
        return conv_load(in + w * stride, s, k, r);
    }
};

// A operand of the weight-gradient GEMM: dz[co][pix] stored as [B][Cout][H][W].
struct DeltaKC {
    static constexpr bool KC = true;
    const float *dz;
    int64_t stride;
    int Cout, HW;
    struct RowCtx { int off; bool ok; };
    struct KCtx { int base; bool ok; };
    __device__ __forceinline__ RowCtx row_ctx(int co, bool ok) const { return {co * HW, ok}; }
    __device__ __forceinline__ KCtx k_ctx(int pix, bool ok) const
    {
        const int b = pix / HW, hw = pix - b * HW;
        return {b * Cout * HW + hw, ok};
    }
    __device__ __forceinline__ float load(int w, const RowCtx &r, const KCtx &k) const
    {
        const bool ok = r.ok && k.ok;
        const float v = (dz + w * stride)[ok ? r.off + k.base : 0];
        return ok ? v : 0.f;
    }
};

// A operand of the data-gradient GEMM: (row = ci, k' = (co, kh, kw)) -> W[co][ci][kh][kw].
template <int KS_>
struct FilterT {
    static constexpr bool KC = true;
    const float *wgt;
    int64_t stride;
    int Cin, KKrt;
    struct RowCtx { int off; bool ok; };
    struct KCtx { int base; bool ok; };
    __device__ __forceinline__ RowCtx row_ctx(int ci, bool ok) const { return {ci * (KS_ > 0 ? KS_ * KS_ : KKrt), ok}; }
    __device__ __forceinline__ KCtx k_ctx(int k, bool ok) const
    {
        const int KK = KS_ > 0 ? KS_ * KS_ : KKrt;
        const int co = k / KK, rr = k - co * KK;
        return {co * Cin * KK + rr, ok};
    }
    __device__ __forceinline__ float load(int w, const RowCtx &r, const KCtx &k) const
    {
        const bool ok = r.ok && k.ok;
        const float v = (wgt + w * stride)[ok ? r.off + k.base : 0];
        return ok ? v : 0.f;
    }
};

// B operand of the data-gradient GEMM: (k' = (co, kh, kw), row = input pixel) -> dz at the
// output position that used this input pixel with that filter tap; zero outside.
template <int KS_>
struct DeltaShiftRC {
    static constexpr bool KC = false;
    const float *dz;
    int64_t stride;
    ConvShape s;
    typedef PixelCtx RowCtx;
    typedef TapCtx KCtx;
    __device__ __forceinline__ RowCtx row_ctx(int pix, bool ok) const { return pixel_ctx(s, s.Cout, pix, ok); }
    __device__ __forceinline__ KCtx k_ctx(int k, bool ok) const { return tap_ctx<KS_>(s, k, -1, ok); }
    __device__ __forceinline__ float load(int w, const RowCtx &r, const KCtx &k) const
    {
        return conv_load(dz + w * stride, s, r, k);
    }
};

// Store C[m = channel][n = pixel] into a [B][C][H][W] tensor, adding a per-channel bias.
struct ChannelPixelOut {
    float *out;
    int64_t stride;
    int C, HW;
    const float *bias;     // per worker at bias[w * bias_stride + channel]; nullptr = none
    int64_t bias_stride;
    __device__ __forceinline__ void store(int w, int, int ch, int pix, float v) const
    {
        if (bias) v += bias[w * bias_stride + ch];
        const int b = pix / HW, hw = pix - b * HW;
        out[w * stride + (int64_t)(b * C + ch) * HW + hw] = v;
    }
};

// Partial sums of a split-k GEMM, inside each worker's scratch block: part[split][m][n].
struct PartialOut {
    float *part;
    int64_t stride;
    int M, N;
    __device__ __forceinline__ void store(int w, int split, int m, int n, float v) const
    {
        part[w * stride + ((int64_t)split * M + m) * N + n] = v;
    }
};

// ReLU + 2x2 max pooling of z [B][C][H][W] -> p [B][C][H/2][W/2]; one thread per output.  code (or null): the window
// codes (0..3: position of the first maximum, 4: maximum not positive).
__global__ __launch_bounds__(256) void relu_pool_fwd_kernel(const float *__restrict__ z, int64_t zstride,
                                                            float *__restrict__ p, int64_t pstride, int planes, int H, int W,
                                                            uint8_t *__restrict__ code, int64_t cstride)
{
    const int w = blockIdx.y;
    const int Ho = H / 2, Wo = W / 2, total = planes * Ho * Wo;
    const int o = blockIdx.x * 256 + threadIdx.x;
    if (o >= total) return;
    const int pl = o / (Ho * Wo), rem = o - pl * Ho * Wo, oh = rem / Wo, ow = rem - oh * Wo;
    const float *src = z + w * zstride + ((int64_t)pl * H + 2 * oh) * W + 2 * ow;
    const float v0 = src[0], v1 = src[1], v2 = src[W], v3 = src[W + 1];
    const float m = fmaxf(fmaxf(v0, v1), fmaxf(v2, v3));
    p[w * pstride + o] = fmaxf(m, 0.f);
    if (code) code[w * cstride + o] = m > 0.f ? (v0 == m ? 0 : v1 == m ? 1 : v2 == m ? 2 : 3) : 4;
}

// Backward of ReLU + max pooling: the pooled gradient goes to the first element of the
// window that attains the (positive) maximum; everything else gets zero.
__global__ __launch_bounds__(256) void relu_pool_bwd_kernel(const float *__restrict__ z, int64_t zstride,
                                                            const float *__restrict__ dp, int64_t pstride,
                                                            float *__restrict__ dz, int planes, int H, int W)
{
    const int w = blockIdx.y;
    const int Ho = H / 2, Wo = W / 2, total = planes * Ho * Wo;
    const int o = blockIdx.x * 256 + threadIdx.x;
    if (o >= total) return;
    const int pl = o / (Ho * Wo), rem = o - pl * Ho * Wo, oh = rem / Wo, ow = rem - oh * Wo;
    const int64_t base = w * zstride + ((int64_t)pl * H + 2 * oh) * W + 2 * ow;
    const float v0 = z[base], v1 = z[base + 1], v2 = z[base + W], v3 = z[base + W + 1];
    const float m = fmaxf(fmaxf(v0, v1), fmaxf(v2, v3));
    const float gsrc = dp[w * pstride + o];
    int arg = -1;
    if (m > 0.f) arg = (v0 == m) ? 0 : (v1 == m) ? 1 : (v2 == m) ? 2 : 3;
    dz[base] = arg == 0 ? gsrc : 0.f;
    dz[base + 1] = arg == 1 ? gsrc : 0.f;
    dz[base + W] = arg == 2 ? gsrc : 0.f;
    dz[base + W + 1] = arg == 3 ? gsrc : 0.f;
}

// With the window codes (0..3: position of the first maximum, 4: maximum not positive): db[ch] = sum of dz over
// batch and pixels = sum of the pooled gradients of the windows whose maximum was positive (each passes its gradient to
// exactly one pixel).  One workgroup per (channel, worker).  QUADS (HWo % 4 == 0: 16-byte aligned planes): a thread takes
// four windows at a time (one 128-bit load of gradients, one 32-bit load of codes).
template <bool QUADS>
__device__ __forceinline__ void channel_sum_code(float *red /* LDS [256] */, const uint8_t *__restrict__ code,
                                                 const float *__restrict__ dp, int B, int C, int HWo, int ch, float *__restrict__ db)
{
    constexpr int V = QUADS ? 4 : 1;
    const int tid = threadIdx.x;
    const int per = HWo / V;                         // steps per (sample, channel) plane
    const int q = tid % per, b0 = tid / per, bstep = 256 / per > 0 ? 256 / per : 1;
    float s = 0.f;
    if (b0 < bstep) {
#pragma unroll 4
        for (int b = b0; b < B; b += bstep) {
            for (int qq = q; qq < per; qq += 256) {      // planes wider than 256 steps
                const int64_t o = (int64_t)(b * C + ch) * HWo + V * qq;
                if constexpr (QUADS) {
                    const float4 g = *(const float4 *)&dp[o];
                    const uint32_t cd = *(const uint32_t *)&code[o];
                    s += (cd & 0xffu) < 4u ? g.x : 0.f;
                    s += ((cd >> 8) & 0xffu) < 4u ? g.y : 0.f;
                    s += ((cd >> 16) & 0xffu) < 4u ? g.z : 0.f;
                    s += (cd >> 24) < 4u ? g.w : 0.f;
                } else {
                    const float g = dp[o];
                    s += code[o] < 4 ? g : 0.f;
                }
            }
        }
    }
    red[tid] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) red[tid] += red[tid + o];
        __syncthreads();
    }
    if (tid == 0) *db = red[0];
}

// What is left of a convolution's parameter gradients once its partial weight gradients are there: their sum in split
// order, and (coded) the bias gradients.  Both layers in one launch: four launches of 5 to 30 us each otherwise,
// none of which fills the chip.  grid = (blocks of layer 1 + blocks of layer 2, workers): ceil(weights / 256) blocks that add
// partial results, then, if coded, one per channel.
struct FinishLayer {
    const float *part;           // [worker][split][weights]
    int splits, weights;
    float *dw, *db;
    const uint8_t *code;         // null: the bias gradient is somebody else's
    const float *dp;
    int C, HWo;
    __host__ __device__ int sum_blocks() const { return (weights + 255) / 256; }
    __host__ __device__ int blocks() const { return sum_blocks() + (code ? C : 0); }
};
__global__ __launch_bounds__(256) void finish_kernel(FinishLayer l1, FinishLayer l2, int64_t wstride, int64_t cstride, int64_t gstride, int B)
{
    __shared__ float red[256];
    const int w = blockIdx.y;
    const bool second = (int)blockIdx.x >= l1.blocks();
    const FinishLayer l = second ? l2 : l1;
    const int blk = blockIdx.x - (second ? l1.blocks() : 0);
    if (blk >= l.sum_blocks()) {
        const int ch = blk - l.sum_blocks();
        const uint8_t *code = l.code + w * cstride;
        const float *dp = l.dp + w * wstride;
        if (l.HWo % 4 == 0) channel_sum_code<true>(red, code, dp, B, l.C, l.HWo, ch, l.db + w * gstride + ch);
        else channel_sum_code<false>(red, code, dp, B, l.C, l.HWo, ch, l.db + w * gstride + ch);
        return;
    }
    const int i = blk * 256 + threadIdx.x;
    if (i >= l.weights) return;
    const float *p = l.part + w * wstride + i;
    float s = 0.f;
    int q = 0;
    for (; q + 8 <= l.splits; q += 8) {              // eight loads in flight, added in split order
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(int64_t)(q + u) * l.weights];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; q < l.splits; ++q) s += p[(int64_t)q * l.weights];
    l.dw[w * gstride + i] = s;
}

// db[ch] = sum over batch and pixels of dz[b][ch][hw]; one workgroup per (channel, worker).
__global__ __launch_bounds__(256) void channel_sum_kernel(const float *__restrict__ dz, int64_t stride, int B, int C,
                                                          int HW, float *__restrict__ db, int64_t dbstride)
{
    __shared__ float red[256];
    const int ch = blockIdx.x, w = blockIdx.y, tid = threadIdx.x;
    float s = 0.f;
    for (int i = tid; i < B * HW; i += 256) {
        const int b = i / HW, hw = i - b * HW;
        s += dz[w * stride + (int64_t)(b * C + ch) * HW + hw];
    }
    red[tid] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) red[tid] += red[tid + o];
        __syncthreads();
    }
    if (tid == 0) db[w * dbstride + ch] = red[0];
}

struct cnn_layout {
    int C0, H, W, C1, C2, KS, F, NC, B;
    int H2, W2, H4, W4, flat;
    int fc_dims[3];
    // parameter offsets inside a row
    int64_t w1, b1, w2, b2, fc;
    // scratch offsets inside a worker's block (floats)
    int64_t z1, p1, z2, p2, dp2, dz2, dp1, dz1, fc_act, part1, part2, filt_fwd, filt_bwd, code1, code2, total;
    int splits1, splits2;
    bool first;                     // conv1's forward pass by convsplit::first_kernel
    bool first_wgrad;               // conv1's weight gradient by conv_first_wgrad.h (otherwise, with split1, by wgrad_kernel)
    bool split1, split2;            // weight gradient of conv1 / all three products of conv2 by conv_split.h
    convsplit::WgradPlan wg1, wg2;
    convsplit::FirstPlan fp;
    convsplit::FirstWgradPlan fw;
};

// The kernels of conv_split.h take every 3 x 3 and 5 x 5 filter whose images fit LDS, however few the channels: with 2 -> 4
// of them on 16 x 16 pixels, where most of a reduction step is padding, the three products take 15 + 15 + 14 us
// (16 workers, batch 32) against 20 + 98 + 17 of the implicit GEMM, with 32 -> 64 channels (64 workers) 255 + 274 + 264
// against 433 + 427 + 448 of LDS-resident fp32 kernels.
// (Layers of up to sixteen output channels are launched with 12 KB less than is asked for here: images at the very edge stay with the
// implicit GEMM and its fp32 products.)
bool conv_split_fits(const convsplit::Shape &s, int workers, bool first, convsplit::WgradPlan &plan)
{
    const size_t most = 160 * 1024;
    if (s.KS != 3 && s.KS != 5) return false;
    if (!convsplit::wgrad_plan(s, workers, plan)) return false;
    if (first) return true;
    const convsplit::Shape back{s.Cout, s.Cin, s.H, s.W, s.KS, s.B};
    return convsplit::forward_lds(s, s.Cout <= 32 ? 1 : 2) <= most && convsplit::forward_lds(back, s.Cin <= 32 ? 1 : 2) <= most;
}

cnn_layout make_layout(const dbw_model &m, int workers)
{
    cnn_layout L{};
    L.C0 = m.dims[0]; L.H = m.dims[1]; L.W = m.dims[2]; L.C1 = m.dims[3]; L.C2 = m.dims[4];
    L.KS = m.dims[5]; L.F = m.dims[6]; L.NC = m.dims[7]; L.B = m.batch;
    L.H2 = L.H / 2; L.W2 = L.W / 2; L.H4 = L.H / 4; L.W4 = L.W / 4;
    L.flat = L.C2 * L.H4 * L.W4;
    L.fc_dims[0] = L.flat; L.fc_dims[1] = L.F; L.fc_dims[2] = L.NC;
    const int64_t KK = (int64_t)L.KS * L.KS;
    L.w1 = 0;
    L.b1 = L.w1 + L.C1 * L.C0 * KK;
    L.w2 = L.b1 + L.C1;
    L.b2 = L.w2 + L.C2 * L.C1 * KK;
    L.fc = L.b2 + L.C2;
    const int64_t B = L.B;
    L.split1 = conv_split_fits({L.C0, L.C1, L.H, L.W, L.KS, L.B}, workers, true, L.wg1);
    L.split2 = conv_split_fits({L.C1, L.C2, L.H2, L.W2, L.KS, L.B}, workers, false, L.wg2);
    L.first = (L.KS == 3 || L.KS == 5) && convsplit::first_plan({L.C0, L.C1, L.H, L.W, L.KS, L.B}, workers, L.fp);
    int64_t o = 0;
    auto take = [&](int64_t n) { const int64_t at = o; o += (n + 63) / 64 * 64; return at; };
    L.z1 = take(L.first && L.split1 ? 0 : B * L.C1 * L.H * L.W);
    L.p1 = take(B * L.C1 * L.H2 * L.W2);
    L.z2 = take(L.split2 ? 0 : B * L.C2 * L.H2 * L.W2);
    L.p2 = take(B * L.flat);
    L.dp2 = take(B * L.flat);
    L.dz2 = take(L.split2 ? 0 : B * L.C2 * L.H2 * L.W2);
    L.dp1 = take(B * L.C1 * L.H2 * L.W2);
    L.dz1 = take(L.split1 ? 0 : B * L.C1 * L.H * L.W);
    L.fc_act = take(dbw_fc_scratch_per_worker(2, L.fc_dims, L.B));
    // split the long pixel reductions of the weight gradients so that the grid fills the chip
    auto pick = [&](int64_t K) { int s = 1; while (s < 32 && K / (s * 2) >= 1024) s *= 2; return s; };
    L.first_wgrad = L.split1 && convsplit::first_wgrad_plan({L.C0, L.C1, L.H, L.W, L.KS, L.B}, workers, L.fw);
    L.splits1 = L.first_wgrad ? L.fw.splits : (L.split1 ? L.wg1.splits : pick(B * L.H * L.W));
    L.splits2 = L.split2 ? L.wg2.splits : pick(B * L.H2 * L.W2);
    L.part1 = take(L.splits1 * L.C1 * L.C0 * KK);
    L.part2 = take(L.splits2 * L.C2 * L.C1 * KK);
    L.filt_fwd = take(L.split2 ? convsplit::filter_floats(L.C1, L.C2, L.KS) : 0);
    L.filt_bwd = take(L.split2 ? convsplit::filter_floats(L.C2, L.C1, L.KS) : 0);
    L.code1 = take((B * L.C1 * L.H2 * L.W2 + 3) / 4);     // one byte per pooled element
    L.code2 = take((B * L.flat + 3) / 4);
    // The workers' blocks start 32 KB apart or a multiple of that.  What lies between was measured on 3 x 32 x 32 images, 64 workers: a
    // block of 6 MB + 14, 15 or 18 KB makes the dense layer's weight gradient 133 to 147 us and the head 41 to 43, multiples of 16 KB (and
    // 65 and 528 KB) 112 to 120 and 35 to 39, whole megabytes too.  Both builds in turn in two processes, without and with the spacing:
    // the round 1646 / 1614 and 1633 / 1615 us; nineteen other networks, this one with 24 or 31 samples or 32 or 48 workers among them,
    // within 0.5 %.  Why these distances and not others was not found.
    L.total = (o + 8191) / 8192 * 8192;
    return L;
}

// 32 x 128 tiles when the GEMM has at most 32 rows (output channels), else 64 x 64
template <class LA, class LB, class EP>
hipError_t conv_gemm(const LA &A, const LB &B, const EP &E, int M, int N, int K, int batch, hipStream_t s,
                     int splits = 1)
{
    if (M <= 32) return bgemm::launch<32>(A, B, E, M, N, K, batch, s, splits);
    return bgemm::launch<64>(A, B, E, M, N, K, batch, s, splits);
}

template <bool POOL, bool EXPAND>
int launch_split_forward(const convsplit::FwdArgs &a, int workers, hipStream_t s)
{
    const int spg = convsplit::samples_per_group(a.s), t = a.s.H * a.s.W / 4;
    const int xt = spg > 1 ? 1 : (t + convsplit::WINDOWS - 1) / convsplit::WINDOWS, mbt = convsplit::row_blocks(a.s.Cout);
    const int MB = convsplit::forward_blocks(a.s.Cout);
    const dim3 grid((a.s.B + spg - 1) / spg * xt, workers, MB == 2 ? mbt / 2 : 1);
    const size_t lds = convsplit::forward_lds(a.s, MB);
    if (MB == 0)
        hipLaunchKernelGGL((convsplit::forward_kernel<0, POOL, EXPAND>), grid, dim3(convsplit::THREADS), lds, s, a);
    else if (MB == 1)
        hipLaunchKernelGGL((convsplit::forward_kernel<1, POOL, EXPAND>), grid, dim3(convsplit::THREADS), lds, s, a);
    else
        hipLaunchKernelGGL((convsplit::forward_kernel<2, POOL, EXPAND>), grid, dim3(convsplit::THREADS), lds, s, a);
    DBW_HIP(hipGetLastError());
    return DBW_OK;
}

int launch_split_wgrad(const convsplit::WgradArgs &a, int workers, hipStream_t s)
{
    const dim3 grid((a.s.B + a.p.sb - 1) / a.p.sb, workers, a.p.groups), block(64 * a.p.waves);
    if (a.s.KS == 3) hipLaunchKernelGGL((convsplit::wgrad_kernel<3, 4>), grid, block, a.p.lds, s, a);
    else if (a.p.paired) hipLaunchKernelGGL((convsplit::wgrad_kernel<5, 4>), grid, block, a.p.lds, s, a);
    else hipLaunchKernelGGL((convsplit::wgrad_kernel<5, 3>), grid, block, a.p.lds, s, a);
    DBW_HIP(hipGetLastError());
    return DBW_OK;
}

template <int KS, int MB, int NB>
int launch_first_wgrad_blocks(const convsplit::FirstWgradArgs &a, int workers, hipStream_t s)
{
    const dim3 grid(a.p.splits, workers, (a.s.Cout + 16 * MB - 1) / (16 * MB));
    hipLaunchKernelGGL((convsplit::first_wgrad_kernel<KS, MB, NB>), grid, dim3(convsplit::THREADS), a.p.lds, s, a);
    DBW_HIP(hipGetLastError());
    return DBW_OK;
}

// Taps of 3 x 3 filters: 9, 18, 27, 36, 45, 54, 63, 72 in one to five blocks of sixteen (the
// last two with one block of output channels only); of 5 x 5: 25, 50, 75 in two, four and five.
int launch_first_wgrad(const convsplit::FirstWgradArgs &a, int workers, hipStream_t s)
{
    auto rows = [&](auto one, auto two) { return a.p.mb == 1 ? one(a, workers, s) : two(a, workers, s); };
    if (a.s.KS == 3) switch (a.p.nb) {
        case 1: return rows(launch_first_wgrad_blocks<3, 1, 1>, launch_first_wgrad_blocks<3, 2, 1>);
        case 2: return rows(launch_first_wgrad_blocks<3, 1, 2>, launch_first_wgrad_blocks<3, 2, 2>);
        case 3: return rows(launch_first_wgrad_blocks<3, 1, 3>, launch_first_wgrad_blocks<3, 2, 3>);
        case 4: return launch_first_wgrad_blocks<3, 1, 4>(a, workers, s);
        default: return launch_first_wgrad_blocks<3, 1, 5>(a, workers, s);
    }
    switch (a.p.nb) {
    case 2: return rows(launch_first_wgrad_blocks<5, 1, 2>, launch_first_wgrad_blocks<5, 2, 2>);
    case 4: return rows(launch_first_wgrad_blocks<5, 1, 4>, launch_first_wgrad_blocks<5, 2, 4>);
    default: return rows(launch_first_wgrad_blocks<5, 1, 5>, launch_first_wgrad_blocks<5, 2, 5>);
    }
}

template <int KS_>
int launch_grad_cnn(dbw_ctx *c, const float *params, const float *bx, const int32_t *by, float *grads,
                    float *loss, hipStream_t s)
{
    const cnn_layout L = make_layout(c->model, c->N);
    const int N = c->N, B = L.B, KK = L.KS * L.KS;
    float *A = c->act;
    const int64_t ws = L.total, ld = c->ld;
    const int64_t xstride = (int64_t)B * L.C0 * L.H * L.W;
    const ConvShape s1{L.C0, L.C1, L.H, L.W, L.KS, L.KS / 2}, s2{L.C1, L.C2, L.H2, L.W2, L.KS, L.KS / 2};
    const int pix1 = B * L.H * L.W, pix2 = B * L.H2 * L.W2;
    auto blocks = [](int64_t n) { return (unsigned)((n + 255) / 256); };
    uint8_t *code1 = (uint8_t *)(A + L.code1), *code2 = (uint8_t *)(A + L.code2);
    const int64_t cs = ws * 4;                         // worker stride of the code maps in bytes
    if (L.first && L.split1) {   // convolution + ReLU + pooling in one kernel
        dbw_timer tm(c, "conv1_forward", s);
        convsplit::FwdArgs g{};
        g.s = {L.C0, L.C1, L.H, L.W, L.KS, B};
        g.in = bx; g.in_stride = xstride;
        g.wgt = params + L.w1; g.wgt_stride = ld;
        g.bias = params + L.b1; g.bias_stride = ld;
        g.out = A + L.p1; g.out_stride = ws;
        g.code = code1; g.code_stride = cs;
        const int per = L.fp.spg * L.fp.iters;
        const dim3 grid((B + per - 1) / per, N, (L.C1 + 31) / 32);
        if (L.KS == 3) hipLaunchKernelGGL(convsplit::first_kernel<3>, grid, dim3(convsplit::THREADS), L.fp.lds, s, g, L.fp);
        else hipLaunchKernelGGL(convsplit::first_kernel<5>, grid, dim3(convsplit::THREADS), L.fp.lds, s, g, L.fp);
        DBW_HIP(hipGetLastError());
    } else {
        {
            dbw_timer tm(c, "conv1_forward", s);
            DBW_HIP(conv_gemm(Dense<true>{params + L.w1, L.C0 * KK, ld}, PatchRC<KS_>{bx, xstride, s1},
                              ChannelPixelOut{A + L.z1, ws, L.C1, L.H * L.W, params + L.b1, ld}, L.C1, pix1,
                              L.C0 * KK, N, s));
        }
        dbw_timer tm(c, "relu_pool_fwd_kernel", s);
        hipLaunchKernelGGL(relu_pool_fwd_kernel, dim3(blocks((int64_t)B * L.C1 * L.H2 * L.W2), N), dim3(256), 0, s,
                           A + L.z1, ws, A + L.p1, ws, B * L.C1, L.H, L.W, code1, cs);
        DBW_HIP(hipGetLastError());
    }
    const convsplit::Shape c2{L.C1, L.C2, L.H2, L.W2, L.KS, B}, c2back{L.C2, L.C1, L.H2, L.W2, L.KS, B};
    convsplit::FwdArgs f{};
    if (L.split2) {
        {
            dbw_timer tm(c, "conv2_prepare", s);
            const dim3 grid(convsplit::prepare_blocks(L.C1, L.C2) + convsplit::prepare_blocks(L.C2, L.C1), N);
            auto *fwd = (split_bf16::u32x4 *)(A + L.filt_fwd), *bwd = (split_bf16::u32x4 *)(A + L.filt_bwd);
            if (L.KS == 3)
                hipLaunchKernelGGL(convsplit::prepare_kernel<9>, grid, dim3(convsplit::PREPARE_THREADS), 0, s, params + L.w2, ld, fwd, bwd, ws / 4, L.C1, L.C2);
            else
                hipLaunchKernelGGL(convsplit::prepare_kernel<25>, grid, dim3(convsplit::PREPARE_THREADS), 0, s, params + L.w2, ld, fwd, bwd, ws / 4, L.C1, L.C2);
            DBW_HIP(hipGetLastError());
        }
        dbw_timer tm(c, "conv2_forward", s);
        f.s = c2;
        f.in = A + L.p1;
        f.in_stride = ws;
        f.filters = (const split_bf16::u32x4 *)(A + L.filt_fwd);
        f.filters_stride = ws / 4;
        f.bias = params + L.b2;
        f.bias_stride = ld;
        f.out = A + L.p2;
        f.out_stride = ws;
        f.code = code2;
        f.code_stride = cs;
        const int rc = launch_split_forward<true, false>(f, N, s);
        if (rc != DBW_OK) return rc;
    } else {
        {
            dbw_timer tm(c, "conv2_forward", s);
            DBW_HIP(conv_gemm(Dense<true>{params + L.w2, L.C1 * KK, ld}, PatchRC<KS_>{A + L.p1, ws, s2},
                              ChannelPixelOut{A + L.z2, ws, L.C2, L.H2 * L.W2, params + L.b2, ld}, L.C2, pix2,
                              L.C1 * KK, N, s));
        }
        dbw_timer tm(c, "relu_pool_fwd_kernel", s);
        hipLaunchKernelGGL(relu_pool_fwd_kernel, dim3(blocks((int64_t)B * L.flat), N), dim3(256), 0, s, A + L.z2, ws,
                           A + L.p2, ws, B * L.C2, L.H2, L.W2, (uint8_t *)nullptr, (int64_t)0);
        DBW_HIP(hipGetLastError());
    }
    {   // fully connected head, forward and backward, down to the gradient of the pooled features
        dbw_fc_args a{};
        a.L = 2;
        a.B = B;
        a.dims = L.fc_dims;
        a.params = params;
        a.grads = grads;
        a.param_off = L.fc;
        a.in = A + L.p2;
        a.in_ld = L.flat;
        a.in_stride = ws;
        a.act = A + L.fc_act;
        a.act_stride = ws;
        a.din = A + L.dp2;
        a.din_ld = L.flat;
        a.din_stride = ws;
        a.y = by;
        a.loss = loss;
        const int rc = dbw_fc_forward_backward(c, a, s);
        if (rc != DBW_OK) return rc;
    }
    // with the window codes the un-pooled delta maps are never materialised: their consumers
    // expand the pooled gradients and the codes on the fly
    if (L.split2) {   // conv2 weight gradient (partial results, then summed in split order)
        dbw_timer tm(c, "conv2_wgrad", s);
        const int rc = launch_split_wgrad({c2, L.wg2, A + L.p1, ws, A + L.dp2, ws, code2, cs, A + L.part2, ws}, N, s);
        if (rc != DBW_OK) return rc;
    } else {
        {
            dbw_timer tm(c, "relu_pool_bwd_kernel", s);
            hipLaunchKernelGGL(relu_pool_bwd_kernel, dim3(blocks((int64_t)B * L.flat), N), dim3(256), 0, s, A + L.z2, ws,
                               A + L.dp2, ws, A + L.dz2, B * L.C2, L.H2, L.W2);
            DBW_HIP(hipGetLastError());
        }
        dbw_timer tm(c, "conv2_wgrad", s);
        DBW_HIP(conv_gemm(DeltaKC{A + L.dz2, ws, L.C2, L.H2 * L.W2}, PatchKC<KS_>{A + L.p1, ws, s2},
                              PartialOut{A + L.part2, ws, L.C2, L.C1 * KK}, L.C2, L.C1 * KK, pix2, N, s,
                              L.splits2));
    }
    if (L.split2) {   // conv2 data gradient = forward convolution of the deltas with flipped filters
        dbw_timer tm(c, "conv2_dgrad", s);
        f.s = c2back;
        f.in = A + L.dp2;
        f.in_code = code2;
        f.in_code_stride = cs;
        f.filters = (const split_bf16::u32x4 *)(A + L.filt_bwd);
        f.bias = nullptr;
        f.out = A + L.dp1;
        f.code = nullptr;
        const int rc = launch_split_forward<false, true>(f, N, s);
        if (rc != DBW_OK) return rc;
    } else {
        {
            dbw_timer tm(c, "channel_sum_kernel", s);
            hipLaunchKernelGGL(channel_sum_kernel, dim3(L.C2, N), dim3(256), 0, s, A + L.dz2, ws, B, L.C2, L.H2 * L.W2,
                               grads + L.b2, ld);
            DBW_HIP(hipGetLastError());
        }
        dbw_timer tm(c, "conv2_dgrad", s);
        DBW_HIP(conv_gemm(FilterT<KS_>{params + L.w2, ld, L.C1, KK}, DeltaShiftRC<KS_>{A + L.dz2, ws, s2},
                              ChannelPixelOut{A + L.dp1, ws, L.C1, L.H2 * L.W2, nullptr, 0}, L.C1, pix2, L.C2 * KK, N,
                              s));
    }
    if (L.first_wgrad) {
        dbw_timer tm(c, "conv1_wgrad", s);
        const int rc = launch_first_wgrad({{L.C0, L.C1, L.H, L.W, L.KS, B}, L.fw, bx, xstride, A + L.dp1, ws, code1, cs, A + L.part1, ws}, N, s);
        if (rc != DBW_OK) return rc;
    } else if (L.split1) {
        dbw_timer tm(c, "conv1_wgrad", s);
        const int rc = launch_split_wgrad({{L.C0, L.C1, L.H, L.W, L.KS, B}, L.wg1, bx, xstride, A + L.dp1, ws, code1, cs, A + L.part1, ws}, N, s);
        if (rc != DBW_OK) return rc;
    } else {
        {
            dbw_timer tm(c, "relu_pool_bwd_kernel", s);
            hipLaunchKernelGGL(relu_pool_bwd_kernel, dim3(blocks((int64_t)B * L.C1 * L.H2 * L.W2), N), dim3(256), 0, s,
                               A + L.z1, ws, A + L.dp1, ws, A + L.dz1, B * L.C1, L.H, L.W);
            DBW_HIP(hipGetLastError());
        }
        {
            dbw_timer tm(c, "conv1_wgrad", s);
            DBW_HIP(conv_gemm(DeltaKC{A + L.dz1, ws, L.C1, L.H * L.W}, PatchKC<KS_>{bx, xstride, s1},
                              PartialOut{A + L.part1, ws, L.C1, L.C0 * KK}, L.C1, L.C0 * KK, pix1, N, s,
                              L.splits1));
        }
        dbw_timer tm(c, "channel_sum_kernel", s);
        hipLaunchKernelGGL(channel_sum_kernel, dim3(L.C1, N), dim3(256), 0, s, A + L.dz1, ws, B, L.C1, L.H * L.W,
                           grads + L.b1, ld);
        DBW_HIP(hipGetLastError());
    }
    const FinishLayer f1{A + L.part1, L.splits1, L.C1 * L.C0 * KK, grads + L.w1, grads + L.b1, L.split1 ? code1 : nullptr, A + L.dp1,
                         L.C1, L.H2 * L.W2};
    const FinishLayer f2{A + L.part2, L.splits2, L.C2 * L.C1 * KK, grads + L.w2, grads + L.b2, L.split2 ? code2 : nullptr, A + L.dp2,
                         L.C2, L.H4 * L.W4};
    dbw_timer tm(c, "conv_finish_kernel", s);
    hipLaunchKernelGGL(finish_kernel, dim3(f1.blocks() + f2.blocks(), N), dim3(256), 0, s, f1, f2, ws, cs, ld, B);
    DBW_HIP(hipGetLastError());
    return DBW_OK;
}

}  // namespace

size_t dbw_cnn_scratch_floats(const dbw_ctx *c) { return (size_t)make_layout(c->model, c->N).total * c->N; }

int dbw_cnn_prepare()
{
    const void *kernels[] = {(const void *)convsplit::forward_kernel<0, true, false>, (const void *)convsplit::forward_kernel<0, false, true>,
                             (const void *)convsplit::forward_kernel<1, true, false>, (const void *)convsplit::forward_kernel<2, true, false>,
                             (const void *)convsplit::forward_kernel<1, false, true>, (const void *)convsplit::forward_kernel<2, false, true>,
                             (const void *)convsplit::first_kernel<3>, (const void *)convsplit::first_kernel<5>,
                             (const void *)convsplit::wgrad_kernel<3, 4>, (const void *)convsplit::wgrad_kernel<5, 3>,
                             (const void *)convsplit::wgrad_kernel<5, 4>};
    for (const void *k : kernels) DBW_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    return DBW_OK;
}

int dbw_launch_grad_cnn(dbw_ctx *c, const float *params, const float *bx, const int32_t *by, float *grads,
                        float *loss, hipStream_t s)
{
    switch (c->model.dims[5]) {
    case 3: return launch_grad_cnn<3>(c, params, bx, by, grads, loss, s);
    case 5: return launch_grad_cnn<5>(c, params, bx, by, grads, loss, s);
    default: return launch_grad_cnn<0>(c, params, bx, by, grads, loss, s);
    }
}
