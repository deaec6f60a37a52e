// Mini-batch gradients of fully connected models for all workers at once (Section 2.1,
// stochastic gradient of the local loss; cross-entropy as in Section 5).  Worker w uses
// row w of the parameter matrix and its own batch: every GEMM below is batched over
// workers with per-worker operands.
//
// Parameter row layout: per layer l, W_l [out][in] then b_l [out].
// Scratch per worker: activations a_1..a_L ([B][dims[l]], a_L = logits) followed by the
// deltas dz_1..dz_L of the same shapes.
#include <algorithm>

#include "bgemm.h"
#include "fc_batch32.h"
#include "fc_head.h"
#include "mlp_chain.h"
#include "mlp_thin.h"
#include "mlp_wgrad.h"
#include "dbw_internal.h"

namespace {

using bgemm::Dense;
using bgemm::Epilogue;

// Softmax, mean loss over the batch and its gradient with respect to the logits; sixteen lanes per sample, which share its
// classes; grid = (chunks, workers) with 256 samples per workgroup.  Cross-entropy:
// dz = (p - onehot(y)) / B.  MSE on the softmax outputs (Appendix B, 2NN): f = sum_c (p_c - o_c)^2,
// dz_k = 2 p_k ((p_k - o_k) - sum_c p_c (p_c - o_c)) / B.
// The loss of a worker is the sum of its workgroups' partial sums: each writes its own to
// loss_part[worker][chunk] and takes a ticket; the last one to arrive adds them in chunk order (so
// the result does not depend on the order of arrival) and puts the ticket counter back to zero.
// A thread per sample walked over the classes alone, in one wavefront or two per worker: 20 workers x 101 samples, 26 classes, 13.3 us
// of a round that took 120.5 and takes 113.6 so; 256-40 on 20 x 1 024 samples 70 -> 56, 784-33 on 6 x 32 40 -> 30.
constexpr int LOSS_THREADS = 1024, LOSS_LANES = 16;
template <class F>
__device__ __forceinline__ float loss_lanes(float v, F op)      // over the lanes of a sample
{
#pragma unroll
    for (int o = 1; o < LOSS_LANES; o <<= 1) v = op(v, __shfl_xor(v, o, LOSS_LANES));
    return v;
}
template <int LOSS>
__global__ __launch_bounds__(LOSS_THREADS) void softmax_loss_kernel(
    int B, int C, const float *__restrict__ logits, int64_t stride_logits, const int32_t *__restrict__ y,
    float *__restrict__ dz, int64_t stride_dz, float *__restrict__ loss, float *__restrict__ loss_part,
    uint32_t *__restrict__ ticket, int32_t *__restrict__ err)
{
    constexpr int AT_ONCE = LOSS_THREADS / LOSS_LANES;
    __shared__ float red[LOSS_THREADS / 64];
    const int chunk = blockIdx.x, chunks = gridDim.x, w = blockIdx.y, tid = threadIdx.x, l = tid % LOSS_LANES;
    const float *z = logits + w * stride_logits;
    float *d = dz + w * stride_dz;
    const float inv_b = 1.0f / (float)B;
    auto add = [](float a, float b) { return a + b; };
    float part = 0.f;                                   // of this lane's samples; the same in the lanes of a sample
    for (int s0 = chunk * 256; s0 < B; s0 += chunks * 256)
        for (int s = s0 + tid / LOSS_LANES; s < min(B, s0 + 256); s += AT_ONCE) {
            const float *zs = z + (int64_t)s * C;
            float m = -INFINITY;
            for (int c = l; c < C; c += LOSS_LANES) m = fmaxf(m, zs[c]);
            m = loss_lanes(m, [](float a, float b) { return fmaxf(a, b); });
            float sum = 0.f;
            for (int c = l; c < C; c += LOSS_LANES) sum += expf(zs[c] - m);
            sum = loss_lanes(sum, add);
            int label = y[(int64_t)w * B + s];
            if (label < 0 || label >= C) {              // clamped for memory safety, reported by dbw_check
                *err = DBW_ERR_INVALID;
                label = label < 0 ? 0 : C - 1;
            }
            const float inv = 1.0f / sum;
            if (LOSS == DBW_LOSS_XENT) {
                for (int c = l; c < C; c += LOSS_LANES)
                    d[(int64_t)s * C + c] = (expf(zs[c] - m) * inv - (c == label ? 1.f : 0.f)) * inv_b;
                part += logf(sum) + m - zs[label];
            } else {
                float f = 0.f, inner = 0.f;
                for (int c = l; c < C; c += LOSS_LANES) {
                    const float p = expf(zs[c] - m) * inv, e = p - (c == label ? 1.f : 0.f);
                    f += e * e;
                    inner += p * e;
                }
                f = loss_lanes(f, add);
                inner = loss_lanes(inner, add);
                for (int c = l; c < C; c += LOSS_LANES) {
                    const float p = expf(zs[c] - m) * inv, e = p - (c == label ? 1.f : 0.f);
                    d[(int64_t)s * C + c] = 2.f * p * (e - inner) * inv_b;
                }
                part += f;
            }
        }
    if (!loss) return;                                  // uniform: nobody asked for the loss
    part += __shfl_xor(part, 16, 64);                   // the samples of a wavefront, then the wavefronts, in a fixed order
    part += __shfl_xor(part, 32, 64);
    if (tid % 64 == 0) red[tid / 64] = part;
    __syncthreads();
    static_assert(LOSS_THREADS / 64 == LOSS_LANES, "one value for each lane of a group");
    part = loss_lanes(red[l], add);
    if (chunks == 1) {
        if (tid == 0) loss[w] = part * inv_b;
        return;
    }
    if (tid == 0) {
        __hip_atomic_store(&loss_part[w * chunks + chunk], part, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();                                // the partial sum is visible before the ticket is taken
        if (atomicAdd(&ticket[w], 1u) == (uint32_t)(chunks - 1)) {
            __threadfence();
            float sum = 0.f;
            for (int k = 0; k < chunks; ++k)
                sum += __hip_atomic_load(&loss_part[w * chunks + k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            loss[w] = sum * inv_b;
            ticket[w] = 0;                              // ready for the next launch
        }
    }
}

// Bias gradient: db[o] = sum over the batch of dz[s][o], for the layers whose weight gradient has a kernel of its own.
// grid = (ceil(C / 32), workers).
__global__ __launch_bounds__(256) void colsum_kernel(int B, int C, const float *__restrict__ dz, int64_t stride_dz,
                                                     float *__restrict__ db, int64_t stride_db)
{
    __shared__ float part[256];
    bgemm::column_sums<8, 32>(B, C, dz + blockIdx.y * stride_dz, db + blockIdx.y * stride_db, 32 * blockIdx.x, part);
}

// Partial sums of a split-k forward GEMM: part[worker][split][m][n].
struct SplitOut {
    float *part;
    int64_t stride;
    int M, N;
    __device__ __forceinline__ void store(int w, int split, int m, int n, float v) const
    {
        part[w * stride + ((int64_t)split * M + m) * N + n] = v;
    }
};

// C[m][n] = act(sum over splits of part[split][m][n] + bias[n]) (bias may be NULL); grid = (ceil(M N / 256), workers).
__global__ __launch_bounds__(256) void fc_reduce_kernel(const float *__restrict__ part, int64_t pstride, int splits,
                                                        int M, int N, const float *__restrict__ bias,
                                                        int64_t bias_stride, int relu, float *__restrict__ C,
                                                        int64_t ldc, int64_t cstride)
{
    const int w = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
    if (i >= M * N) return;
    const int m = i / N, n = i - m * N;
    float s = 0.f;
    for (int sp = 0; sp < splits; ++sp) s += part[w * pstride + (int64_t)sp * M * N + i];
    if (bias) s += bias[w * bias_stride + n];
    if (relu) s = s > 0.f ? s : 0.f;
    C[w * cstride + (int64_t)m * ldc + n] = s;
}

// A long reduction with few output tiles (e.g. batch 32 x 512 outputs over k = 4096, or any
// small model) leaves most of the chip idle and each workgroup waiting on its own chain of
// loads; split k then, up to MAX_SPLITS ways, keeping at least two k-steps per split.
constexpr int MAX_SPLITS = 16;          // partial-sum slots per output in the scratch block
constexpr int GEMM_MAX_SPLITS = 8;
int forward_splits(int M, int N, int K, int workers)
{
    const int64_t tiles = (int64_t)((M + 63) / 64) * ((N + 63) / 64) * workers;
    int splits = 1;
    while (splits < GEMM_MAX_SPLITS && tiles * splits < 640 && K / (splits * 2) >= 2 * bgemm::BK) splits *= 2;
    return splits;
}

// The streaming kernels for a batch of exactly 32 apply to a layer in -> out when the shapes
// divide evenly and every operand row starts on a 16-byte boundary.
bool batch32_layer(int B, int in, int out, int64_t ld_params, int64_t w_off, const float *params, const float *grads)
{
    return B == 32 && in % 512 == 0 && out % 32 == 0 && ld_params % 4 == 0 && w_off % 4 == 0 &&
           fc32::aligned16(params) && fc32::aligned16(grads);
}

// LDS that a workgroup of the head may take.  More than 16 classes in several chunks: two workgroups to a compute unit, or the layer's own
// kernels are faster (497-18 on 19 workers x 1 024 samples 66 us, with chunks that fill a unit's LDS 72; 256-25 on 6 x 1 024 39 and 26).
size_t head_lds_limit(int C, int B) { return C > fchead::TILE_C && B > 64 ? 80 * 1024 : fchead::LDS_LIMIT; }
// The shapes that the head takes for some number of workers, and the chunks that it then has at most: only these need memory for its
// partial sums, which is as much as a chunk's W for every 16 samples.
bool head_fits(int H, int C, int B)
{
    return C <= fchead::MAX_C && fchead::lds_bytes(H, C, 16) <= head_lds_limit(C, B) && (B + fchead::MAX_S - 1) / fchead::MAX_S <= fchead::MAX_CHUNKS;
}
int head_max_chunks(int B) { return std::min((B + 15) / 16, fchead::MAX_CHUNKS); }

// The fused classifier head (fc_head.h) takes the last layer when it is narrow enough.
struct HeadPlan {
    bool use;
    int chunks, S;
    int64_t part;          // floats of partial sums per worker
};
HeadPlan head_plan(int L, const int32_t *dims, int B, int workers)
{
    const int H = dims[L - 1], C = dims[L];
    HeadPlan hp{false, 0, 0, 0};
    if (!head_fits(H, C, B)) return hp;
    auto fits = [&](int S) { return fchead::lds_bytes(H, C, S) <= head_lds_limit(C, B); };
    // Longer batches: W is staged, and a partial sum of dW written and read, once per chunk, so as many samples to a chunk as leave work for the
    // chip.  Rounds, chunks of 16 / 32: 784-10 on 6 workers x 1 024 (192 chunks of 32) 31.2 / 24.2 us, on 30 x 150 30.7 / 23.5, 256-10 on 6 x
    // 1 024 19.2 / 17.0, 4 x 1 024 (128) 17.1 / 17.1, 784-10 on 20 x 100 (80) 19.6 / 20.2, behind other
    // layers 133-111-42-10 on 16 x 256 (128) 65.5 / 67.5, 300-100-10 on 40 x 100 (160) 36.9 / 36.0; of 32 / 64, two workgroups to a compute unit:
    // 128-10 on 64 x 1 024 39.7 / 31.7, 200-10 on 60 x 300 23.1 / 21.8.
    int S;
    const int whole = B <= 16 ? 16 : (B <= 32 ? 32 : 64);
    if (B <= 64 && fits(whole))
        S = whole;                                   // one chunk per worker: no partial sums at all
    else if (fchead::lds_bytes(H, C, 64) <= 80 * 1024 && (int64_t)((B + 63) / 64) * workers >= 256)
        S = 64;
    else
        S = fits(32) && (int64_t)((B + 31) / 32) * workers >= (L == 1 ? 128 : 160) ? 32 : 16;
    const int chunks = (B + S - 1) / S;
    if (chunks > fchead::MAX_CHUNKS) return hp;
    // More than 16 classes in chunks of a short batch that does not fit whole, one workgroup to a compute unit: the layer's own kernels from half of
    // the chip on (978-17 on 61 workers x 64 samples 42.4 / 30.5 us, 784-20 on 44 x 48 31.4 / 25.7, 784-26 on 32 x 64 30.5 / 32.3).  Behind other
    // layers the head saves them more (400-600-20 on 64 x 33 106.5 / 113.1).
    if (L == 1 && C > fchead::TILE_C && chunks > 1 && B <= 64 && fchead::lds_bytes(H, C, S) > 80 * 1024 && (int64_t)chunks * workers > 128) return hp;
    hp.use = true;
    hp.chunks = chunks;
    hp.S = S;
    hp.part = chunks > 1 ? (int64_t)chunks * fchead::partial_floats(H, C, L > 1) : 0;
    return hp;
}

// The whole chain of layers in one launch (mlp_chain.h) applies to equal hidden widths of 128, 256 or 512, an
// input width that divides by 16, at most 16 classes, and operands on 16-byte boundaries.  S = samples per
// workgroup: the one that needs the least time when every CU takes one workgroup at a time (ties: the larger).
struct ChainPlan {
    bool use;
    int S, chunks;
    size_t lds;
};
ChainPlan chain_plan(int L, const int32_t *dims, int B, int workers, int grad_path)
{
    ChainPlan cp{false, 0, 0, 0};
    if (grad_path == DBW_GRAD_LAYERS || L < 2 || L > mlpchain::MAX_L || dims[L] > fchead::TILE_C) return cp;
    const int H = dims[1];
    if (H != 128 && H != 256 && H != 512) return cp;
    for (int l = 2; l < L; ++l)
        if (dims[l] != H) return cp;
    if (dims[0] % 16 != 0 || dims[0] <= 0) return cp;
    int64_t best = 0;
    for (int S = 64; S >= 16; S -= 16) {
        if (mlpchain::lds_bytes(dims[0], H, dims[L], S, L) > fchead::LDS_LIMIT) continue;
        const int chunks = (B + S - 1) / S;
        if (chunks > fchead::MAX_CHUNKS) continue;
        const int64_t cost = ((int64_t)chunks * workers + 255) / 256 * S;
        if (cp.S == 0 || cost < best) {
            best = cost;
            cp.S = S;
            cp.chunks = chunks;
        }
    }
    if (cp.S == 0) return cp;
    // worth it when the workgroups keep at least half of the chip busy; otherwise the layered path, which
    // splits its products over all CUs, wins
    if (grad_path != DBW_GRAD_CHAIN && (int64_t)B * workers * 2 < best * 256) return cp;
    cp.lds = mlpchain::lds_bytes(dims[0], H, dims[L], cp.S, L);
    cp.use = true;
    return cp;
}

using mlpthin::ThinPlan;
using mlpthin::thin_forward;
using mlpthin::thin_plan;

template <bool BACK>
hipError_t launch_thin(const ThinPlan &tp, const mlpthin::FwdArgs &f, hipStream_t s)
{
    const int tiles = (f.N + 16 * tp.CB - 1) / (16 * tp.CB) * f.workers;
    const dim3 grid((tiles + mlpthin::XCDS - 1) / mlpthin::XCDS * mlpthin::XCDS, tp.blocks, tp.splits), block(mlpthin::FWD_THREADS);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, s, f); };
    switch (8 * tp.RB + tp.CB) {
    case 8 * 1 + 1: go(mlpthin::forward_kernel<1, 1, BACK>); break;
    case 8 * 2 + 1: go(mlpthin::forward_kernel<2, 1, BACK>); break;
    case 8 * 3 + 1: go(mlpthin::forward_kernel<3, 1, BACK>); break;
    case 8 * 4 + 1: go(mlpthin::forward_kernel<4, 1, BACK>); break;
    case 8 * 1 + 2: go(mlpthin::forward_kernel<1, 2, BACK>); break;
    case 8 * 2 + 2: go(mlpthin::forward_kernel<2, 2, BACK>); break;
    case 8 * 3 + 2: go(mlpthin::forward_kernel<3, 2, BACK>); break;
    default: go(mlpthin::forward_kernel<4, 2, BACK>); break;
    }
    return hipGetLastError();
}

// Weight and bias gradients of layers 1 .. layers in one launch (mlp_wgrad.h), from the deltas and activations
// in the workers' scratch blocks; extra workgroups add the head's per-chunk sums when it has any.
struct WgradPlan {
    int layers;                 // dW_l and db_l for l = 1 .. layers
    bool last_db;               // false: somebody else (the head) computes db of layer `layers`
    const int64_t *a_off, *dz_off, *w_off;
    int64_t w_end;              // end of b_layers in the parameter row
    int64_t per, split_floats;
    bool chain;                 // the chain kernel has run
};
// The tiles of that launch: 64 x 64 when they alone give every CU two workgroups, else 64 x 32; if that still leaves CUs idle, the
// batch is split as well (partial tiles to scratch, one more launch to add them).  begin, if not null: the first tile of every layer.
// Batches of up to 64 samples take mlp_thin.h.  Longer ones, up to 255, while there is little to multiply (tiles x samples): one launch
// instead of two or three, and the average on the way, but the fp32 instruction instead of six of bf16; less of it where there are layers
// between, whose data gradient bgemm::backward_kernel computes in the same launch.  Rounds, bgemm.h / mlp_thin.h: 784-500-10 on 32 workers
// x 128 (0.9 M) 139 / 124 us, 784-200-10 on 32 x 200 (0.6 M) 116 / 97, 64 x 255 (3.4 M) 381 / 468; 300-300-300-10 on 16 x 200 (0.5 M) 112 / 92,
// 63 x 200 (1.3 M) 298 / 314.  Only where the forward products are mlp_thin.h's as well, whose rounding makes up for that of these sums: dW of
// 784-300 on 32 x 200, whose forward product is bgemm.h's, 2.89e-7 with bgemm.h, 2.97e-7 here; 784-200 on 32 x 128 1.84, 1.53.  (784-500-10 on 32 x
// 200 would be 196 / 185 us.)  Behind the chain (whose alternative, mlp_wgrad.h, shares a tile among four wavefronts) not with fewer tiles than
// SIMDs: 784-128-10 on 16 x 200 43.8 / 44.8, 784-512-10 on 32 x 128 130 / 118.
constexpr int64_t THIN_WORK = 1400000, THIN_WORK_DEEP = 700000;
struct WgradTiles {
    bool thin;                  // one wavefront per 32 x 64 tile, no split (mlp_thin.h)
    int tn, tiles;
};
WgradTiles wgrad_tiles(int layers, const int32_t *dims, int B, int N, bool chain, int *begin)
{
    auto count = [&](int tm, int tn, int *begin) {
        int t = 0;
        for (int l = 1; l <= layers; ++l) {
            if (begin) begin[l] = t;
            t += ((dims[l] + tm - 1) / tm) * ((dims[l - 1] + tn - 1) / tn);
        }
        if (begin) begin[layers + 1] = t;
        return t;
    };
    WgradTiles r{};
    const int64_t tiles = (int64_t)count(mlpthin::WG_TM, mlpthin::WG_TN, nullptr) * N;
    r.thin = B <= 64 || (B <= mlpthin::MAX_B && tiles * B <= (layers == 1 ? THIN_WORK : THIN_WORK_DEEP) && (!chain || tiles >= 1024));
    for (int l = 1; l <= layers && r.thin && !chain; ++l) r.thin = thin_forward(B, thin_plan(B, dims[l - 1], dims[l], N, false));
    r.tn = !r.thin && (int64_t)count(64, 64, nullptr) * N >= 512 ? 64 : 32;
    r.tiles = r.thin ? count(mlpthin::WG_TM, mlpthin::WG_TN, begin) : count(64, r.tn, begin);
    return r;
}

int launch_grouped_wgrad(dbw_ctx *c, const dbw_fc_args &a, const WgradPlan &wp, const fchead::Args &h, int head_chunks,
                         hipStream_t s)
{
    const int B = a.B, N = c->N;
    const int32_t *dims = a.dims;
    const int64_t wstride = a.act_stride;
    mlpwgrad::Args q{};
    q.B = B; q.layers = wp.layers; q.workers = N;
    const WgradTiles wt = wgrad_tiles(wp.layers, dims, B, N, wp.chain, q.tile_begin);
    const bool thin = wt.thin;
    const int tn = wt.tn, tiles = wt.tiles;
    for (int l = 1; l <= wp.layers; ++l) {
        q.n_rows[l] = dims[l];
        q.n_cols[l] = dims[l - 1];
        q.want_db[l] = l < wp.layers || wp.last_db;
        q.dz_off[l] = wp.dz_off[l];
        q.a[l] = l == 1 ? a.in : a.act + wp.a_off[l - 1];
        q.a_ld[l] = l == 1 ? a.in_ld : dims[l - 1];
        q.a_stride[l] = l == 1 ? a.in_stride : wstride;
        q.w_off[l] = wp.w_off[l];
    }
    q.w_off[wp.layers + 1] = wp.w_end;
    q.dz = a.act; q.dz_stride = wstride;
    q.grads = a.averaged ? a.out : a.grads; q.g_stride = c->ld;
    if (a.averaged) q.avg = a.avg;
    q.part = a.act + 2 * wp.per; q.part_stride = wstride;
    const int64_t len = wp.w_end - wp.w_off[1];
    int splits = (int)std::min<int64_t>(8, std::max<int64_t>(1, 512 / ((int64_t)tiles * N)));
    splits = std::min(splits, (B + 63) / 64);
    splits = (int)std::min<int64_t>(splits, std::max<int64_t>(1, wp.split_floats / len));
    if (thin) splits = 1;
    q.splits = splits;
    q.kper = ((B + splits - 1) / splits + 15) / 16 * 16;
    const int head_blocks = head_chunks > 1 ? (int)((fchead::partial_floats(h.H, h.C, h.bprev_off >= 0) + 255) / 256) : 0;
    {
        dbw_timer tm(c, "mlp_wgrad_kernel", s);
        auto whole_xcds = [](int n) { return (n + mlpwgrad::XCDS - 1) / mlpwgrad::XCDS * mlpwgrad::XCDS; };
        const int tile_wgs = thin ? (tiles * N + mlpwgrad::WAVES - 1) / mlpwgrad::WAVES : tiles * N * splits;
        const dim3 grid(whole_xcds(head_blocks * N) + whole_xcds(tile_wgs));
        auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(mlpwgrad::THREADS), 0, s, q, h, head_chunks, head_blocks); };
        if (thin && B <= 16) go(mlpthin::wgrad_kernel<4, false>);
        else if (thin && B <= 32) go(mlpthin::wgrad_kernel<8, false>);
        else if (thin && B <= 64) go(mlpthin::wgrad_kernel<16, false>);
        else if (thin && (B + 35) / 36 * 9 <= (B + 31) / 32 * 8) go(mlpthin::wgrad_kernel<9, true>);      // the less padding
        else if (thin) go(mlpthin::wgrad_kernel<8, true>);
        else if (tn == 64) go(mlpwgrad::kernel<4>);
        else go(mlpwgrad::kernel<2>);
        DBW_HIP(hipGetLastError());
    }
    if (splits > 1) {
        dbw_timer tm(c, "mlp_reduce_kernel", s);
        hipLaunchKernelGGL(mlpwgrad::reduce_kernel, dim3((unsigned)((len / 4 + 255) / 256), N), dim3(256), 0, s, q);
        DBW_HIP(hipGetLastError());
    }
    return DBW_OK;
}

int64_t act_floats(int L, const int32_t *dims, int B)
{
    int64_t n = 0;
    for (int l = 1; l <= L; ++l) n += (int64_t)B * dims[l];
    return (n + 3) / 4 * 4;          // the deltas and the partial sums behind them keep the 16-byte alignment
}

}  // namespace

int64_t dbw_fc_scratch_per_worker(int L, const int32_t *dims, int B)
{
    int64_t part = 0;
    for (int l = 1; l <= L; ++l) part = std::max<int64_t>(part, (int64_t)MAX_SPLITS * B * dims[l]);
    part = (part + 3) / 4 * 4;
    if (head_fits(dims[L - 1], dims[L], B))      // partial sums of the fused head, at its smallest chunk size, behind the split partials
        part += (int64_t)head_max_chunks(B) * fchead::partial_floats(dims[L - 1], dims[L], L > 1);
    return 2 * act_floats(L, dims, B) + (part + 3) / 4 * 4;
}

bool dbw_fc_chain_shape_ok(int L, const int32_t *dims, int B, int workers)
{
    return chain_plan(L, dims, B, workers, DBW_GRAD_CHAIN).use;
}

// Forward and backward pass of a stack of fully connected layers for all workers.
int dbw_fc_forward_backward(dbw_ctx *c, dbw_fc_args &a, hipStream_t s)
{
    const int L = a.L, B = a.B, N = c->N;
    const int32_t *dims = a.dims;
    const int64_t per = act_floats(L, dims, B), wstride = a.act_stride;
    // offsets inside a worker's scratch block and parameter row
    int64_t a_off[9], dz_off[9], w_off[9], b_off[9];
    int64_t ao = 0, po = a.param_off;
    for (int l = 1; l <= L; ++l) {
        a_off[l] = ao;
        dz_off[l] = per + ao;
        ao += (int64_t)B * dims[l];
        w_off[l] = po;
        b_off[l] = po + (int64_t)dims[l] * dims[l - 1];
        po = b_off[l] + dims[l];
    }
    float *act = a.act;
    const float *params = a.params;
    float *grads = a.grads;

    HeadPlan head = head_plan(L, dims, B, N);
    ChainPlan chain = chain_plan(L, dims, B, N, a.grad_path);
    if (chain.use && !(a.din == nullptr && a.in_ld % 4 == 0 && a.in_stride % 4 == 0 && fc32::aligned16(a.in) &&
                       fc32::aligned16(params) && c->ld % 4 == 0 && a.param_off % 4 == 0 && fc32::aligned16(act) &&
                       wstride % 4 == 0 && per % 4 == 0))
        chain.use = false;
    if (a.grad_path == DBW_GRAD_CHAIN && !chain.use) return DBW_ERR_UNSUPPORTED;
    if (chain.use) {      // the head runs inside the chain, on the chain's chunks
        head.use = true;
        head.S = chain.S;
        head.chunks = chain.chunks;
    }
    const int L_gemm = chain.use ? 0 : (head.use ? L - 1 : L);         // layers that go through the forward GEMM kernels
    // The output of layer L - 1 feeds nothing but the head.  When its forward product is split along k, the
    // head sums the partial products itself (same order, then bias and ReLU) and the reduction launch is saved.
    int head_splits = 0;
    const bool head_can_sum = head.use && L >= 2 && dims[L - 1] % 4 == 0 && b_off[L - 1] % 4 == 0 && c->ld % 4 == 0 &&
                              fc32::aligned16(params) && wstride % 4 == 0 && fc32::aligned16(act) && (2 * per) % 4 == 0;

    // forward: a_l = relu(a_{l-1} W_l^T + b_l), no ReLU on the logits
    for (int l = 1; l <= L_gemm; ++l) {
        Dense<true> A, Bm;
        if (l == 1)
            A = {a.in, a.in_ld, a.in_stride};
        else
            A = {act + a_off[l - 1], dims[l - 1], wstride};
        Bm = {params + w_off[l], dims[l - 1], c->ld};
        if (batch32_layer(B, dims[l - 1], dims[l], c->ld, w_off[l], params, grads) && A.ld % 4 == 0 &&
            A.stride % 4 == 0 && fc32::aligned16(A.p) && wstride % 4 == 0 && a_off[l] % 4 == 0 && fc32::aligned16(act)) {
            int subs = 1;                                // slices of a workgroup: while two workgroups to a compute unit are left
            while (subs < 4 && dims[l - 1] % (2 * subs * fc32::KSLICE) == 0 && (int64_t)dims[l - 1] / (2 * subs * fc32::KSLICE) * N >= 512) subs *= 2;
            const int slices = dims[l - 1] / (subs * fc32::KSLICE), nf = dims[l] / 128;
            if (dims[l] % 128 == 0 && nf <= 4 && slices <= MAX_SPLITS) {      // split along k, inputs read once
                float *part = act + 2 * per;
                {
                    dbw_timer tm(c, subs == 4 ? "fc32_forward_4slices" : subs == 2 ? "fc32_forward_2slices" : "fc32_forward", s);
                    const dim3 grid(slices, N), block(fc32::THREADS);
                    const float *Wl = params + w_off[l];
                    auto go = [&](auto kern) {
                        hipLaunchKernelGGL(kern, grid, block, 0, s, dims[l - 1], subs, A.p, A.ld, A.stride, Wl, c->ld, part,
                                           wstride);
                    };
                    switch (nf) {
                    case 1: go(fc32::forward_ksplit_kernel<1>); break;
                    case 2: go(fc32::forward_ksplit_kernel<2>); break;
                    case 3: go(fc32::forward_ksplit_kernel<3>); break;
                    default: go(fc32::forward_ksplit_kernel<4>); break;
                    }
                    DBW_HIP(hipGetLastError());
                }
                if (head_can_sum && l == L - 1 && slices <= 16) {
                    head_splits = slices;
                    continue;
                }
                dbw_timer tm(c, "fc_reduce_kernel", s);
                hipLaunchKernelGGL(fc_reduce_kernel, dim3((B * dims[l] + 255) / 256, N), dim3(256), 0, s, part, wstride,
                                   slices, B, dims[l], params + b_off[l], c->ld, l < L ? 1 : 0, act + a_off[l],
                                   (int64_t)dims[l], wstride);
                DBW_HIP(hipGetLastError());
                continue;
            }
            const int blocks = (N + fc32::XCDS - 1) / fc32::XCDS * fc32::XCDS * (dims[l] / 32);
            dbw_timer tm(c, "fc32_forward", s);
            hipLaunchKernelGGL(fc32::forward_kernel, dim3(blocks), dim3(fc32::THREADS), 0, s, N, dims[l], dims[l - 1],
                               A.p, A.ld, A.stride, params + w_off[l], c->ld, params + b_off[l], c->ld, l < L ? 1 : 0,
                               act + a_off[l], (int64_t)dims[l], wstride);
            DBW_HIP(hipGetLastError());
            continue;
        }
        // short batches: operands straight from global memory into matrix-instruction fragments (mlp_thin.h)
        const bool may_split = head_can_sum && l == L - 1 && dims[l] <= fchead::RUN;
        ThinPlan tp = thin_plan(B, dims[l - 1], dims[l], N, may_split);
        if (may_split && !thin_forward(B, tp))             // in one part (784-200-10 on 32 x 128: the round 72.6 us with the GEMM kernel, 67.1 so)
            tp = thin_plan(B, dims[l - 1], dims[l], N, false);
        if (a.grad_path == DBW_GRAD_AUTO && B <= mlpthin::MAX_B && dims[l - 1] >= 4 && (l > 1 || fc32::aligned16(a.in)) && thin_forward(B, tp)) {
            mlpthin::FwdArgs f{};
            f.B = B; f.K = dims[l - 1]; f.N = dims[l]; f.workers = N; f.relu = l < L ? 1 : 0;
            f.splits = tp.splits; f.kper = tp.kper;
            f.a = A.p; f.a_ld = A.ld; f.a_stride = A.stride;
            f.params = params; f.p_stride = c->ld; f.w_off = w_off[l]; f.b_off = b_off[l];
            f.out = tp.splits > 1 ? act + 2 * per : act + a_off[l]; f.out_ld = dims[l]; f.out_stride = wstride;
            dbw_timer tm(c, "mlp_thin_forward", s);
            DBW_HIP(launch_thin<false>(tp, f, s));
            if (tp.splits > 1) head_splits = tp.splits;
            continue;
        }
        const int splits = forward_splits(B, dims[l], dims[l - 1], N);
        if (splits > 1) {
            float *part = act + 2 * per;
            {
                dbw_timer tm(c, "mlp_forward_gemm", s);
                DBW_HIP(bgemm::launch<64>(A, Bm, SplitOut{part, wstride, B, dims[l]}, B, dims[l], dims[l - 1], N, s,
                                          splits));
            }
            if (head_can_sum && l == L - 1) {
                head_splits = splits;
                continue;
            }
            dbw_timer tm(c, "fc_reduce_kernel", s);
            hipLaunchKernelGGL(fc_reduce_kernel, dim3((B * dims[l] + 255) / 256, N), dim3(256), 0, s, part, wstride,
                               splits, B, dims[l], params + b_off[l], c->ld, l < L ? 1 : 0, act + a_off[l],
                               (int64_t)dims[l], wstride);
            DBW_HIP(hipGetLastError());
            continue;
        }
        Epilogue E{act + a_off[l], dims[l], wstride, params + b_off[l], c->ld, nullptr, 0, 0, l < L ? 1 : 0};
        dbw_timer tm(c, "mlp_forward_gemm", s);
        DBW_HIP(bgemm::launch<64>(A, Bm, E, B, dims[l], dims[l - 1], N, s));
    }
    // Weight gradients of the layers the GEMM kernels would take: all of them in one launch when the library may
    // choose.  Batches of 256 and more: mlp_wgrad.h, four wavefronts per tile, which share the samples, where every operand allows 128-bit
    // accesses.  Shorter ones: mlp_thin.h, a tile per wavefront, on any widths (a batch that starts off a 16-byte boundary, which no
    // allocation does, keeps the GEMM kernels, which have been tested on it).  The batch-32 streaming kernels keep their layers.
    const int Lw = head.use ? L - 1 : L;
    bool grouped = !chain.use && a.grad_path == DBW_GRAD_AUTO && Lw >= 1 && fc32::aligned16(a.in);
    const WgradTiles wt = wgrad_tiles(Lw, dims, B, N, chain.use, nullptr);
    const bool thin = wt.thin;
    if (B <= mlpthin::MAX_B) {
        grouped = grouped && thin;
        for (int l = 1; l <= Lw && grouped; ++l) grouped = dims[l - 1] >= 4 && dims[l] >= 2;
    } else {
        grouped = grouped && a.in_ld % 4 == 0 && a.in_stride % 4 == 0 && fc32::aligned16(grads) &&
                  c->ld % 4 == 0 && a.param_off % 4 == 0 && fc32::aligned16(act) && wstride % 4 == 0;
        // (also the head's classes, of more than 16: there the layers below took the GEMM kernels before the head took the last one, and
        // mlp_wgrad.h rounds more: dW of 64-48-25 on 300 samples 1.19e-7, 1.39; 32 workers 43.6 us a round, 35.8; 16 x 600 256-100-25 59, 51)
        for (int l = 0; l <= (dims[L] > fchead::TILE_C ? L : Lw) && grouped; ++l) grouped = dims[l] % 4 == 0;
    }
    for (int l = 1; l <= Lw && grouped; ++l)
        grouped = !batch32_layer(B, dims[l - 1], dims[l], c->ld, w_off[l], params, grads);
    // The average on the way, where the head and one grouped launch store all gradients
    a.averaged = a.out && head.use && ((chain.use && chain.chunks > 1) || grouped || L == 1) && (L == 1 || (c->ld % 4 == 0 && fc32::aligned16(a.out) && fc32::aligned16(params)));
    if (a.averaged && (L > 1 || head.chunks == 1)) {
        const bool wide = wt.tn == 64;
        if (c->mix == DBW_MIX_DENSE)
            a.averaged = N <= average_dense(L, B, wide || thin);
        else
            a.averaged = c->max_deg <= average_list(L, B, N) &&
                         c->nnz <= average_degree(L, B, (int64_t)wt.tiles * N, wide, thin, 4 * c->d * N) * (int64_t)N;
    }
    // A short batch is one chunk of the head per worker, so that its sums over the batch are final.  When the grouped
    // launch follows, which adds per-chunk sums on the side, smaller chunks cost nothing and put the head on more CUs
    // (784-200-10, 64 samples, 32 workers: 16.1 -> 10.9 us with four chunks of 16).
    if (grouped && head.use && B <= 64)
        while (head.S > 16 && (int64_t)head.chunks * N < 256) {
            head.S /= 2;
            head.chunks = (B + head.S - 1) / head.S;
        }
    int64_t split_floats = 0;                            // the split partials of the layers, which the head's own follow
    for (int q = 1; q <= L; ++q) split_floats = std::max<int64_t>(split_floats, (int64_t)MAX_SPLITS * B * dims[q]);
    fchead::Args h{};
    if (head.use) {
        // last layer, loss and its whole backward pass in one launch (with the chain: the layers below as well)
        h.B = B; h.H = dims[L - 1]; h.C = dims[L]; h.S = head.S;
        if (L == 1) {
            h.a = a.in; h.a_ld = a.in_ld; h.a_stride = a.in_stride;
            h.da = a.din; h.da_ld = a.din_ld; h.da_stride = a.din_stride;
            h.mask = 0;
            h.bprev_off = -1;
        } else {
            h.a = act + a_off[L - 1]; h.a_ld = dims[L - 1]; h.a_stride = wstride;
            if (head_splits > 0) {      // partial products [split][B][H] instead of the finished activations
                h.a = act + 2 * per;
                h.splits = head_splits;
                h.in_bias_off = b_off[L - 1];
            }
            h.da = act + dz_off[L - 1]; h.da_ld = dims[L - 1]; h.da_stride = wstride;
            h.mask = 1;
            h.bprev_off = b_off[L - 1];
        }
        h.params = params; h.grads = grads; h.p_stride = c->ld; h.w_off = w_off[L]; h.b_off = b_off[L];
        h.y = a.y; h.loss = a.loss;
        h.part = act + 2 * per + (split_floats + 3) / 4 * 4; h.part_stride = wstride;
        h.err = c->err;
        if (a.averaged) {
            h.avg = a.avg;
            h.grads = a.out;
        }
        if (chain.use) {
            mlpchain::Args g{};
            g.B = B; g.L = L; g.K0 = dims[0]; g.H = dims[1]; g.C = dims[L];
            g.chunks = chain.chunks; g.workers = N; g.loss_kind = a.loss_kind;
            g.x = a.in; g.x_ld = a.in_ld; g.x_stride = a.in_stride;
            g.params = params; g.p_stride = c->ld;
            g.act = act; g.act_stride = wstride;
            for (int l = 1; l <= L; ++l) {
                g.w_off[l] = w_off[l]; g.b_off[l] = b_off[l]; g.a_off[l] = a_off[l]; g.dz_off[l] = dz_off[l];
            }
            h.a = nullptr; h.da = nullptr;
            g.head = h;
            const int total = chain.chunks * N;
            const dim3 grid((total + mlpchain::XCDS - 1) / mlpchain::XCDS * mlpchain::XCDS);
            auto go = [&](auto kern) -> int {
                dbw_timer tm(c, "mlp_chain_kernel", s);
                hipLaunchKernelGGL(kern, grid, dim3(mlpchain::THREADS), chain.lds, s, g);
                DBW_HIP(hipGetLastError());
                return DBW_OK;
            };
            const int rb = chain.S / 16, cb = dims[1] / 128;
            int rc = DBW_ERR_UNSUPPORTED;
            switch (rb * 8 + cb) {
            case 1 * 8 + 1: rc = go(mlpchain::kernel<1, 1>); break;
            case 1 * 8 + 2: rc = go(mlpchain::kernel<1, 2>); break;
            case 1 * 8 + 4: rc = go(mlpchain::kernel<1, 4>); break;
            case 2 * 8 + 1: rc = go(mlpchain::kernel<2, 1>); break;
            case 2 * 8 + 2: rc = go(mlpchain::kernel<2, 2>); break;
            case 2 * 8 + 4: rc = go(mlpchain::kernel<2, 4>); break;
            case 3 * 8 + 1: rc = go(mlpchain::kernel<3, 1>); break;
            case 3 * 8 + 2: rc = go(mlpchain::kernel<3, 2>); break;
            case 3 * 8 + 4: rc = go(mlpchain::kernel<3, 4>); break;
            case 4 * 8 + 1: rc = go(mlpchain::kernel<4, 1>); break;
            case 4 * 8 + 2: rc = go(mlpchain::kernel<4, 2>); break;
            case 4 * 8 + 4: rc = go(mlpchain::kernel<4, 4>); break;
            }
            if (rc != DBW_OK) return rc;

            // weight and bias gradients of the layers below the head, and the head's per-chunk sums
            const WgradPlan wp{L - 1, false, a_off, dz_off, w_off, w_off[L], per, split_floats, true};
            const int rc2 = launch_grouped_wgrad(c, a, wp, h, head.chunks, s);
            if (rc2 != DBW_OK) return rc2;
            return DBW_OK;
        } else {
        // Few workgroups: several of them to a chunk, which all stage it and form its logits and share the columns of what follows.  Not where
        // the chunk is a sum of split products, most of the work then.
        int parts = 1;
        if (head_splits == 0) parts = std::max(1, std::min((h.H + fchead::RUN - 1) / fchead::RUN, 256 / (head.chunks * N)));
        const int items = head.chunks * N;
        const dim3 grid = parts == 1 ? dim3(head.chunks, N) : dim3(items < 8 ? 8 * parts : items * parts);
        const size_t lds = fchead::lds_bytes(h.H, h.C, h.S);
        const bool vec = h.H % 4 == 0 && h.a_ld % 4 == 0 && h.a_stride % 4 == 0 && (uintptr_t)h.a % 16 == 0;
        const bool mse = a.loss_kind == DBW_LOSS_MSE;
        auto go = [&](auto kern) -> int {
            dbw_timer tm(c, "fc_head_kernel", s);
            hipLaunchKernelGGL(kern, grid, dim3(fchead::THREADS), lds, s, h, head.chunks, items, parts);
            DBW_HIP(hipGetLastError());
            return DBW_OK;
        };
        const bool mix = a.averaged && head.chunks == 1;
        auto go_split = [&](auto loss, auto ct) -> int {
            constexpr int LOSS = decltype(loss)::value, CT = decltype(ct)::value;
            if (mix && head_splits > 0) return go(fchead::kernel<LOSS, true, true, true, CT>);
            if (mix && vec) return go(fchead::kernel<LOSS, true, false, true, CT>);
            if (mix) return go(fchead::kernel<LOSS, false, false, true, CT>);
            if (head_splits > 0) return go(fchead::kernel<LOSS, true, true, false, CT>);
            return vec ? go(fchead::kernel<LOSS, true, false, false, CT>) : go(fchead::kernel<LOSS, false, false, false, CT>);
        };
        auto go_classes = [&](auto loss) -> int {
            return h.C <= fchead::TILE_C ? go_split(loss, std::integral_constant<int, 1>{}) : go_split(loss, std::integral_constant<int, 2>{});
        };
        const int rc = mse ? go_classes(std::integral_constant<int, DBW_LOSS_MSE>{}) : go_classes(std::integral_constant<int, DBW_LOSS_XENT>{});
        if (rc != DBW_OK) return rc;
        }
        if (head.chunks > 1 && !grouped) {          // (the grouped weight-gradient launch adds them otherwise)
            const int64_t E = fchead::partial_floats(h.H, h.C, L > 1);
            dbw_timer tm(c, "fc_head_reduce", s);
            hipLaunchKernelGGL(fchead::reduce_kernel, dim3((unsigned)((E + 255) / 256), N), dim3(256), 0, s, h, head.chunks);
            DBW_HIP(hipGetLastError());
        }
    } else {
        const int chunks = std::min((B + 255) / 256, DBW_LOSS_CHUNKS);
        const dim3 grid(chunks, N);
        dbw_timer tm(c, "softmax_loss_kernel", s);
        if (a.loss_kind == DBW_LOSS_MSE)
            hipLaunchKernelGGL(softmax_loss_kernel<DBW_LOSS_MSE>, grid, dim3(LOSS_THREADS), 0, s, B, dims[L], act + a_off[L], wstride,
                               a.y, act + dz_off[L], wstride, a.loss, c->loss_part, c->loss_ticket, c->err);
        else
            hipLaunchKernelGGL(softmax_loss_kernel<DBW_LOSS_XENT>, grid, dim3(LOSS_THREADS), 0, s, B, dims[L], act + a_off[L], wstride,
                               a.y, act + dz_off[L], wstride, a.loss, c->loss_part, c->loss_ticket, c->err);
        DBW_HIP(hipGetLastError());
    }
    // backward
    for (int l = Lw; l >= 1; --l) {
        const bool fast = batch32_layer(B, dims[l - 1], dims[l], c->ld, w_off[l], params, grads) && wstride % 4 == 0 &&
                          dz_off[l] % 4 == 0 && fc32::aligned16(act);
        // the data gradient: dz_{l-1} = (dz_l W_l) masked by a_{l-1} > 0, or that of the stack's input, unmasked
        const bool dgrad32 = l > 1 ? fast && a_off[l - 1] % 4 == 0 && dz_off[l - 1] % 4 == 0
                                   : a.din && fast && a.din_ld % 4 == 0 && a.din_stride % 4 == 0 && fc32::aligned16(a.din);
        bool dgrad_gemm = !dgrad32 && (l > 1 || a.din);
        const auto dg = bgemm::split_problem(
            Dense<true>{act + dz_off[l], dims[l], wstride}, Dense<false>{params + w_off[l], dims[l - 1], c->ld},
            l > 1 ? Epilogue{act + dz_off[l - 1], dims[l - 1], wstride, nullptr, 0, act + a_off[l - 1], dims[l - 1], wstride, 0}
                  : Epilogue{a.din, a.din_ld, a.din_stride, nullptr, 0, nullptr, 0, 0, 0},
            B, dims[l - 1], dims[l]);
        const ThinPlan dgrad_thin = thin_plan(B, dims[l], dims[l - 1], N, false);
        bool bias = !grouped && !(head.use && l == L - 1);   // (the head has written the bias gradient of the layer below it)
        if (!grouped) {   // dW_l = dz_l^T a_{l-1}
            Dense<false> A{act + dz_off[l], dims[l], wstride}, Bm;
            if (l == 1)
                Bm = {a.in, a.in_ld, a.in_stride};
            else
                Bm = {act + a_off[l - 1], dims[l - 1], wstride};
            if (fast && Bm.ld % 4 == 0 && Bm.stride % 4 == 0 && fc32::aligned16(Bm.p)) {
                dbw_timer tm(c, "fc32_wgrad", s);
                hipLaunchKernelGGL(fc32::wgrad_kernel, dim3(dims[l - 1] / 512, dims[l] / 32, N), dim3(fc32::THREADS), 0, s,
                                   dims[l], dims[l - 1], act + dz_off[l], (int64_t)dims[l], wstride, Bm.p, Bm.ld, Bm.stride,
                                   grads + w_off[l], c->ld);
                DBW_HIP(hipGetLastError());
            } else {
                // with the data and the bias gradient of the layer in one launch; few output tiles and a long batch: split
                // the reduction like the forward pass does
                const int cols = B >= bgemm::LONG_BATCH ? 8 : 32;
                const bgemm::BiasSums bs{act + dz_off[l], wstride, bias ? grads + b_off[l] : nullptr, c->ld, B, dims[l],
                                         (dims[l] + cols - 1) / cols};
                int splits = forward_splits(dims[l], dims[l - 1], B, N);
                int64_t part_cap = 0;
                for (int q = 1; q <= L; ++q) part_cap = std::max<int64_t>(part_cap, (int64_t)MAX_SPLITS * B * dims[q]);
                if ((int64_t)splits * dims[l] * dims[l - 1] > part_cap) splits = 1;
                if (splits > 1) {
                    float *part = act + 2 * per;
                    {
                        dbw_timer tm(c, "mlp_wgrad_gemm", s);
                        DBW_HIP(bgemm::launch_backward(bgemm::split_problem(A, Bm, SplitOut{part, wstride, dims[l], dims[l - 1]}, dims[l],
                                                                            dims[l - 1], B, splits),
                                                       dgrad_gemm ? &dg : nullptr, bs, N, s));
                    }
                    dbw_timer tm(c, "fc_reduce_kernel", s);
                    hipLaunchKernelGGL(fc_reduce_kernel, dim3((dims[l] * dims[l - 1] + 255) / 256, N), dim3(256), 0, s, part,
                                       wstride, splits, dims[l], dims[l - 1], (const float *)nullptr, (int64_t)0, 0,
                                       grads + w_off[l], (int64_t)dims[l - 1], c->ld);
                    DBW_HIP(hipGetLastError());
                } else {
                    Epilogue E{grads + w_off[l], dims[l - 1], c->ld, nullptr, 0, nullptr, 0, 0, 0};
                    dbw_timer tm(c, "mlp_wgrad_gemm", s);
                    DBW_HIP(bgemm::launch_backward(bgemm::split_problem(A, Bm, E, dims[l], dims[l - 1], B), dgrad_gemm ? &dg : nullptr,
                                                   bs, N, s));
                }
                dgrad_gemm = bias = false;
            }
        }
        if (bias) {
            dbw_timer tm(c, "colsum_kernel", s);
            hipLaunchKernelGGL(colsum_kernel, dim3((dims[l] + 31) / 32, N), dim3(256), 0, s, B, dims[l], act + dz_off[l], wstride,
                               grads + b_off[l], c->ld);
            DBW_HIP(hipGetLastError());
        }
        if (l > 1 && dgrad32) {
            dbw_timer tm(c, "fc32_dgrad", s);
            hipLaunchKernelGGL(fc32::dgrad_kernel<4>, dim3(dims[l - 1] / 128, N), dim3(fc32::THREADS), 0, s, dims[l],
                               dims[l - 1], act + dz_off[l], (int64_t)dims[l], wstride, params + w_off[l], c->ld,
                               act + a_off[l - 1], (int64_t)dims[l - 1], wstride, act + dz_off[l - 1],
                               (int64_t)dims[l - 1], wstride);
            DBW_HIP(hipGetLastError());
        } else if (dgrad32) {
            dbw_timer tm(c, "fc32_dgrad", s);
            hipLaunchKernelGGL(fc32::dgrad_kernel<1>, dim3(dims[0] / 512, N), dim3(fc32::THREADS), 0, s, dims[1], dims[0],
                               act + dz_off[1], (int64_t)dims[1], wstride, params + w_off[1], c->ld,
                               (const float *)nullptr, (int64_t)0, (int64_t)0, a.din, a.din_ld, a.din_stride);
            DBW_HIP(hipGetLastError());
        } else if (dgrad_gemm && grouped && thin && dims[l] >= 4 && !(l == 1 && bgemm::aligned(dg.A, dg.M, dg.K) && bgemm::aligned(dg.B, dg.N, dg.K)) && thin_forward(B, dgrad_thin)) {
            // (The gradient of a stack's own input, wide and with a short reduction, stays on the GEMM kernel where rows are aligned: 16 workers x
            // 50 samples, 128 -> 1568 12.4 us, here 14.8.  Elsewhere that would be the split form: rounds of 290 -> 600 on 5 x 32 139, 127.)
            mlpthin::FwdArgs f{};
            f.B = B; f.K = dims[l]; f.N = dims[l - 1]; f.workers = N;
            f.splits = 1; f.kper = dgrad_thin.kper;
            f.a = act + dz_off[l]; f.a_ld = dims[l]; f.a_stride = wstride;
            f.params = params; f.p_stride = c->ld; f.w_off = w_off[l];
            f.out = l > 1 ? act + dz_off[l - 1] : a.din; f.out_ld = l > 1 ? dims[l - 1] : a.din_ld; f.out_stride = l > 1 ? wstride : a.din_stride;
            f.mask = l > 1 ? act + a_off[l - 1] : nullptr;
            dbw_timer tm(c, "mlp_thin_dgrad", s);
            DBW_HIP(launch_thin<true>(dgrad_thin, f, s));
        } else if (dgrad_gemm) {
            // Next to another kernel's weight gradient the launch is short, and the fp32 instruction with unguarded 16-byte loads is
            // faster unless both the reduction and the grid are long (four wavefronts for every compute unit and more): 10 x 256
            // samples, 500 -> 400 units 33.2 us, split 29.5; 10 x 1 024 68, 60; but 4 x 256 22.9, 25.0, 10 x 16 20.3, 23.6, and
            // 10 x 1 024, 128 -> 384 23.8, 27.5, 32 x 64 samples, 32 -> 64 11.1, 13.0.
            const bool fp32 =
                bgemm::aligned(dg.A, dg.M, dg.K) && bgemm::aligned(dg.B, dg.N, dg.K) && (dg.K < 5 * bgemm::BK || dg.tiles() * N <= 256);
            dbw_timer tm(c, fp32 ? "mlp_dgrad_gemm" : "mlp_dgrad_split", s);
            if (fp32)
                DBW_HIP(bgemm::launch<64>(Dense<true, true>{dg.A.p, dg.A.ld, dg.A.stride}, Dense<false, true>{dg.B.p, dg.B.ld, dg.B.stride}, dg.E,
                                          dg.M, dg.N, dg.K, N, s));
            else
                DBW_HIP(bgemm::launch_split(dg, N, s));
        }
    }
    if (grouped) {
        const WgradPlan wp{Lw, !head.use, a_off, dz_off, w_off, b_off[Lw] + dims[Lw], per, split_floats, false};
        return launch_grouped_wgrad(c, a, wp, h, head.use ? head.chunks : 1, s);
    }
    return DBW_OK;
}

// The fused head uses up to 159 KB of dynamic LDS: allow that once, at create, so that no
// attribute call falls into a stream capture of the first round.
int dbw_fc_prepare()
{
    static bool done = false;
    if (done) return DBW_OK;
    const void *kernels[] = {(const void *)fchead::kernel<DBW_LOSS_MSE, true, false, false, 1>, (const void *)fchead::kernel<DBW_LOSS_MSE, false, false, false, 1>,
                             (const void *)fchead::kernel<DBW_LOSS_MSE, true, true, false, 1>, (const void *)fchead::kernel<DBW_LOSS_MSE, true, false, true, 1>,
                             (const void *)fchead::kernel<DBW_LOSS_MSE, false, false, true, 1>, (const void *)fchead::kernel<DBW_LOSS_MSE, true, true, true, 1>,
                             (const void *)fchead::kernel<DBW_LOSS_XENT, true, false, false, 1>, (const void *)fchead::kernel<DBW_LOSS_XENT, false, false, false, 1>,
                             (const void *)fchead::kernel<DBW_LOSS_XENT, true, true, false, 1>, (const void *)fchead::kernel<DBW_LOSS_XENT, true, false, true, 1>,
                             (const void *)fchead::kernel<DBW_LOSS_XENT, false, false, true, 1>, (const void *)fchead::kernel<DBW_LOSS_XENT, true, true, true, 1>,
                             (const void *)fchead::kernel<DBW_LOSS_MSE, true, false, false, 2>, (const void *)fchead::kernel<DBW_LOSS_MSE, false, false, false, 2>,
                             (const void *)fchead::kernel<DBW_LOSS_MSE, true, true, false, 2>, (const void *)fchead::kernel<DBW_LOSS_MSE, true, false, true, 2>,
                             (const void *)fchead::kernel<DBW_LOSS_MSE, false, false, true, 2>, (const void *)fchead::kernel<DBW_LOSS_MSE, true, true, true, 2>,
                             (const void *)fchead::kernel<DBW_LOSS_XENT, true, false, false, 2>, (const void *)fchead::kernel<DBW_LOSS_XENT, false, false, false, 2>,
                             (const void *)fchead::kernel<DBW_LOSS_XENT, true, true, false, 2>, (const void *)fchead::kernel<DBW_LOSS_XENT, true, false, true, 2>,
                             (const void *)fchead::kernel<DBW_LOSS_XENT, false, false, true, 2>, (const void *)fchead::kernel<DBW_LOSS_XENT, true, true, true, 2>,
                             (const void *)mlpchain::kernel<1, 1>, (const void *)mlpchain::kernel<1, 2>,
                             (const void *)mlpchain::kernel<1, 4>, (const void *)mlpchain::kernel<2, 1>,
                             (const void *)mlpchain::kernel<2, 2>, (const void *)mlpchain::kernel<2, 4>,
                             (const void *)mlpchain::kernel<3, 1>, (const void *)mlpchain::kernel<3, 2>,
                             (const void *)mlpchain::kernel<3, 4>, (const void *)mlpchain::kernel<4, 1>,
                             (const void *)mlpchain::kernel<4, 2>, (const void *)mlpchain::kernel<4, 4>};
    for (const void *k : kernels)
        DBW_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)fchead::LDS_LIMIT));
    done = true;
    return DBW_OK;
}

size_t dbw_mlp_scratch_floats(const dbw_ctx *c)
{
    return (size_t)dbw_fc_scratch_per_worker(c->model.n_layers, c->model.dims, c->model.batch) * c->N;
}

int dbw_launch_grad_mlp(dbw_ctx *c, const float *params, const float *bx, const int32_t *by, float *grads,
                        float *loss, const average::Args &avg, float *out, bool *averaged, hipStream_t s)
{
    const dbw_model &m = c->model;
    dbw_fc_args a{};
    a.L = m.n_layers;
    a.dims = m.dims;
    a.B = m.batch;
    a.loss_kind = m.loss;
    a.params = params;
    a.grads = grads;
    a.param_off = 0;
    a.in = bx;
    a.in_ld = m.dims[0];
    a.in_stride = (int64_t)m.batch * m.dims[0];
    a.act = c->act;
    a.act_stride = dbw_fc_scratch_per_worker(m.n_layers, m.dims, m.batch);
    a.y = by;
    a.loss = loss;
    a.grad_path = m.grad_path;
    a.avg = avg;
    a.out = out;
    const int rc = dbw_fc_forward_backward(c, a, s);
    if (averaged) *averaged = a.averaged;
    return rc;
}
