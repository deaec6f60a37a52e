// Several gradient-free consensus rounds in one pass over the parameters.
//
// Without gradients, r rounds are X' = P(k+r-1) ... P(k+1) P(k) X (rows are workers): the product
// Phi of the consensus matrices (Section 3.1) is N x N, so it is formed first, with one tiny
// kernel per round that applies that round's selected-neighbour lists to the running product, and
// the N x d parameter matrix is then multiplied once on the matrix cores instead of being
// streamed r times.
#include "dbw_internal.h"

namespace {

// Phi = identity on the first N rows, zero elsewhere.  grid = Npad, block = Npad.
__global__ void phi_identity_kernel(int N, int Npad, float *__restrict__ phi)
{
    const int i = blockIdx.x, c = threadIdx.x;
    phi[(size_t)i * Npad + c] = (i == c && i < N) ? 1.0f : 0.0f;
}

// next = P(k) prev with row i of P(k) given by self_w[i] and the first p[i] entries of row i of
// (sel_idx, sel_w), summed in that fixed order.  grid = N, block = Npad.
__global__ void phi_step_kernel(int Npad, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ p,
                                const int32_t *__restrict__ sel_idx, const float *__restrict__ sel_w,
                                const float *__restrict__ self_w, const float *__restrict__ prev,
                                float *__restrict__ next)
{
    __shared__ int32_t s_idx[DBW_DENSE_MAX_N];
    __shared__ float s_w[DBW_DENSE_MAX_N];
    const int i = blockIdx.x, c = threadIdx.x;
    const int beg = rowptr[i], cnt = p[i];
    if (c < cnt) {                                     // cnt <= N - 1 < Npad = blockDim.x
        s_idx[c] = sel_idx[beg + c];
        s_w[c] = sel_w[beg + c];
    }
    __syncthreads();
    float acc = self_w[i] * prev[(size_t)i * Npad + c];
    // the loads of eight neighbours are in flight together; the sum keeps its order
    int k = 0;
    for (; k + 8 <= cnt; k += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = prev[(size_t)s_idx[k + u] * Npad + c];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = fmaf(s_w[k + u], v[u], acc);
    }
    for (; k < cnt; ++k) acc = fmaf(s_w[k], prev[(size_t)s_idx[k] * Npad + c], acc);
    next[(size_t)i * Npad + c] = acc;
}

// Row-major Phi -> the order in which the dense mixing kernel reads it: [row block of 32][k pair][lane],
// lane = 32 (column & 1) + (row & 31).  Padding rows [N, Npad) become zero whatever the buffer holds there.
// grid = Npad, block = Npad.
__global__ void phi_fragment_kernel(int N, int Npad, const float *__restrict__ phi, float *__restrict__ frag)
{
    const int i = blockIdx.x, c = threadIdx.x;
    const int KB = Npad / 2;
    frag[((size_t)(i >> 5) * KB + (c >> 1)) * 64 + (c & 1) * 32 + (i & 31)] = i < N ? phi[(size_t)i * Npad + c] : 0.0f;
}

// Several rounds' products in one launch, for graphs whose neighbour lists fit LDS: the columns of Phi are independent,
// so a workgroup takes TAIL_COLS of them through all rounds, the running product in LDS.  It starts from the
// identity (prev null) or from a row-major product, and leaves the fragment order above (frag) or a row-major product
// (next).  Sums as in phi_step_kernel.  Round q's lists are the tail arrays' q-th, the last round's the context's
// selection state if last_state.  A launch per round and selection (13 us a round) becomes two launches for up to
// DBW_TAIL_ROUNDS rounds: 8 rounds of 128 workers with 8
// neighbours 117 -> 33 us, 64 workers in a complete graph 137 -> 77.  What is left is a chain of dependent LDS reads, list entry and then
// product, in every round: four entries at a time, and a thread for every element of 256 rows x 4 columns (eight columns on
// 512 threads, entry by entry / so): the first example, with 20 000 columns averaged, 36.2 / 26.1; 256 workers, 8 neighbours, 12
// rounds, 10 000 columns 76.7 / 45.3; 60 workers in a complete graph, 6 rounds 56.7 / 37.9.  grid = Npad / TAIL_COLS.
constexpr int TAIL_COLS = 4, TAIL_THREADS = 1024, TAIL_STAGE = 8;
__global__ __launch_bounds__(TAIL_THREADS) void phi_tail_kernel(
    int N, int Npad, int nnz, int rounds, int last_state, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ tail_p,
    const int32_t *__restrict__ tail_idx, const float *__restrict__ tail_w, const float *__restrict__ tail_self,
    const int32_t *__restrict__ p, const int32_t *__restrict__ sel_idx, const float *__restrict__ sel_w,
    const float *__restrict__ self_w, const float *__restrict__ prev, float *__restrict__ next, float *__restrict__ frag)
{
    __shared__ float phi[2][DBW_DENSE_MAX_N * TAIL_COLS];
    __shared__ int2 list[DBW_TAIL_LINKS];                                // (neighbour, weight) of the rounds staged
    __shared__ int2 row[TAIL_STAGE * DBW_DENSE_MAX_N];                   // (length, own weight)
    __shared__ int32_t rp[DBW_DENSE_MAX_N + 1];
    const int tid = threadIdx.x, col = tid % TAIL_COLS, c0 = blockIdx.x * TAIL_COLS;
    for (int i = tid; i <= N; i += TAIL_THREADS) rp[i] = rowptr[i];
    for (int e = tid; e < N * TAIL_COLS; e += TAIL_THREADS) {
        const int i = e / TAIL_COLS, c = c0 + e % TAIL_COLS;
        phi[0][e] = prev ? prev[(size_t)i * Npad + c] : (i == c ? 1.0f : 0.0f);
    }
    const int stage = min(min(rounds, TAIL_STAGE), DBW_TAIL_LINKS / max(nnz, 1));
    int cur = 0;
    for (int q0 = 0; q0 < rounds; q0 += stage) {
        const int n = min(stage, rounds - q0);
        __syncthreads();
        for (int e = tid; e < n * nnz; e += TAIL_THREADS) {
            const int q = q0 + e / nnz, k = e % nnz;
            const bool state = last_state && q == rounds - 1;
            list[e] = make_int2(state ? sel_idx[k] : tail_idx[(size_t)q * nnz + k],
                                __float_as_int(state ? sel_w[k] : tail_w[(size_t)q * nnz + k]));
        }
        for (int e = tid; e < n * N; e += TAIL_THREADS) {
            const int q = q0 + e / N, i = e % N;
            const bool state = last_state && q == rounds - 1;
            row[e] = make_int2(state ? p[i] : tail_p[(size_t)q * N + i], __float_as_int(state ? self_w[i] : tail_self[(size_t)q * N + i]));
        }
        __syncthreads();
        for (int q = 0; q < n; ++q) {
            for (int i = tid / TAIL_COLS; i < N; i += TAIL_THREADS / TAIL_COLS) {
                const int2 r = row[q * N + i];
                const int2 *l = &list[q * nnz + rp[i]];
                float acc = __int_as_float(r.y) * phi[cur][i * TAIL_COLS + col];
                for (int k = 0; k < r.x; k += 4) {       // four neighbours under way (behind the last: that one again, not added)
                    int2 e[4];
                    float v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) e[u] = l[min(k + u, r.x - 1)];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = phi[cur][e[u].x * TAIL_COLS + col];
#pragma unroll
                    for (int u = 0; u < 4; ++u) acc = k + u < r.x ? fmaf(__int_as_float(e[u].y), v[u], acc) : acc;
                }
                phi[cur ^ 1][i * TAIL_COLS + col] = acc;
            }
            cur ^= 1;
            __syncthreads();
        }
    }
    for (int e = tid; e < Npad * TAIL_COLS; e += TAIL_THREADS) {
        // frag wants consecutive rows next to each other, a row-major product consecutive columns
        const int i = frag ? e % Npad : e / TAIL_COLS, cl = frag ? e / Npad : e % TAIL_COLS, c = c0 + cl;
        const float v = i < N ? phi[cur][i * TAIL_COLS + cl] : 0.0f;
        if (frag) frag[((size_t)(i >> 5) * (Npad / 2) + (c >> 1)) * 64 + (c & 1) * 32 + (i & 31)] = v;
        else next[(size_t)i * Npad + c] = v;
    }
}

// The product of the r rounds' consensus matrices, in fragment order, through the kernel above.
int launch_tail_product(dbw_ctx *c, const float *t, const int32_t *b, int r, hipStream_t s)
{
    for (int q = 0; q < r; q += DBW_TAIL_ROUNDS) {
        const int n = r - q < DBW_TAIL_ROUNDS ? r - q : DBW_TAIL_ROUNDS;
        const bool last = q + n == r;
        const int rc = dbw_launch_select_tail(c, t + (size_t)q * c->N, b + (size_t)q * c->N, n, last, s);
        if (rc != DBW_OK) return rc;
        dbw_timer tm(c, "phi_tail_kernel", s);
        const int k = q / DBW_TAIL_ROUNDS;                               // the products alternate between two buffers
        hipLaunchKernelGGL(phi_tail_kernel, dim3(c->Npad / TAIL_COLS), dim3(TAIL_THREADS), 0, s, c->N, c->Npad, c->nnz, n,
                           last ? 1 : 0, c->rowptr, c->tail_p, c->tail_idx, c->tail_w, c->tail_self, c->p, c->sel_idx, c->sel_w,
                           c->self_w, q ? c->phi[(k - 1) & 1] : (const float *)nullptr, last ? (float *)nullptr : c->phi[k & 1],
                           last ? c->phi_frag : (float *)nullptr);
        DBW_HIP(hipGetLastError());
    }
    return DBW_OK;
}

}  // namespace

int dbw_launch_consensus_rounds(dbw_ctx *c, const float *x, float *out, const float *t, const int32_t *b, int r,
                                hipStream_t s)
{
    if (c->nnz <= DBW_TAIL_LINKS) {
        const int rc = launch_tail_product(c, t, b, r, s);
        return rc != DBW_OK ? rc : dbw_launch_mix_dense(c, x, nullptr, out, 0.f, nullptr, s, c->phi_frag);
    }
    const int Npad = c->Npad;
    float *cur = c->phi[0], *nxt = c->phi[1];
    {
        dbw_timer tm(c, "phi_identity_kernel", s);
        hipLaunchKernelGGL(phi_identity_kernel, dim3(Npad), dim3(Npad), 0, s, c->N, Npad, cur);
        DBW_HIP(hipGetLastError());
    }
    for (int q = 0; q < r; ++q) {
        const int rc = dbw_launch_select(c, t + (size_t)q * c->N, b + (size_t)q * c->N, s);
        if (rc != DBW_OK) return rc;
        dbw_timer tm(c, "phi_step_kernel", s);
        hipLaunchKernelGGL(phi_step_kernel, dim3(c->N), dim3(Npad), 0, s, Npad, c->rowptr, c->p, c->sel_idx, c->sel_w,
                           c->self_w, cur, nxt);
        DBW_HIP(hipGetLastError());
        float *tmp = cur;
        cur = nxt;
        nxt = tmp;
    }
    {
        dbw_timer tm(c, "phi_fragment_kernel", s);
        hipLaunchKernelGGL(phi_fragment_kernel, dim3(Npad), dim3(Npad), 0, s, c->N, Npad, cur, c->phi_frag);
        DBW_HIP(hipGetLastError());
    }
    return dbw_launch_mix_dense(c, x, nullptr, out, 0.f, nullptr, s, c->phi_frag);
}
