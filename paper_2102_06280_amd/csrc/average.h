// The consensus average on a gradient's way to memory (Section 2.1, average first):
//   out_i = P_ii x_i + sum over selected j of P_ij x_j - lr_i g_i
// A worker's new parameters need its own gradient only, so the kernel that has computed one can finish the element, instead of writing
// it for a pass over all parameters that reads it back.  Same terms in the same order as mix_csr.hip, or, in a context that averages
// densely, as mix_dense.hip's fp32 kernels (all workers, ascending; those not waited for with weight 0, so that an infinity or a NaN of
// any worker reaches every row): the results are those of a gradient pass and an averaging pass, bit for bit.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace average {

// x null: gradients are stored as they are
struct Args {
    const float *x;                  // the parameters the gradients were taken at [workers][ld]
    int64_t ld;
    const int32_t *rowptr, *p, *sel_idx;
    const float *sel_w, *self_w;
    const float *dense;              // P(k) as mix_dense_kernel holds it, of a context that averages densely, else null
    int workers;
    const float *lr_vec;             // a rate per worker, or null
    float lr;
};

// What one worker adds up, to be fetched well before use: the row that it starts with (its own; densely worker 0's) with its weight, and
// the others, the first NEAR of them here, the same in every lane (in scalar registers).  Not one per lane: a lane that takes no part
// in a branch may lose what it holds to the other side of the branch.
constexpr int NEAR = 8;
struct Row {
    int beg, cnt, first, idx[NEAR];
    float wt[NEAR], self, eta;
};
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) { return __builtin_bit_cast(float, uniform(__builtin_bit_cast(int, v))); }
// P_ij of up to 32 workers: A fragments of v_mfma_f32_32x32x2_f32
__device__ __forceinline__ float dense_weight(const Args &a, int i, int j) { return uniform(a.dense[(j >> 1) * 64 + 32 * (j & 1) + i]); }
__device__ __forceinline__ Row row(const Args &a, int w)
{
    Row r{};
    if (a.x) {
        if (a.dense) {
            r.cnt = a.workers - 1;
#pragma unroll
            for (int k = 0; k < NEAR; ++k) {
                r.idx[k] = k < r.cnt ? 1 + k : 0;
                r.wt[k] = dense_weight(a, w, r.idx[k]);
            }
            r.self = dense_weight(a, w, 0);
        } else {
            r.beg = uniform(a.rowptr[w]);
            r.cnt = uniform(a.p[w]);
            r.first = w;
#pragma unroll
            for (int k = 0; k < NEAR; ++k) {
                const int at = k < r.cnt ? r.beg + k : 0;
                r.idx[k] = uniform(a.sel_idx[at]);
                r.wt[k] = uniform(a.sel_w[at]);
            }
            r.self = uniform(a.self_w[w]);
        }
        r.eta = uniform(a.lr_vec ? a.lr_vec[w] : a.lr);
    }
    return r;
}

// V: float or a vector of floats
template <class V>
struct lanes {
    static constexpr int n = sizeof(V) / sizeof(float);
};
// A V in memory on any 4-byte boundary.  A structure: an attribute that lowers the alignment of a type which depends on a template's
// argument, or is one, is dropped, and the load promises the boundary of the whole vector.
template <class V>
struct __attribute__((packed, aligned(4))) any_boundary {
    V v;
};
static_assert(alignof(any_boundary<float __attribute__((ext_vector_type(4)))>) == 4, "no boundary beyond a float's");
template <class V>
__device__ __forceinline__ V fma(float w, V x, V acc)
{
    if constexpr (lanes<V>::n == 1) {
        return fmaf(w, x, acc);
    } else {
#pragma unroll
        for (int e = 0; e < lanes<V>::n; ++e) acc[e] = fmaf(w, x[e], acc[e]);
        return acc;
    }
}

// acc[n] = sum over j of P_ij x_j, the row's first term first, at `base` (uniform) + off[n] (bytes) of the rows of worker i = w and its neighbours, which
// waits for no gradient.  w is the same for a wavefront; a lane without an element gives any offset of the row.  The elements
// of several neighbours are fetched at a time (behind the last of them: the first row's once more).  ALL: a dense row may be longer than NEAR.
template <class V, int N, bool ALL>
__device__ __forceinline__ void gather(const Args &a, const Row &r, int w, int64_t base, const uint32_t (&off)[N], V (&acc)[N])
{
    constexpr int U = N * lanes<V>::n >= 16 ? 2 : 4;
    auto load = [&](int j, V (&v)[N]) {
        const char *row = (const char *)(a.x + (int64_t)j * a.ld + base);
#pragma unroll
        for (int n = 0; n < N; ++n) v[n] = ((const any_boundary<V> *)(row + off[n]))->v;
    };
    auto add = [&](float wt, const V (&v)[N]) {
#pragma unroll
        for (int n = 0; n < N; ++n) acc[n] = fma<V>(wt, v[n], acc[n]);
    };
    load(r.first, acc);
#pragma unroll
    for (int k = 0; k < NEAR; k += U) {
        if (k > 0 && k >= r.cnt) break;
        V v[U][N];
#pragma unroll
        for (int u = 0; u < U; ++u) load(k + u < r.cnt ? r.idx[k + u] : r.first, v[u]);
        if (k == 0) {
#pragma unroll
            for (int n = 0; n < N; ++n) acc[n] = r.self * acc[n];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k + u < r.cnt) add(r.wt[k + u], v[u]);
    }
    auto far = [&](auto entry) {
        for (int k = NEAR; k < r.cnt; k += U) {
            V v[U][N];
            float wt[U];
#pragma unroll
            for (int u = 0; u < U; ++u) load(entry(min(k + u, r.cnt - 1), wt[u]), v[u]);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k + u < r.cnt) add(wt[u], v[u]);
        }
    };
    if (ALL && a.dense) {
        far([&](int k, float &wt) { wt = dense_weight(a, w, 1 + k); return 1 + k; });
    } else {
        far([&](int k, float &wt) { wt = uniform(a.sel_w[r.beg + k]); return uniform(a.sel_idx[r.beg + k]); });
    }
}

// g[n], gradients of worker w there -> the new parameters.
template <class V, int N, bool ALL = false>
__device__ __forceinline__ void apply(const Args &a, const Row &r, int w, int64_t base, const uint32_t (&off)[N], V (&g)[N])
{
    V acc[N];
    gather<V, N, ALL>(a, r, w, base, off, acc);
#pragma unroll
    for (int n = 0; n < N; ++n) g[n] = fma<V>(-r.eta, g[n], acc[n]);
}

// One gradient of a lane, to `out` (the worker's row).
template <bool ALL = false>
__device__ __forceinline__ void store(const Args &a, const Row &r, int w, float *out, int64_t at, float g)
{
    float v[1] = {g};
    if (a.x) {
        const uint32_t off[1] = {(uint32_t)(4 * at)};
        apply<float, 1, ALL>(a, r, w, 0, off, v);
    }
    out[at] = v[0];
}

}  // namespace average
