// Internal declarations shared by the library's translation units (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "average.h"
#include "dbw.h"
#include "dbw_measure.h"

#define DBW_HIP(call)                                   \
    do {                                                \
        hipError_t e_ = (call);                         \
        if (e_ != hipSuccess) return DBW_ERR_HIP;       \
    } while (0)

constexpr int DBW_DENSE_MAX_N = 256;   // the dense mixing kernel keeps all of P(k) in registers
// the dense mixing kernel adds 32-bit per-lane byte offsets of a few rows to 64-bit uniform bases
constexpr int64_t DBW_DENSE_MAX_LD = (int64_t)UINT32_MAX / (40 * 4);
constexpr int DBW_SELECT_LDS_KEYS = 2048;
constexpr int DBW_FUSED_SELECT_MAX_N = 256;   // threshold rule + selection in one workgroup up to this many workers
constexpr int DBW_LOSS_CHUNKS = 16;     // workgroups per worker in the loss kernel, at most
constexpr int DBW_TILES_MAX_N = 256;   // the tile-major mixing kernel holds one 256-byte piece per worker in LDS

// Gradient-free rounds of graphs with at most this many links (directed) are selected and multiplied together, up to
// DBW_TAIL_ROUNDS of them per pair of launches.
constexpr int DBW_TAIL_LINKS = 4096;
constexpr int DBW_TAIL_ROUNDS = 16;

// The kernels that store a fully connected model's gradients form the average themselves (average.h) up to this many neighbours per
// worker, on average, and rows whose byte offsets fit 32 bits.  A neighbour's row is then read once per reader, from the L2 or
// the last-level cache, instead of staying in LDS.  Rounds, us, with a pass of its own / on the way: 32 workers, 784-200-10, batch 64,
// with 4, 8 and 31 neighbours 54.2 / 46.7, 54.7 / 52.0 and 54.9 / 76.5; 48 workers, 300-92-10, batch 32, 8 neighbours 28.6 /
// 30.1; 24 workers, 784-10, batch 32, 23 neighbours 23.5 / 42.3.
constexpr int DBW_AVERAGE_DEGREE = 6;
// Fewer where the parameters of a single layer fill an XCD's L2 of 4 MB, which the neighbours' rows are then fetched past: 784-10, batch 32,
// on 64, 96 and 128 workers (4 MB) with 6 neighbours 20.8 / 19.0, 21.0 / 22.0 and 21.9 / 23.5, with 4 on 128 21.6 / 21.5, on 192 25.2 / 26.8,
// with 2 on 192 24.6 / 25.5.
// Fewer for the gradients of several layers (B samples), which come in so many tiles: fewer than a quarter of the chip's wavefronts,
// and the launch that is saved is worth more; many rounds of them, and the tiles hide one another's fetches; in between every
// neighbour shows.  Batches of up to 64, a wavefront per tile: 784-36-10, batch 64, with 4 neighbours on 37 workers (962 tiles) 33.5 / 36.2,
// batch 16, with 6 on 40 (1 040) 26.8 / 32.3; 784-64-10, batch 8, 6 on 48 (1 248) 32.9 / 35.2; 784-200-10, batch 64, with 4 on 128, where 80 MB
// of parameters leave the L2 before the neighbours ask for them, 141.6 / 150.4.  Longer ones, four
// wavefronts per tile, in tiles of 64 x 64 (so many tiles that it need not be halves): 400-384-10, batch 256, 6 on 40 133 / 138, 256-384-10 on
// 24 71.3 / 72.4.
constexpr int average_degree(int L, int B, int64_t tiles, bool wide, bool thin, int64_t bytes)
{
    if (L == 1) return bytes < (int64_t)5 << 19 ? DBW_AVERAGE_DEGREE : (bytes < (int64_t)5 << 20 ? 4 : 0);
    // (mlp_thin.h on more than 64 samples, which it takes up to some 90 MB of parameters: with a pass / on the way, 4 neighbours, 784-200-10 on 64 x
    // 128, 41 MB, 118.9 / 121.1, 784-256-10 on 64 x 100, 51 MB, 138.0 / 124.3, 1024-256-10 on 64 x 96, 67 MB, 165.9 / 150.4, 1200-256-10 on 64 x
    // 100, 79 MB, 174.8 / 172.1; with 6 the third 167.8 / 153.9, 784-200-10 on 32 x 128 72.2 / 69.1)
    if (B > 64 && thin) return DBW_AVERAGE_DEGREE;
    if (B > 64) return wide ? 4 : DBW_AVERAGE_DEGREE;
    if (tiles < 512) return tiles < 256 ? DBW_AVERAGE_DEGREE : 4;
    if (tiles < 2048) return B > 32 ? (tiles < 1024 ? 2 : 4) : (B > 16 ? 4 : 2);
    return B <= 32 || bytes < (int64_t)64 << 20 ? DBW_AVERAGE_DEGREE : 2;
}
// The longest list sets the kernel's end: a tile of that worker fetches its neighbours a few at a time, which the products before
// hide the less the shorter they are.  So a round takes the pass if some worker has more neighbours than this (L layers, B samples,
// N workers); not so a single layer whose samples are summed over several workgroups, since the launch that adds those sums has
// a thread per value and the chip for itself.  A ring whose worker 0 has as many neighbours as said: 64 workers, 300-92-10, batch
// 32, 6, 8, 10 and 16 neighbours 31.7 / 30.1, 31.6 / 31.0, 31.5 / 32.5 and 31.6 / 39.8 (32 workers, 8 and 10: 25.7 / 26.0, 25.7 /
// 27.4); 32 workers, 784-200-10, batch 64, 10, 12 and 16 54.7 / 51.7, 55.1 / 55.2 and 55.1 / 60.4; 784-10, batch 32, 12 and 16 on 32
// workers 20.5 / 19.1 and 20.6 / 20.3, 8, 10 and 16 on 64 20.5 / 20.4, 20.5 / 21.5 and 20.7 / 22.8; 256-256-256-10 on 32, batch
// 256, 16 neighbours 96.6 / 89.8, batch 1 024, 24 neighbours 255 / 262.  A star of 64 workers, 784-200-10: 88 / 157.  Stars of 64
// and 256 workers, 256-10, batch 1 024: 71 / 59 and 259 / 210.
constexpr int average_list(int L, int B, int N) { return B > 64 ? 16 : (B > 32 || (L == 1 && N <= 48) ? 12 : 8); }
// A context that averages densely adds up all workers' rows, on the way as in the pass: up to as many workers as a kernel has at
// hand, fewer for the shortest batches, or, for batches of more than 64 in tiles of 64 x 32 and for single layers, twelve, and any for a
// single layer with several workgroups' sums (up to 23, with so few neighbours on average).  784-10, batch 32, on 6, 10, 12 and 16 workers
// 20.7 / 18.1, 20.7 / 18.9, 22.0 / 21.0 and 21.8 / 23.4; 784-200-10, batch 64, on 7, 10 and 12 40.7 / 36.4, 43.1 / 42.7 and 46.3 / 48.6;
// 784-36-10, batch 16, on 8 and 9 26.2 / 27.3 and 25.9 / 28.3; 256-256-256-10, batch 256, on 10 and 12 61.8 / 57.1 and 63.1 / 60.0; in tiles
// of 64 x 64, 784-384-384-10 on 9, 11 and 12 132.6 / 132.6, 151.8 / 158.1 and 159.9 / 167.7; 256-10, batch 1 024, on 12, 20 and 22 25.8 /
// 22.3, 32.7 / 29.2 and 32.9 / 30.2.
constexpr int average_dense(int L, int B, bool wide) { return L == 1 || (B > 64 && !wide) ? 12 : (B > 16 ? average::NEAR + 1 : 7); }
constexpr int64_t DBW_AVERAGE_MAX_D = (int64_t)1 << 29;

struct dbw_timing_slot {
    const char *name;
    hipEvent_t start, stop;
};

struct dbw_ctx {
    int32_t N = 0;
    int64_t d = 0, ld = 0;
    int32_t nnz = 0, max_deg = 0;
    int32_t order = DBW_ORDER_CTA;
    int32_t mix = DBW_MIX_CSR;
    int32_t layout = DBW_LAYOUT_ROWS;
    int32_t Npad = 0;                 // N rounded up to a power of two >= 32 (dense path)
    dbw_model model{};
    int64_t in_dim = 0;               // floats per sample
    bool may_average = false;         // the kernels that store a round's gradients may form the average on the way
    bool selected = false;

    std::vector<int32_t> h_rowptr, h_colidx, h_links;

    // device: graph
    int32_t *rowptr = nullptr, *colidx = nullptr;
    // device: selection state of the current round
    int32_t *p = nullptr;             // [N]
    uint8_t *mask = nullptr;          // [nnz]
    float *wait = nullptr;            // [N]
    uint8_t *listed = nullptr;        // [N] scratch of the round-time kernel
    int32_t *sel_idx = nullptr;       // [nnz] row i: first p_i entries = selected neighbours, ascending
    float *sel_w = nullptr;           // [nnz] their weights
    float *self_w = nullptr;          // [N]
    float *Wdense = nullptr;          // [Npad*Npad] in MFMA A-fragment order (dense path only)
    float *phi[2] = {nullptr, nullptr};   // [Npad*Npad] running product of consensus matrices (N <= 256)
    float *phi_frag = nullptr;        // the product in MFMA A-fragment order
    // selections of several gradient-free rounds at once (N <= 256, nnz <= DBW_TAIL_LINKS), else null
    int32_t *tail_p = nullptr;        // [DBW_TAIL_ROUNDS][N]
    float *tail_self = nullptr;       // [DBW_TAIL_ROUNDS][N]
    int32_t *tail_idx = nullptr;      // [DBW_TAIL_ROUNDS][nnz]
    float *tail_w = nullptr;          // [DBW_TAIL_ROUNDS][nnz]
    int32_t *err = nullptr;           // [1] deferred status
    // device: threshold rule
    int32_t *links = nullptr;         // [2*(N-1)]
    uint8_t *visited = nullptr;       // [N-1]
    int32_t *n_visited = nullptr;     // [1]
    // device: model scratch
    float *grads = nullptr;           // [N*ld] when a model is attached
    float *act = nullptr;             // activations / deltas
    float *loss_part = nullptr;       // [N][DBW_LOSS_CHUNKS] partial loss sums of the loss kernel
    uint32_t *loss_ticket = nullptr;  // [N] arrival counters of the loss kernel, zero between launches
    size_t act_floats = 0;

    // timing
    bool timing = false;
    std::vector<dbw_timing_slot> slots;
    std::vector<hipEvent_t> free_events;
};

struct dbw_timer {
    dbw_ctx *c;
    hipStream_t s;
    hipEvent_t stop = nullptr;
    dbw_timer(dbw_ctx *ctx, const char *name, hipStream_t st);
    ~dbw_timer();
};

// api.hip: CSR rows strictly ascending, in range, loop-free, symmetric (DBW_ERR_GRAPH otherwise)
int dbw_validate_graph(int32_t N, const int32_t *rowptr, const int32_t *colidx);
// select.hip
int dbw_launch_select(dbw_ctx *c, const float *t, const int32_t *b, hipStream_t s);
// Selections of rounds 0 .. rounds - 1 (t, b [rounds][N]) into the context's tail arrays; if last, those of the
// last round go to the context's selection state instead, as dbw_launch_select leaves it.
int dbw_launch_select_tail(dbw_ctx *c, const float *t, const int32_t *b, int rounds, bool last, hipStream_t s);
int dbw_launch_round_time(dbw_ctx *c, float *out, hipStream_t s);
int dbw_launch_dtur(dbw_ctx *c, const float *t, int32_t *b_out, float *theta_out, hipStream_t s);
bool dbw_fused_dtur_select_fits(const dbw_ctx *c);
int dbw_launch_dtur_select(dbw_ctx *c, const float *t, int32_t *b_out, float *theta_out, hipStream_t s);
int dbw_launch_dtur_reset(dbw_ctx *c, hipStream_t s);
int dbw_launch_dense_weights(dbw_ctx *c, float *P, hipStream_t s);
// Order in which the workgroups of an average over column tiles take them, a round of tiles being one to each.  Workgroups go round the
// eight XCDs; numbered by XCD (TOGETHER), neighbouring tiles, which share cache lines unless every row starts on one, are worked on by one XCD at
// a time, whose L2 then fetches a shared line once and writes it once.  Rows of odd length without padding, 48 workers x 1 000 003 columns
// with gradients 131 -> 121 us, 128 x 2 800 001 1093 -> 872, densely 128 x 1 000 001 446 -> 381, 256 x 500 001 555 -> 502; rows on lines the
// same to within what differs from card to card (64 x 2 160 000 314 -> 308; 128 x 2 800 000, local step first, 822 -> 826 on one, 811 -> 796 on another).  The tiles of a last, partial round go to the XCDs in turn, or half of the chip would have them all (densely 34
// workers x 47 710 columns 12.2 us, 14.1 so).
template <bool TOGETHER, class T>
struct TileWalk {
    T whole, n_tiles;                 // tiles of whole rounds, and all
    T grid, block;
    __device__ __forceinline__ TileWalk(T n) : whole(n / (T)gridDim.x * (T)gridDim.x), n_tiles(n), grid((T)gridDim.x), block((T)blockIdx.x) {}
    __device__ __forceinline__ T first() const      // (a grid has no more workgroups than there are tiles)
    {
        return TOGETHER && grid % 8 == 0 ? (block % 8) * (grid / 8) + block / 8 : block;
    }
    __device__ __forceinline__ T next(T t) const      // n_tiles or more: none
    {
        if (!TOGETHER) return t + grid;
        return t + grid < whole ? t + grid : (t < whole ? whole + block : n_tiles);
    }
};
// mix_csr.hip
// Learning rate of a round as the mixing kernels see it: one value for all workers, or
// eta_j per worker read from device memory (Section 2.1).
struct dbw_lr_scalar {
    float v;
    __device__ __forceinline__ float at(int) const { return v; }
};
struct dbw_lr_vector {
    const float *v;
    __device__ __forceinline__ float at(int j) const { return v[j]; }
};

// lr_vec (device, N) overrides lr when it is not null.
int dbw_launch_mix_csr(dbw_ctx *c, const float *x, const float *g, float *out, float lr, const float *lr_vec,
                       hipStream_t s);
// mix_dense.hip
// W (A-fragment order, Npad x Npad) defaults to the matrix of the last selection.
int dbw_launch_mix_dense(dbw_ctx *c, const float *x, const float *g, float *out, float lr, const float *lr_vec,
                         hipStream_t s, const float *W = nullptr);
// mix_tiles.hip (tile-major layout)
int dbw_launch_mix_tiles(dbw_ctx *c, const float *x, const float *g, float *out, float lr, const float *lr_vec,
                         hipStream_t s);
int dbw_launch_layout_convert(dbw_ctx *c, const float *src, float *dst, int to_tiles, hipStream_t s);
// consensus.hip
int dbw_launch_consensus_rounds(dbw_ctx *c, const float *x, float *out, const float *t, const int32_t *b, int r,
                                hipStream_t s);
// grad_mlp.hip / grad_cnn.hip
// A stack of fully connected layers dims[0] -> ... -> dims[L] with ReLU between layers and
// softmax cross-entropy on top, for all workers.  Parameters of the stack start at float
// offset param_off inside each worker's row (row stride c->ld); gradients go to the same
// offsets of `grads`.  `in` is the stack's input [B][in_ld] per worker; `act` is scratch of
// act_stride floats per worker (see dbw_fc_scratch_per_worker); `din`, if not null,
// receives the gradient with respect to the input.
struct dbw_fc_args {
    int L, B, loss_kind;
    const int32_t *dims;
    const float *params;
    float *grads;
    int64_t param_off;
    const float *in;
    int64_t in_ld, in_stride;
    float *act;
    int64_t act_stride;
    float *din;
    int64_t din_ld, din_stride;
    const int32_t *y;
    float *loss;
    int grad_path;          // DBW_GRAD_*
    // A round's average, if the kernels that store the gradients may form it on the way (average.h); then out is where the
    // new parameters go, and averaged tells the caller whether that has happened (otherwise `grads` has the gradients).
    average::Args avg;
    float *out;
    bool averaged;
};
int64_t dbw_fc_scratch_per_worker(int L, const int32_t *dims, int B);
bool dbw_fc_chain_shape_ok(int L, const int32_t *dims, int B, int workers);   // DBW_GRAD_CHAIN can take this model
int dbw_fc_prepare();   // one-time kernel attributes of the fully connected path
int dbw_fc_forward_backward(dbw_ctx *c, dbw_fc_args &a, hipStream_t s);
size_t dbw_mlp_scratch_floats(const dbw_ctx *c);
// out, if not null: averages on the way to there where that is faster, and says so in *averaged (see dbw_fc_args).
int dbw_launch_grad_mlp(dbw_ctx *c, const float *params, const float *bx, const int32_t *by, float *grads,
                        float *loss, const average::Args &avg, float *out, bool *averaged, hipStream_t s);
int dbw_cnn_prepare();  // one-time kernel attributes of the convolutions
size_t dbw_cnn_scratch_floats(const dbw_ctx *c);
int dbw_launch_grad_cnn(dbw_ctx *c, const float *params, const float *bx, const int32_t *by, float *grads,
                        float *loss, hipStream_t s);
