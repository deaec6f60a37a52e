// The sizes of the short-batch forward kernel's work (mlp_thin.h): host code without HIP, so that a test can compile it by itself.
#pragma once

#include <stdint.h>

namespace mlpthin {

constexpr int FWD_WAVES = 8;             // wavefronts of a workgroup
constexpr int MAX_B = 255;               // samples

// How mlp_thin.h's forward_kernel cuts up a product of B x K by K x N: blocks of at most 64 samples, tiles of 32 or 16 outputs, and, where the
// sums may be left to the reader, parts of the reduction: whatever gives the shortest time, in cycles, for the compute unit with most
// workgroups.  A wavefront takes every eighth chunk of 16 k, for which the matrix instructions (two wavefronts to a SIMD) and the loads take about
// as long as said here; a part more is a sum more for the reader, the head (and none where the head's workgroups would rather share its
// chunks by runs of columns: 784-420-10 on 20 workers x 19 samples 44 us, in two parts 47).  Rounds, with nothing for the loads beside the
// instructions and 500 for a part / so: 784-700-30 on 64 x 64 (tiles of 16 outputs / 32) 252 / 232 us, 256-168-10 on 32 x 64 (two parts / one) 35.2 /
// 34.1, 1024-200-10 on 16 x 64 40.2 / 39.0; with 1 500 for a part 784-128-10 on 8 x 32 26.5 instead of 25.9.
struct ThinPlan {
    int RB, CB, blocks, splits, kper;
    int64_t wgs;
};
inline ThinPlan thin_plan(int B, int K, int N, int workers, bool may_split)
{
    ThinPlan best{};
    int64_t least = 0;
    const int chunks = (K + 15) / 16, blocks = (B + 63) / 64, RB = ((B + blocks - 1) / blocks + 15) / 16;
    for (int splits = 1; splits <= (may_split ? 8 : 1); splits *= 2)
        for (int CB = 2; CB >= 1; --CB) {
            const int kper = (chunks + splits - 1) / splits;
            if (splits > 1 && kper < FWD_WAVES) continue;
            const int64_t wgs = (int64_t)((N + 16 * CB - 1) / (16 * CB)) * blocks * splits * workers;
            const int64_t iter = 256 * RB * CB + 100 * (RB + CB);
            const int64_t cost = (wgs + 255) / 256 * ((kper + FWD_WAVES - 1) / FWD_WAVES) * iter + 800 * (splits - 1);
            if (best.wgs == 0 || cost < least) {
                least = cost;
                best = {RB, CB, blocks, splits, kper, wgs};
            }
        }
    return best;
}

// More tiles, of longer batches: the GEMM kernel, whose wavefronts share what they fetch; 1023-511-509-10 on 30 x 250 151 us, mlp_thin.h
// 229, 784-500-10 on 32 x 200 76 and 82, x 128 46 and 46, 300-300-300-10 on 32 x 128 51 and 41.
inline bool thin_forward(int B, const ThinPlan &tp) { return B <= 64 || tp.wgs * tp.CB <= 2048; }

}  // namespace mlpthin
