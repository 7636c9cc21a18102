// mfma_plan.h -- host arithmetic of the int8 matrix-core passes (no HIP here): how many
// terms one int32 sum may take, and how a launch splits its work.
#pragma once
#include <algorithm>
#include <cstdint>

namespace cox {

// The passes sum int8 limbs (-128 .. 127) times counts (0 .. 2) in int32: over subjects
// in X~' R, over columns in the eta update and the dense product.  256 K <= 2^31 for K
// <= 2^23; beyond it many equal limbs (tied residuals, equal coefficients) would wrap.
// A longer sum is taken in runs of at most this many terms (a multiple of every
// stage), added in int64 or FP64.
constexpr int64_t kMfmaMaxSum = (int64_t(1) << 23) - 128;

// Shares that hold a sum of nstage stages of `stage` terms to kMfmaMaxSum each
constexpr int64_t min_shares(int64_t nstage, int64_t stage)
{
    return (nstage + kMfmaMaxSum / stage - 1) / (kMfmaMaxSum / stage);
}

constexpr int64_t kMaxSplit = 16;  // shares of a block that is split only to fill the chip

// The dense product over nblk blocks of subjects, nstage stages of 64 columns each, one
// workgroup resident per compute unit: blocks below nfull fill whole rounds, those of
// the last, partly filled one are split into ksplit runs of stages where that saves time.
// Its cost is rounds of shares x (their stages + the fill and flush of a workgroup,
// about 6 stages); a share's sums of one block take block_words of the `room`.  With
// no number of compute units (ncu = 0: the device did not give it) or no room nothing is
// split.  From kMfmaMaxSum columns on every block is, and ksplit = 0 says that there is
// no room for it.
struct DensePlan {
    int64_t nfull;
    int ksplit;
};
inline DensePlan dense_plan(int64_t nblk, int64_t nstage, int64_t ncu, int64_t block_words, int64_t room)
{
    const int64_t kmin = min_shares(nstage, 64), slots = std::max<int64_t>(1, ncu);
    const int64_t ntail = kmin > 1 ? nblk : ncu > 0 ? nblk % ncu : 0;
    DensePlan d{nblk - ntail, kmin > 1 ? 0 : 1};
    int64_t best = kmin > 1 ? INT64_MAX : nstage + 6;
    for (int64_t k = std::max<int64_t>(2, kmin); k <= std::max(kMaxSplit, kmin) && k <= nstage && ntail > 0; ++k) {
        if (k * ntail * block_words > room) break;
        const int64_t c = (ntail * k + slots - 1) / slots * ((nstage + k - 1) / k + 6);
        if (c < best) {
            best = c;
            d.ksplit = (int)k;
        }
    }
    return d;
}

// Shares each block of the last round's `ntail` blocks of X~' R is split into (shape
// 15), of nstage stages of 128 subjects each, on `slots` resident workgroups: the split
// with the least
//     rounds of shares x (stages of a share + the fill and flush of a workgroup)
//     + the shares' partial sums, written and read once (a stage moves 32 KB of X
//     per compute unit in about 1.5 us; the sums move at about 4 TB/s).
// A part-filled round costs a whole one, so 196 blocks of 1,563 stages on 256
// slots take 4 rounds of 313 stages in fifths (1.91 ms at 200,000 x 50,000 x 64;
// 2.09 ms unsplit), and 3 blocks of 24 stages take 2 stages in
// twelfths (15 us; 21 us in thirds).  At least min_shares (the caller then gives every
// block as ntail); 0: no room for the sums of ptail columns in that many.
inline int xtr_split(int64_t ntail, int64_t nstage, int64_t slots, int64_t ptail, int B, int64_t room)
{
    constexpr int64_t kFill = 6;
    const int64_t kmin = min_shares(nstage, 128);
    int best = 0;
    double cost = 1e300;
    for (int64_t k = kmin; k <= std::max(kMaxSplit, kmin) && k <= nstage && (k == 1 || k * ptail <= room); ++k) {
        const double c = (double)((ntail * k + slots - 1) / slots * ((nstage + k - 1) / k + kFill)) +
                         (k > 1 ? 16.0 * (double)(k * ptail) * B / 6e6 : 0.0);
        if (c < cost) {
            cost = c;
            best = (int)k;
        }
    }
    return best;
}

// The room the two plans are given in the handle's buffer of partial sums, whatever more it
// holds: columns over all shares of X~' R per vector, up to 6 shares of a full round of
// columns and 16 of a small problem's, and words of the dense product's sums, up to 12 M;
// at least the shares that int32 sums need.  X~' R's cost rule leaves out that shares of
// a block read different limb rows at once, so room for more costs time (400,000 x
// 500,000 x 64: 38.6 ms in elevenths, 38.2 in the thirds taken within this).
inline int64_t xtr_room(int64_t n, int64_t p, int64_t ncu)
{
    const int64_t k = min_shares((n + 127) / 128, 128);
    return std::max(std::min(6 * ncu * 256, kMaxSplit * p), k > 1 ? k * p : 0);
}
inline int64_t dense_room(int64_t n, int64_t p)
{
    const int64_t k = min_shares((p + 63) / 64, 64), rows = (n + 511) / 512 * 512 * 3 * 32;
    return std::max(std::min(int64_t(12) << 20, kMaxSplit * rows), k > 1 ? k * rows : 0);
}

}  // namespace cox
