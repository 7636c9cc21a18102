// mfma_plan.h -- host arithmetic of the int8 matrix-core passes (no HIP here): how a
// launch splits its work.
#pragma once
#include <cstdint>

namespace cox {

// The dense product over nblk blocks of subjects, nstage stages of 64 columns each, one
// workgroup resident per compute unit: blocks below nfull fill whole rounds, those of
// the last, partly filled one are split into ksplit runs of stages where that saves time.
// Its cost is rounds of shares x (their stages + the fill and flush of a workgroup,
// about 6 stages); a share's sums of one block take block_words of the `room`.  With
// no number of compute units (ncu = 0: the device did not give it) or no room nothing is
// split.
struct DensePlan {
    int64_t nfull;
    int ksplit;
};
inline DensePlan dense_plan(int64_t nblk, int64_t nstage, int64_t ncu, int64_t block_words, int64_t room)
{
    const int64_t ntail = ncu > 0 ? nblk % ncu : 0;
    DensePlan d{nblk - ntail, 1};
    int64_t best = nstage + 6;
    for (int64_t k = 2; k <= 16 && k <= nstage && ntail > 0; ++k) {
        if (k * ntail * block_words > room) break;
        const int64_t c = (ntail * k + ncu - 1) / ncu * ((nstage + k - 1) / k + 6);
        if (c < best) {
            best = c;
            d.ksplit = (int)k;
        }
    }
    return d;
}

}  // namespace cox
