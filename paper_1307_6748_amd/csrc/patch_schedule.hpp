// How many blocks of sweeps a patch solve queues before the host looks at its
// state again.  Host code without HIP, so that it can be tested on its own.
#pragma once
#include <algorithm>
#include <cmath>

namespace isis {

// Most blocks queued between two looks: 64 blocks of 4 sweeps are about 600
// launches, which queue faster than they run.
constexpr int kPatchBatch = 64;

// Blocks of the next batch after one of `batch` blocks took the RMS defect from
// r0 to rms: as many as the mean factor per block predicts until tol, four
// times the last batch at most.  These factors rise towards their asymptotic
// value, so the prediction errs on the early side and few launches run past
// the block that meets tol.  One block where less than one is left, or where
// the defect did not fall: a block that turns out not to be needed costs its
// launches (68^3 chameleon, blocks of 50 sweeps: up to 8 blocks in these cases
// made a solve 12.5 ms long, one 8.3).
inline int next_patch_batch(int batch, double r0, double rms, double tol)
{
    const double rho = std::pow(rms / r0, 1.0 / batch);
    const double left = std::log(tol / rms) / std::log(rho);
    if (!(rho < 1.0) || !(left >= 1.0)) return 1;
    return (int)std::min({std::ceil(left), 4.0 * batch, (double)kPatchBatch});
}

}  // namespace isis
