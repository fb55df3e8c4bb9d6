// Row-pair step: FP32 blocks, LDS rows of 176 values, grid rows 1 node short of whole units.
#include <algorithm>

#include "rstep_launch.hpp"

namespace sparc {

int rstep_f32_p176_r1(const RStepArgs<float> &a, const GatherArgs<float, float> &g, int natoms, int ncb, int nitems, int ngb,
       int nthreads, int nh, bool prev, bool strm, hipStream_t s)
{
    return rstep_dispatch<float, 176, 1>(a, g, natoms, ncb, nitems, ngb, nthreads, nh, prev, strm, s);
}

}  // namespace sparc
