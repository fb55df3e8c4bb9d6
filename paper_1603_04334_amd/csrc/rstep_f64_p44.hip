// Row-pair step: FP64 blocks, LDS rows of 44 values, grid rows of whole units.
#include <algorithm>

#include "rstep_launch.hpp"

namespace sparc {

int rstep_f64_p44(const RStepArgs<double> &a, const GatherArgs<double, double> &g, int natoms, int ncb, int nitems, int ngb,
       int nthreads, int nh, bool prev, bool strm, hipStream_t s)
{
    return rstep_dispatch<double, 44, 0>(a, g, natoms, ncb, nitems, ngb, nthreads, nh, prev, strm, s);
}

}  // namespace sparc
