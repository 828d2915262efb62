// plane_f64.hip -- the one-kernel y/z passes in double precision, compiled apart from
// the rest of the pipeline so the builds run in parallel.
#include "plane.h"

#define MMX_PLANE_T double
namespace mmx {
template <>
hipError_t launch_plane<double>(const Plan& p)
{
    const int M = p.P[0] / 2;
    const long nb = (long)M * (p.batch > 1 ? p.batch : 1);
    MMX_PLANE_F64(MMX_PLANE_CASE)
    return hipErrorInvalidValue;
}
}  // namespace mmx
