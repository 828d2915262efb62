// plane_f32.hip -- the one-kernel y/z passes in single precision, compiled apart from
// the rest of the pipeline so the builds run in parallel.
#include "plane.h"

#define MMX_PLANE_T float
namespace mmx {
template <>
hipError_t launch_plane<float>(const Plan& p)
{
    const int M = p.P[0] / 2;
    const long nb = (long)M * (p.batch > 1 ? p.batch : 1);
    MMX_PLANE_F32(MMX_PLANE_CASE)
    return hipErrorInvalidValue;
}
}  // namespace mmx
