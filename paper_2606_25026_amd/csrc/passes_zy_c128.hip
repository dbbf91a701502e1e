// z passes of the four-pass step, complex128.
#include "passes_zy.hpp"

namespace wdm {

hipError_t launch_zy_kick_c128(const Launch& L, int nx, int ny, int nz, ZOp op, KickMode kick,
                             bool extended) {
    return ZyLaunch<double>::kick(L, nx, ny, nz, op, kick, extended);
}
hipError_t launch_zy_density_c128(const Launch& L, int nx, int ny, int nz, DensOp op, int keep,
                                const double* rescale) {
    return ZyLaunch<double>::density(L, nx, ny, nz, op, keep, rescale);
}
hipError_t launch_spec_form_c128(const Launch& L, int nx, int ny, int nz, bool to_split) {
    return ZyLaunch<double>::form(L, nx, ny, nz, to_split);
}

}  // namespace wdm
