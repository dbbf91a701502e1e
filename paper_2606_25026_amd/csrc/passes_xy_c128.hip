// Plane passes of the four-pass step, complex128.
#include "passes_xy.hpp"

namespace wdm {

hipError_t launch_xy_kinetic_c128(const Launch& L, int nx, int ny, int nz) {
    return XyLaunch<double, kPlaneKinetic>::run(L, nx, ny, nz);
}
hipError_t launch_xy_green_c128(const Launch& L, int nx, int ny, int nz) {
    return XyLaunch<double, kPlaneGreen>::run(L, nx, ny, nz);
}

}  // namespace wdm
