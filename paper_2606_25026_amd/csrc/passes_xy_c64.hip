// Plane passes of the four-pass step, complex64.
#include "passes_xy.hpp"

namespace wdm {

hipError_t launch_xy_kinetic_c64(const Launch& L, int nx, int ny, int nz) {
    return XyLaunch<float, kPlaneKinetic>::run(L, nx, ny, nz);
}
hipError_t launch_xy_green_c64(const Launch& L, int nx, int ny, int nz) {
    return XyLaunch<float, kPlaneGreen>::run(L, nx, ny, nz);
}

}  // namespace wdm
