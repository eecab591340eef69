// the kernels that form the ghosts and the wave speeds of a state that comes from the host
#include "gks_kernels.h"

namespace gks {
template __global__ void k_ghost_fill<double>(MeshDev, LayerW<double> *, LayerG<double> *);
template __global__ void k_ghost_fill<float>(MeshDev, LayerW<float> *, LayerG<float> *);
template __global__ void k_speed<double>(MeshDev, Phys, const LayerW<double> *);
template __global__ void k_speed<float>(MeshDev, Phys, const LayerW<float> *);
}  // namespace gks
