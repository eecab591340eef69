#include "gks_indicator.h"

namespace gks {
template __global__ void k_features<double>(MeshDev, double, const LayerW<double> *, const LayerG<double> *, float *);
template __global__ void k_features<float>(MeshDev, double, const LayerW<float> *, const LayerG<float> *, float *);
}  // namespace gks
