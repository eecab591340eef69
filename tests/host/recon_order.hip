// the reconstruction's ways through its LDS: plain, indicator on and read back, wet/dry
#include "gks_kernels.h"

namespace gks {
#define INSTANCE(R, ...)                                                                                    \
    template __global__ void k_recon<R, __VA_ARGS__>(MeshDev, Phys, const LayerW<R> *, const LayerG<R> *, IndArgs, \
                                                     GpRecs<R>, R *, R *);
INSTANCE(double, 0, 0, 0)
INSTANCE(double, 1, 0, 0)
INSTANCE(double, 0, 0, 1)
INSTANCE(float, 0, 1, 0)
INSTANCE(float, 1, 0, 0)
INSTANCE(float, 2, 0, 0)
}  // namespace gks
