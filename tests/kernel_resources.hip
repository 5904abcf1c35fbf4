// The gather kernels whose residency tests/test_kernel_resources.py checks, instantiated for the compiler's report.
#include "gather_kernel.hip"

namespace shflbw {
#define GATHER(V, WN, WAVES, OutT, Geom, SPLIT) \
    template __global__ void shflbw_gather_kernel<V, WN, WAVES, 2, OutT, Geom, false, SPLIT>(PackedView, Geom, int, GatherOrder);
GATHER(32, 64, 8, _Float16, GeomLinearBuf, 1)
GATHER(64, 64, 8, _Float16, GeomLinearBuf, 1)
GATHER(64, 64, 8, float, GeomLinearBuf, 1)
GATHER(128, 64, 8, _Float16, GeomLinearBuf, 1)
}  // namespace shflbw
