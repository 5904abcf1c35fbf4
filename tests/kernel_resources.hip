// The gather kernels whose residency tests/test_kernel_resources.py checks, instantiated for the compiler's report.
#include "gather_kernel.hip"

namespace shflbw {
#define GATHER(V, WN, WAVES, OutT, Geom, SPLIT) \
    template __global__ void shflbw_gather_kernel<V, WN, WAVES, 2, OutT, Geom, false, SPLIT>(PackedView, Geom, int, GatherOrder);
GATHER(32, 64, 8, _Float16, GeomLinearBuf, 1)
GATHER(64, 64, 8, _Float16, GeomLinearBuf, 1)
GATHER(64, 64, 8, float, GeomLinearBuf, 1)
GATHER(128, 64, 8, _Float16, GeomLinearBuf, 1)
GATHER(64, 64, 2, float, GeomLinearBuf, 2)
GATHER(128, 64, 2, _Float16, GeomRows, 2)
GATHER(64, 64, 8, _Float16, GeomConvRuns<false>, 1)
GATHER(64, 64, 2, _Float16, GeomConvRuns<false>, 2)
GATHER(64, 64, 4, _Float16, GeomConvRuns<false>, 4)
GATHER(64, 64, 4, float, GeomConvRuns<true>, 4)
GATHER(128, 64, 2, _Float16, GeomConvRuns<false>, 2)
GATHER(128, 64, 4, _Float16, GeomConvRuns<true>, 4)
}  // namespace shflbw
