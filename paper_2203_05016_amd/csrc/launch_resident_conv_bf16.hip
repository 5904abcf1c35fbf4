// Launchers of the slab kernel with a resident slab, bfloat16 operands, convolutions.
#define SHFLBW_LAUNCH_CONV 1
#define SHFLBW_LAUNCH_BF true
#define SHFLBW_LAUNCH_NAME run_resident_bf16
#define SHFLBW_LAUNCH_OUT16 __bf16
#include "launch_resident.inc"
