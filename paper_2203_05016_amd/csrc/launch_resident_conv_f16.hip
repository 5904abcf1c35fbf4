// Launchers of the slab kernel with a resident slab, binary16 operands, convolutions.
#define SHFLBW_LAUNCH_CONV 1
#define SHFLBW_LAUNCH_BF false
#define SHFLBW_LAUNCH_NAME run_resident_f16
#define SHFLBW_LAUNCH_OUT16 _Float16
#include "launch_resident.inc"
