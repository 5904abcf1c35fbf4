// Launchers of the slab kernel with a resident slab, binary16 operands, linear layers.
#define SHFLBW_LAUNCH_CONV 0
#define SHFLBW_LAUNCH_BF false
#define SHFLBW_LAUNCH_NAME run_resident_f16
#define SHFLBW_LAUNCH_OUT16 _Float16
#include "launch_resident.inc"
