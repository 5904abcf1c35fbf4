// Gather-kernel launchers for binary16 operands, NCHW convolutions with a stride of two along x, 16-bit results.
#define SHFLBW_LAUNCH_CONV 2
#define SHFLBW_LAUNCH_BF false
#define SHFLBW_LAUNCH_NAME run_gather_f16
#define SHFLBW_LAUNCH_OUT16 _Float16
#include "launch_gather.inc"
