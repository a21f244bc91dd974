// The yz pass of uneven and walled planes on the matrix cores, complex float.
#define PFT_MP_T float
#include "mpair.inc"
