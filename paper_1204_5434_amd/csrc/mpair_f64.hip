// The yz pass of uneven and walled planes on the matrix cores, complex double.
#define PFT_MP_T double
#include "mpair.inc"
