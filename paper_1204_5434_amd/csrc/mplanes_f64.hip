// The yz pass on the matrix cores, complex double.
#define PFT_MP_T double
#include "mplanes.inc"
