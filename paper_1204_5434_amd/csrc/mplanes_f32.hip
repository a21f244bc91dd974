// The yz pass on the matrix cores, complex float.
#define PFT_MP_T float
#include "mplanes.inc"
