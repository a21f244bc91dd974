// The yz pass on the matrix cores, complex double.
#define PFT_MP_T double
#define PFT_MPLANE_LIST PFT_MPLANE_F64
#include "mplanes.inc"
