// The yz pass on the matrix cores, complex float.
#define PFT_MP_T float
#define PFT_MPLANE_LIST PFT_MPLANE_F32
#include "mplanes.inc"
