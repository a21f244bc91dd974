// Matrix-core passes, complex double.
#define PFT_MP_T double
#define PFT_MPLANE_LIST PFT_MPLANE_F64
#define PFT_MX_LIST PFT_MX_F64
#include "mplanes.inc"
