// Matrix-core passes, complex float.
#define PFT_MP_T float
#define PFT_MPLANE_LIST PFT_MPLANE_F32
#define PFT_MX_LIST PFT_MX_F32
#include "mplanes.inc"
