// Axis passes on the matrix cores, complex float.
#define PFT_MP_T float
#define PFT_MX_LIST PFT_MX_F32
#define PFT_MZ_LIST PFT_MZ_F32
#define PFT_MWALL_LIST PFT_MWALL_F32
#include "maxis.inc"
