// Axis passes on the matrix cores, complex double.
#define PFT_MP_T double
#define PFT_MX_LIST PFT_MX_F64
#define PFT_MZ_LIST PFT_MZ_F64
#define PFT_MWALL_LIST PFT_MWALL_F64
#include "maxis.inc"
