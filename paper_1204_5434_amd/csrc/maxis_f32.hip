// Axis passes on the matrix cores, complex float.
#define PFT_MP_T float
#define PFT_MLINE_LIST PFT_MLINE_F32
#include "maxis.inc"
