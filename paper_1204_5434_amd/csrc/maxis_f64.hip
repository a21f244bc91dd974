// Axis passes on the matrix cores, complex double.
#define PFT_MP_T double
#define PFT_MLINE_LIST PFT_MLINE_F64
#include "maxis.inc"
