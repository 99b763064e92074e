// The LDS-staged forward kernel for long tables once more, for spline degrees 4 and 5 (window of six rows).
#define KAN_MAXK 6
#define KAN_NS kan_k5
#include "kan_lds_rows.hip"
