// Short-range force adjoint in double precision (the kernels of pair.hip).
#define P3M_PAIR_PART 3
#include "pair.hip"
