// Short-range force adjoint in single precision (the kernels of pair.hip).
#define P3M_PAIR_PART 2
#include "pair.hip"
