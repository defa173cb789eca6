// Short-range pair sum in double precision (the kernels of pair.hip).
#define P3M_PAIR_PART 1
#include "pair.hip"
