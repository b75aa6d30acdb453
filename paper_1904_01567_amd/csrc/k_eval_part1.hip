// Evaluation kernels of every fourth padded dwell count, compiled apart from
// the others so that the parts build in parallel.
#define GMCO_EVAL_PART 1
#include "k_eval.hip"
