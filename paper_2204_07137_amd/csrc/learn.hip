// The learning-episode update kernels (actor and critic Adam, TD-lambda, critic fit, target
// critic) and the policy-parameter gradient, which shares their MLP kernels, in FP32 and FP64.
#include <hip/hip_runtime.h>
#include <math.h>
#include <type_traits>
#include "sim_types.h"

namespace sim_l32 {
typedef float real;
#include "sim_math.h"
#include "sim_gemm.h"
#include "sim_layers.h"
#include "sim_learn.h"
}  // namespace sim_l32

namespace sim_l64 {
typedef double real;
#include "sim_math.h"
#include "sim_gemm.h"
#include "sim_layers.h"
#include "sim_learn.h"
}  // namespace sim_l64
