// The master problem with one wave per signal: see launch rules in api.hip and master_body.h.
#include <float.h>
#include <limits.h>

#include <type_traits>

#include "../../include/bmpl.h"
#include "bmpl_internal.h"
#include "pursuit.h"
#include "wave_ops.h"

namespace bmpl {
namespace {
constexpr int NT = 64;
}  // namespace
}  // namespace bmpl

#include "master_body.h"

namespace bmpl {

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void solve_wave_kernel(SolveArgs a) { solve_body<false, false, 1>(a); }

}  // namespace bmpl
