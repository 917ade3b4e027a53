// The FP32 partial-MTTKRP kernels (pm_f32_body.hpp) of the left side, one M tile per group.
#include "pm_f32_body.hpp"

namespace nncpk {
template const void* pm_f32_form<0, false>(int, int, bool);
}  // namespace nncpk
