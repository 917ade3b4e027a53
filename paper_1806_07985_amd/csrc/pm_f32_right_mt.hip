// The FP32 partial-MTTKRP kernels (pm_f32_body.hpp) of the right side, several M tiles per group.
#include "pm_f32_body.hpp"

namespace nncpk {
template const void* pm_f32_form<1, true>(int, int, bool);
}  // namespace nncpk
