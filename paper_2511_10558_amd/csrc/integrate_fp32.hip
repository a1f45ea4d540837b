// The persistent integration of the FP32-factorisation form.
#include "integrate_kernels.hpp"

namespace abdf {

Persistent integrate_wide_fp32(const DeviceNet &n) { return integrate_wide<true>(n); }

}  // namespace abdf
