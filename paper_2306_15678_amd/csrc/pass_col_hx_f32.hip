// Half-exchange column-pass kernels, float instantiation (compiled as its
// own unit, so that the other column kernels are built without them).
#include "pass_kernels.hpp"

namespace ssfm {

template <typename R, class P, int KIND>
hipError_t launch_hx(const PassArgs<R>& a, hipStream_t s, const LaunchEv* ev) {
  if constexpr (!P::HX)
    return hipErrorInvalidValue;
  else
    return launch_built<R, P, KIND>(a, s, ev);
}

#define SSFM_HX_INST(NN, VV, ...)                                                               \
  template hipError_t launch_hx<float, ColPlanSel<NN, VV>::P, COL_FWD>(                         \
      const PassArgs<float>&, hipStream_t, const LaunchEv*);                                    \
  template hipError_t launch_hx<float, ColPlanSel<NN, VV>::P, COL_ADJ>(                         \
      const PassArgs<float>&, hipStream_t, const LaunchEv*);                                    \
  template hipError_t launch_hx<float, ColPlanSel<NN, VV>::P, COL_INV>(                         \
      const PassArgs<float>&, hipStream_t, const LaunchEv*);                                    \
  template hipError_t launch_hx<float, ColPlanSel<NN, VV>::P, COL_FD>(                          \
      const PassArgs<float>&, hipStream_t, const LaunchEv*);
SSFM_COL_PLANS(SSFM_HX_INST)
#undef SSFM_HX_INST

}  // namespace ssfm
