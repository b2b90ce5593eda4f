// One instantiation of the C ABI bodies: compiled once per (lattice, precision,
// variant) with LBM_INSTANTIATE_Q, _QS, _REAL and _V defined (see build.py).
#include "ops.hpp"

namespace lbmh {

using TheOps = Ops<LBM_INSTANTIATE_Q, LBM_INSTANTIATE_QS, LBM_INSTANTIATE_REAL, LBM_INSTANTIATE_V>;
template struct RunPrimal<TheOps>;
template struct RunObjective<TheOps>;
template struct RunAdjoint<TheOps>;
template struct RunReset<TheOps>;
template struct RunSetState<TheOps>;
template struct RunGradient<TheOps>;
template struct RunGradientPenalty<TheOps>;
template struct RunFields<TheOps>;
template struct RunGetState<TheOps>;
template struct RunGetAdjoint<TheOps>;
template struct RunMaps<TheOps>;
template struct RunSetDesign<TheOps>;
template struct RunOneshot<TheOps>;
template struct RunGetDesign<TheOps>;
template struct RunWriteStatic<TheOps>;
template struct RunPrimalBatch<TheOps>;
template struct RunAdjointBatch<TheOps>;

}  // namespace lbmh
