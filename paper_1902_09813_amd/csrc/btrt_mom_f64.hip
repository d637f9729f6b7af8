// Moment-form sweeps (btrt_mom.h) in F64 storage, instantiated in this
// translation unit alone.

#include "btrt_mom.h"

namespace btrtk {

hipError_t mom_f64(const SweepArgs<double>& a, int src_kind, int kmode, const LaunchCfg& cfg, hipStream_t s)
{
    return mom_sweep_with<double, 0>(a, src_kind, kmode, cfg, s);
}

LaunchCfg mom_resolve_f64(const SweepArgs<double>& a, int src_kind, int kmode, const LaunchCfg& cfg)
{
    return mom_resolve_with<double, 0>(a, src_kind, kmode, cfg);
}

}  // namespace btrtk
