// raycast_ea.hip -- ray-casting kernel instances of the emission-absorption model
// (every voxel type, channel count, kernel flavour and statistics mode).
#include "raycast_kernels.h"

namespace sg {

const void* raycast_kernel_absorption(int bpv, int channels, bool stats, bool gather,
                                      bool loop, bool mb) {
  return model_kernel<kModelAbsorption>(bpv, channels, stats, gather, loop, mb);
}

const void* raycast_kernel_split(int bpv, bool mb) {
  if (bpv == 1)
    return mb ? reinterpret_cast<const void*>(raycast_gather_split<uint8_t, true>)
              : reinterpret_cast<const void*>(raycast_gather_split<uint8_t, false>);
  return mb ? reinterpret_cast<const void*>(raycast_gather_split<uint16_t, true>)
            : reinterpret_cast<const void*>(raycast_gather_split<uint16_t, false>);
}

}  // namespace sg
