// Declarations shared by the translation units of libdlfp (not part of the ABI).
#ifndef DLFP_INTERNAL_H
#define DLFP_INTERNAL_H

#include "dlfp.h"

namespace dlfp {

// DLFP_OK if dims are supported; *group receives Hq / Hkv.
int check_dims(const dlfp_dims* dims, int* group);

// Workgroups of an attention launch that write `records` append records: about
// two records per wavefront, a multiple of 8; none past 16, where the records
// take a launch of their own first.  (At the start of the attention launch each
// append workgroup holds a slot of a compute unit, which pushes long prefill
// units to share compute units: on Qwen3-0.6B shapes chunks of 512-2048 prompt
// tokens took 15-20% longer in one launch, while chunks of 64-256 gained 6-8%
// per iteration from dropping the second launch.)  The split policy plans for
// the count that the launch uses.
inline int append_workgroups(int64_t records) {
  const int64_t wgs = records > 0 ? (records + 63) / 64 * 8 : 0;
  return wgs <= 16 ? (int)wgs : 0;
}

}  // namespace dlfp

#endif  // DLFP_INTERNAL_H
