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

// Whether the decode units are each the work of a workgroup, else of a
// wavefront.  Without prefill units: of a workgroup, but for units of at most 192
// keys that are more than the resident workgroups (two per compute unit) and all
// resident as wavefronts (eight): a workgroup is then mostly its start and its sum
// (114 decoders of 29-58 keys, g = 2, 912 units: 9.0 us, a workgroup of four
// wavefronts each 11.1; 116 of 16 keys: 9.0 and 12.3; 70 of 138 keys: 14.0 and
// 17.8; from 200 keys on, at fewer units and in more than one round workgroups
// are as fast or faster, 217 decoders of 23 keys, 3472 units, 29.0 and 48.6).
// Beside prefill units: when all workgroups fit the resident slots of the device
// even with a workgroup to each unit, each gets one: the launch is short and its
// end, where a wavefront's unit streams alone at a quarter of what the compute
// unit could take, is most of it (g = 8, 6 decoders of 250-2000 keys beside 47
// new tokens: 18.9 -> 11.8 us; g = 4, 10 of 442-3536 beside 2: 21.7 -> 17.8 us).
// Not for units of up to 128 keys, one step of a workgroup, which the built-in
// split makes where the prefill share sets the launch time (11 decoders of 38-304
// keys beside 796 tokens over 858, g = 2: 34.8 us, a workgroup each 35.3 us).  The two round their probabilities
// against different reference maxima, so the rule takes only what the metadata
// holds: the append records count also where another call writes them, and the
// one- and two-launch forms give equal bits.
inline bool decode_by_workgroup(const dlfp_meta& m, int64_t compute_units) {
  if (m.num_prefill_units == 0)
    return m.num_units <= 2 * compute_units || m.num_units > 8 * compute_units ||
           m.decode_split_tokens > 192;
  return (int64_t)m.num_units + append_workgroups(m.num_append) <= 2 * compute_units &&
         m.decode_split_tokens > 128;
}

}  // namespace dlfp

#endif  // DLFP_INTERNAL_H
