// How the launches behind blocks of views read what the parts of a short step's image list have left (LocalResult).  Thousands of small
// workgroups do, so what each of them needs is one load of a part a lane, with the scalar loads of the codes beside it, and a sum over the lanes
// in registers: a unit is then found by its number, and every worker has as many whatever a part holds.  us a step of 96 ->
// 64, 4000 views, 19 000 ids, with a share of the workers for every part, whose units two scalar loads find / so: spread evenly, M = 4, 54.8 /
// 49.8; of Zipf 1.5 125 / 105; one image 90 / 71, M = 2 115 / 77; 19 000 images in one part of 32 205 / 131.
#pragma once

#include "gear_internal.hpp"

namespace gear {
namespace {

// For whole wavefronts: a lane has what belongs to its part.
struct LocalState {
  int code;           // what has gone wrong with the step (0: nothing), the same for all who ask
  int units, emits;   // of all parts
  int units_to;       // units of the parts up to the lane's, its own among them; all of them beyond the parts
  int place, slot;    // what the numbers of the part's units and emissions lack to their places
};

// lists: whether more than the code is wanted
__device__ __forceinline__ LocalState local_state(const LocalResult &local, bool lists) {
  static_assert(kMaxParts == 32, "two rows of lanes");
  const int lane = threadIdx.x & 63;
  lists = lists || local.ready_cap >= 0;
  int4 own = make_int4(0, 0, 0, 0);
  if (lists && lane < local.n_parts) own = reinterpret_cast<const int4 *>(local.parts)[lane];
  uint32_t bad = 0u;
  for (int g = 0; g < local.n_codes; g += kCodeGroup) {
    const uint32_t *w = reinterpret_cast<const uint32_t *>(local.codes + g);
#pragma unroll
    for (int k = 0; k < kCodeGroup / 4; ++k) bad |= w[k];
  }
  LocalState s = {};
  s.code = bad ? GEAR_ERR_RANGE : 0;
  if (!lists) return s;
  const int both = own.z | own.w << 16;   // a list has less than 65 536 ids
  int to = both;
  to += __builtin_amdgcn_mov_dpp(to, 0x111, 0xf, 0xf, true);   // from one lane lower, in a row of sixteen
  to += __builtin_amdgcn_mov_dpp(to, 0x112, 0xf, 0xf, true);   // two
  to += __builtin_amdgcn_mov_dpp(to, 0x114, 0xf, 0xf, true);
  to += __builtin_amdgcn_mov_dpp(to, 0x118, 0xf, 0xf, true);
  const int first_row = __builtin_amdgcn_readlane(to, 15);
  if (lane >= 16) to += first_row;
  const uint32_t all = (uint32_t)__builtin_amdgcn_readlane(to, kMaxParts - 1);
  s.units = (int)(all & 0xffffu), s.emits = (int)(all >> 16);
  s.units_to = to & 0xffff;
  s.place = own.x - ((to - both) & 0xffff);
  s.slot = (int)((uint32_t)(to - both) >> 16);
  if (!s.code && local.ready_cap >= 0 && s.emits > local.ready_cap) s.code = GEAR_ERR_CAPACITY;
  return s;
}

// the part that unit `i` of all lies in
__device__ __forceinline__ int part_of_unit(const LocalState &s, int i) { return __popc((uint32_t)__ballot(s.units_to <= i)); }

}  // namespace
}  // namespace gear
