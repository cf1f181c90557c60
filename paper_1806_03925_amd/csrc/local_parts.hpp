// How the launches behind blocks of views read what the parts of a short step's image list have left (LocalResult).  Thousands of small
// workgroups do, so what each of them needs is two scalar loads side by side, and it takes units of one part alone; emissions of the
// lower parts are added up by those that emit.
#pragma once

#include "gear_internal.hpp"

namespace gear {
namespace {

struct LocalState {
  int code;                 // what has gone wrong with the step (0: nothing), the same for all who ask
  int part, below, units;   // the part asked for
};

// sum over the lower `parts` parts' emissions; by whole wavefronts
__device__ __forceinline__ int emits_of(const LocalResult &local, int parts) {
  static_assert(kMaxParts == 32, "two rows of lanes");
  const int lane = threadIdx.x & 63;
  int v = lane < parts ? local.parts[lane].emits : 0;
  v += __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);    // lane ^ 1
  v += __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true);    // lane ^ 2
  v += __builtin_amdgcn_mov_dpp(v, 0x124, 0xf, 0xf, true);   // four lanes on, in a row of sixteen
  v += __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true);   // eight
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16);
}

__device__ __forceinline__ LocalState local_state(const LocalResult &local, int part) {   // `part` the same in a wavefront
  LocalState s;
  const int4 own = reinterpret_cast<const int4 *>(local.parts)[part];
  s.part = part, s.below = own.x, s.units = own.z;
  uint32_t bad = 0u;
  for (int g = 0; g < local.n_codes; g += kCodeGroup) {
    const uint32_t *w = reinterpret_cast<const uint32_t *>(local.codes + g);
#pragma unroll
    for (int k = 0; k < kCodeGroup / 4; ++k) bad |= w[k];
  }
  asm volatile("" ::"s"(s.below), "s"(s.units));   // here, beside the others, not behind the branch that looks at `code`
  s.code = bad ? GEAR_ERR_RANGE : 0;
  if (local.ready_cap >= 0 && !s.code && emits_of(local, local.n_parts) > local.ready_cap) s.code = GEAR_ERR_CAPACITY;
  return s;
}

}  // namespace
}  // namespace gear
