// What the two launches that finish an embedding update share: the tables, and the second level of its sums (update.hip).
#pragma once

#include "gear_internal.hpp"

namespace gear {
namespace {

constexpr int kChunk = 16;

struct EmbeddingTable {
  const int32_t *keys;   // sorted ids
  const int32_t *perm;   // batch position of each sorted position
  int n;
  void *rows;            // embedding table
  int col0;              // first column of this table's slice inside a dx row
  float *part_first;     // [chunks x d] partial of a run that began in an earlier chunk
  float *part_last;      // [chunks x d] partial of a run that begins here and goes on
  Moments mom;           // Adam: fp32 moment tables of the same shape as `rows` (only touched rows move)
};

// level 2: one wavefront per chunk; if a border-crossing run starts in this chunk the wave adds
// the run's partials in chunk order (lane = column) and writes the row; AHEAD partials in flight
template <typename ET, int AHEAD>
__device__ __forceinline__ void embedding_span(const EmbeddingTable &t, int chunk, int d, const Optim &opt) {
  const int lane = threadIdx.x & 63;
  const int q_begin = chunk * kChunk;
  if (q_begin >= t.n) return;
  const int q_last = min(t.n, q_begin + kChunk) - 1;
  if (q_last + 1 >= t.n) return;              // nothing after this chunk
  const int key = t.keys[q_last], next = t.keys[q_last + 1], previous = q_begin > 0 ? t.keys[q_begin - 1] : -1;
  if (next != key) return;                    // the last run ends inside this chunk
  if (previous == key) return;                // the run began in an earlier chunk: not ours
  const int s1 = wave_search(t.keys, q_last + 1, t.n, key, true, lane);   // where the run ends
  const int k_last = (s1 - 1) / kChunk;
  for (int c = lane; c < d; c += kWave) {
    float sum = t.part_last[(size_t)chunk * d + c];
    int k = chunk + 1;
    for (; k + AHEAD <= k_last + 1; k += AHEAD) {   // added in order, requested together
      float v[AHEAD];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) v[i] = t.part_first[(size_t)(k + i) * d + c];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) sum += v[i];
    }
    for (; k <= k_last; ++k) sum += t.part_first[(size_t)k * d + c];
    const size_t at = (size_t)key * d + c;
    ET *cell = static_cast<ET *>(t.rows) + at;
    *cell = from_f32<ET>(optim_apply(opt, to_f32<ET>(*cell), sum, t.mom.m + at, t.mom.v + at));
  }
}


}  // namespace

// both tables of a step; the partials of either lie in `partials`
inline void embedding_tables(const gear_config &cfg, const GroupProblem &users, const GroupProblem &urls, void *user_emb,
                             void *url_emb, float *partials, const Moments &mom_user, const Moments &mom_url,
                             EmbeddingTable *tu, EmbeddingTable *tl) {
  const int d = cfg.emb_dim;
  const size_t per = (size_t)((cfg.max_batch + kChunk - 1) / kChunk) * d;
  *tu = {users.sorted_keys, users.perm, users.n, user_emb, 0, partials, partials + per, mom_user};
  *tl = {urls.sorted_keys, urls.perm, urls.n, url_emb, d, partials + 2 * per, partials + 3 * per, mom_url};
}

}  // namespace gear
