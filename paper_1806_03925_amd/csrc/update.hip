// SGD on the touched embedding rows (Section 3, step 4: the Fastgear Worker applies the Sparse
// Part's gradients every step).
//
// The gradient of a row is the sum of dLoss/dx over the views that used it.  After the stable
// sort by id those views are a run of the sorted positions, ascending in batch position.  Zipf
// traffic makes a few runs thousands of views long, so the sum has a fixed two-level shape that
// depends on the data only, never on scheduling: the sorted positions are cut into chunks of kChunk
// and a worker adds the rows of its chunk run by run, in order.  A run that lies inside one
// chunk is finished on the spot (one read-modify-write of the row).  A run that crosses chunk
// borders leaves one partial per chunk; the worker of the chunk where the run starts then adds
// those partials in chunk order and writes the row.  No atomics anywhere.
//
// A worker is d/4 lanes, each owning one float4 column group of the row.
//
// Beside a long dLoss/dx product both levels run on the helper stream in launches of their own, the image counters with
// them: there they cost nothing (in k_accumulate, which is bound by memory, the counters' scattered words were 7 us of a
// step of 65 536 views).  In a shorter step level 2 rides with the accumulation, or, on one stream, level 1 and the
// counters with the accumulation and level 2 with the parameter update.
#include "embedding_common.hpp"

namespace gear {
namespace {

template <typename ET>
__global__ void __launch_bounds__(256) k_embedding_chunks(EmbeddingWork w, int lanes, const int32_t *__restrict__ status) {
  if (*status != 0) return;
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  if (blockIdx.y == 2)
    count_images(w.plan, w.counts, tid, gridDim.x * blockDim.x);
  else
    embedding_chunk<ET, 8>(w.table[blockIdx.y], tid, w.dx, 2 * w.d, w.d, lanes, w.opt);
}

template <typename ET>
__global__ void __launch_bounds__(256) k_embedding_spans(EmbeddingWork w, const int32_t *__restrict__ status) {
  if (*status != 0) return;
  embedding_span<ET, 32>(w.table[blockIdx.y], blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave, w.d, w.opt);
}

}  // namespace

EmbeddingWork embedding_work(const gear_config &cfg, const GroupProblem &users, const GroupProblem &urls, const float *dx,
                             void *user_emb, void *url_emb, float *partials, const Optim &opt, const Moments &mom_user,
                             const Moments &mom_url, const AccumPlan &plan, int32_t *counts) {
  const int d = cfg.emb_dim;
  const size_t per = (size_t)((cfg.max_batch + kChunk - 1) / kChunk) * d;
  EmbeddingWork w;
  w.table[0] = {users.sorted_keys, users.perm, users.n, user_emb, 0, partials, partials + per, mom_user};
  w.table[1] = {urls.sorted_keys, urls.perm, urls.n, url_emb, d, partials + 2 * per, partials + 3 * per, mom_url};
  w.dx = dx;
  w.d = d;
  w.bf16 = cfg.emb_dtype == GEAR_BF16;
  w.opt = opt;
  w.plan = plan;
  w.counts = counts;
  return w;
}

// level 1 and the counters of the images, and with `both_levels` what is left of the update
hipError_t launch_embedding_update(const EmbeddingWork &w, bool both_levels, const int32_t *status, hipStream_t s) {
  const int lanes = embedding_lanes(w.d), chunks = embedding_chunks(w);
  const dim3 grid((unsigned)(((long long)chunks * lanes + 255) / 256), 3), grid2((chunks + 3) / 4, 2);
  if (w.bf16) {
    hipLaunchKernelGGL(k_embedding_chunks<bf16_t>, grid, dim3(256), 0, s, w, lanes, status);
    if (both_levels) hipLaunchKernelGGL(k_embedding_spans<bf16_t>, grid2, dim3(256), 0, s, w, status);
  } else {
    hipLaunchKernelGGL(k_embedding_chunks<float>, grid, dim3(256), 0, s, w, lanes, status);
    if (both_levels) hipLaunchKernelGGL(k_embedding_spans<float>, grid2, dim3(256), 0, s, w, status);
  }
  return hipGetLastError();
}

size_t embedding_partial_floats(const gear_config &cfg) {
  return 4 * (size_t)((cfg.max_batch + kChunk - 1) / kChunk) * cfg.emb_dim;
}

}  // namespace gear
