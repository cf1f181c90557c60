// Slowgear-side gradient bookkeeping and the DFV cache refresh.
//
// Section 3, step 5: every occurrence of an image in a page view yields (image id, dLoss/dDFV);
// with mean pooling that gradient is dLoss/dx of the view's DFV slot divided by the view's image
// count (Eq. 1, left factor).  For a bf16 MLP that slot is kept in bf16 like every other delta of the
// network; sums, accumulators and emitted averages are fp32.  Section 1, third point and Section 3, step 6: all gradients of an
// image are kept until M have arrived; their average is then handed on and collecting starts
// afresh.  Keeping the running sum of an unfinished group in grad_accum[image] is the same thing
// as keeping the gradients themselves, because only their sum is ever used.
//
// Work is cut into units of at most M rows (see the plan in group.hip), one workgroup per unit,
// rows added in arrival order (flat CSR order continuing the earlier steps): no float atomics.
#include "accum_device.hpp"
#include "block_sums.hpp"

namespace gear {
namespace {

// dx: the DFV slot of dLoss/dx, [B x D].  One workgroup per unit, D / Cols<GT>::N threads.
// kChunks needs 132 registers where the units alone take 44: three wavefronts a SIMD, which still have 72 KB of rows in
// flight on a CU, as much as a memory latency asks for.  kSpans has eight partials of a long run in flight: 59 (with 32
// in flight 138).
template <typename GT, int RIDE, bool AT>
__global__ void __launch_bounds__(256, RIDE >= kChunks ? 3 : 1)
k_accumulate(AccumPlan plan, const GT *__restrict__ dx, int D, float *__restrict__ accum, int M,
             int32_t *__restrict__ ready_ids, float *__restrict__ ready_grads, std::conditional_t<RIDE == kNoRide, NoWork, RideWork> emb,
             std::conditional_t<RIDE == kChunksAndSums, BlockSums, NoWork> sums, const int32_t *__restrict__ status) {
  if (*status != 0) return;
  int block = blockIdx.x, blocks = gridDim.x;
  if constexpr (RIDE == kSpans) {
    if (block < 2 * emb.blocks) {
      const int second = block >= emb.blocks ? 1 : 0;
      const int chunk = (block - second * emb.blocks) * (blockDim.x / kWave) + threadIdx.x / kWave;
      if (emb.w.bf16)
        embedding_span<bf16_t, 8>(emb.w.table[second], chunk, emb.w.d, emb.w.opt);
      else
        embedding_span<float, 8>(emb.w.table[second], chunk, emb.w.d, emb.w.opt);
      return;
    }
    block -= 2 * emb.blocks;
    blocks -= 2 * emb.blocks;
  }
  if constexpr (RIDE >= kChunks) {
    if (chunks_ride(plan, emb, block)) return;
    block -= 2 * emb.blocks + emb.count_blocks;
    blocks -= 2 * emb.blocks + emb.count_blocks;
  }
  if constexpr (RIDE == kChunksAndSums) {
    if (block < emb.sum_blocks) return block_sums<GT>(sums, block * blockDim.x + threadIdx.x);
    block -= emb.sum_blocks;
    blocks -= emb.sum_blocks;
  }
  accumulate_units<GT, AT, false>(plan, LocalState{}, dx, D, accum, nullptr, M, ready_ids, ready_grads, block, blocks, threadIdx.x, blockDim.x);
}

// dfv_cache[ids[r]] = rows[r]; one wavefront per row, 16-byte pieces
__global__ void __launch_bounds__(256) k_refresh(uint4 *__restrict__ cache, int64_t n_images, int vec_per_row,
                                                 const int32_t *__restrict__ ids, const uint4 *__restrict__ rows,
                                                 int64_t n, int32_t *status, const int32_t *__restrict__ n_dev) {
  if (n_dev) n = min((int64_t)max(*n_dev, 0), n);  // the row count is only known on the device
  const int lane = threadIdx.x & 63;
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
  for (int64_t r = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; r < n; r += waves) {
    const int64_t id = ids ? (int64_t)ids[r] : r;
    if (id < 0 || id >= n_images) {
      if (status && lane == 0) atomicCAS(status, 0, GEAR_ERR_RANGE);
      continue;
    }
    for (int v = lane; v < vec_per_row; v += kWave) cache[id * vec_per_row + v] = rows[r * vec_per_row + v];
  }
}

}  // namespace

// emb (may be NULL): level 1 of its update and the counters, or level 2 if `level2`, ride along
hipError_t launch_accumulate(const gear_config &cfg, const GroupProblem &img, const AccumPlan &plan,
                             const void *dx_dfv, float *grad_accum, int32_t M, int32_t *ready_ids,
                             float *ready_grads, const EmbeddingWork *emb, bool level2, const BlockSums *sums, const int32_t *status,
                             hipStream_t s, hipEvent_t stop) {
  if (img.n <= 0 && !emb) return leave(stop, s);
  const int D = cfg.dfv_dim;
  const int cols = cfg.mlp_dtype == GEAR_BF16 ? 8 : 4;
  int threads = ((D / cols + 63) / 64) * 64;
  if (threads > 256) threads = 256;
  int blocks = img.n < 32768 ? img.n : 32768;
  RideWork work;
  if (emb) {
    work.w = *emb;
    work.lanes = level2 ? kWave : embedding_lanes(emb->d);
    work.blocks = (int)(((long long)embedding_chunks(*emb) * work.lanes + threads - 1) / threads);
    work.count_blocks = level2 ? 0 : (img.n + 4 * threads - 1) / (4 * threads);
    if (work.count_blocks > 256) work.count_blocks = 256;
    work.sum_blocks = sums ? (int)((block_sums_threads(*sums) + threads - 1) / threads) : 0;
    blocks += 2 * work.blocks + work.count_blocks + work.sum_blocks;
  }
  if ((sums && (!emb || level2 || plan.row_at)) || plan.local.parts) return hipErrorInvalidValue;
#define GEAR_ACC(T, R, AT, EMB, SUMS)                                                                                            \
  launch_leaving(stop, k_accumulate<T, R, AT>, dim3(blocks), threads, 0, s, plan, (const T *)dx_dfv, D, grad_accum, M, ready_ids, \
                 ready_grads, EMB, SUMS, status)
#define GEAR_ACC_T(T)              \
  if (!emb)                        \
    GEAR_ACC(T, kNoRide, false, NoWork{}, NoWork{}); \
  else if (level2)                 \
    GEAR_ACC(T, kSpans, false, work, NoWork{}); \
  else if (sums)                   \
    GEAR_ACC(T, kChunksAndSums, false, work, *sums); \
  else if (plan.row_at)            \
    GEAR_ACC(T, kChunks, true, work, NoWork{}); \
  else                             \
    GEAR_ACC(T, kChunks, false, work, NoWork{})
  if (cfg.mlp_dtype == GEAR_BF16) {
    GEAR_ACC_T(bf16_t);
  } else {
    GEAR_ACC_T(float);
  }
#undef GEAR_ACC_T
#undef GEAR_ACC
  return hipGetLastError();
}

hipError_t launch_refresh(int dtype, void *dfv_cache, int64_t n_images, int dim, const int32_t *ids,
                          const void *rows, int64_t n, int32_t *status, hipStream_t s, const int32_t *n_dev) {
  if (n <= 0) return hipSuccess;
  const int vec_per_row = (int)((size_t)dim * dtype_bytes(dtype) / 16);
  int64_t want = (n + 3) / 4;
  const int blocks = (int)(want < 16384 ? want : 16384);
  hipLaunchKernelGGL(k_refresh, dim3(blocks), dim3(256), 0, s, (uint4 *)dfv_cache, n_images, vec_per_row, ids,
                     (const uint4 *)rows, n, status, n_dev);
  return hipGetLastError();
}

}  // namespace gear
