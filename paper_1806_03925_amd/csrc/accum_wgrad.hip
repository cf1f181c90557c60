// The end of a short step but for its parameters, one launch: weight gradients, accumulation, embedding update.
#include "accum_device.hpp"
#include "tn_tile.hpp"

namespace gear {
namespace {

// The accumulation (accum.hip) beside the weight-gradient products, for a step in blocks of views whose products all go on small tiles: neither
// needs the other, and a launch less is 4 us of a step of 30 to 90 (512 views fp32 38 / 34 us a step,
// 4096 85.5 / 80.5, 5000 of one image 67 / 63.5, 1000 bf16 50.7 / 44.3).  The products' workgroups come first, they take longest; with three stages instead of
// four three workgroups fit on a CU, and the units, of which a workgroup then has several side by side, run between them.
template <typename GT> struct BesideTile;
template <> struct BesideTile<float> { using C = TnTile<float, 1, 1, 3>; };
template <> struct BesideTile<bf16_t> { using C = TnTile<bf16_t, 2, 2, 3>; };
struct BesideWork {
  RideWork ride;
  TnTileArgs tn;
  int tn_blocks, K, splits;
  int unit_threads;   // 64, 128 or 256
};
template <typename GT, bool PARTS>
__global__ void __launch_bounds__(256, 3)
k_accumulate_wgrad(AccumPlan plan, const GT *__restrict__ dx, int D, float *__restrict__ accum, int M, int32_t *__restrict__ ready_ids,
                   float *__restrict__ ready_grads, BesideWork w, const int32_t *__restrict__ status) {
  using C = typename BesideTile<GT>::C;
  static_assert(C::THREADS == 256, "one size of workgroup");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[C::STAGES * C::STAGE_BYTES];
  int block = blockIdx.x, blocks = gridDim.x;
  if (block < w.tn_blocks) return tn_tile<C>(w.tn, w.K, w.splits, nullptr, xcd_remap(block, w.tn_blocks), lds);   // into the workspace only
  block -= w.tn_blocks;
  blocks -= w.tn_blocks;
  LocalState local = {};
  if constexpr (PARTS) {
    local = local_state(plan.local, true);
    if (local.code != 0) return;
  } else {
    if (*status != 0) return;
  }
  if (chunks_ride(plan, w.ride, block)) return;
  block -= 2 * w.ride.blocks + w.ride.count_blocks;
  blocks -= 2 * w.ride.blocks + w.ride.count_blocks;
  const int side = 256 / w.unit_threads, which = __builtin_amdgcn_readfirstlane((int)threadIdx.x / w.unit_threads);
  accumulate_units<GT, true, PARTS>(plan, local, dx, D, accum, w.ride.w.counts, M, ready_ids, ready_grads, block * side + which, blocks * side,
                                    (int)threadIdx.x - which * w.unit_threads, w.unit_threads);
}

}  // namespace

// `emb`: level 1 of its update and the counters ride along
hipError_t launch_accumulate_wgrad(const gear_config &cfg, const GroupProblem &img, const AccumPlan &plan, const void *dx_dfv,
                                   float *grad_accum, int32_t M, int32_t *ready_ids, float *ready_grads, const EmbeddingWork &emb,
                                   const TnProblem *p, int count, int K, int splits, const int32_t *status, hipStream_t s) {
  if (count < 1 || count > GEAR_MAX_LAYERS || splits < 1 || !plan.row_at) return hipErrorInvalidValue;
  const int D = cfg.dfv_dim, threads = 256;
  BesideWork w;
  w.ride.w = emb;
  w.ride.lanes = embedding_lanes(emb.d);
  w.ride.blocks = (int)(((long long)embedding_chunks(emb) * w.ride.lanes + threads - 1) / threads);
  w.ride.count_blocks = (img.n + 4 * threads - 1) / (4 * threads);
  if (w.ride.count_blocks > 256) w.ride.count_blocks = 256;
  if (plan.local.parts) w.ride.count_blocks = 0;   // the units do
  w.ride.sum_blocks = 0;
  w.K = K;
  w.splits = splits;
  const bool bf16 = cfg.mlp_dtype == GEAR_BF16;
  const int edge = bf16 ? BesideTile<bf16_t>::C::BM : BesideTile<float>::C::BM;
  w.tn_blocks = tn_tile_args(p, count, edge, &w.tn) * splits;
  const int pieces = D / (bf16 ? 8 : 4);
  w.unit_threads = pieces <= 64 ? 64 : pieces <= 128 ? 128 : 256;
  const int side = threads / w.unit_threads;
  int units = (img.n + side - 1) / side;
  if (units > 32768) units = 32768;
  const dim3 grid((unsigned)(w.tn_blocks + 2 * w.ride.blocks + w.ride.count_blocks + units));
  if (bf16 && plan.local.parts) return hipErrorInvalidValue;
  if (bf16)
    hipLaunchKernelGGL((k_accumulate_wgrad<bf16_t, false>), grid, dim3(threads), 0, s, plan, (const bf16_t *)dx_dfv, D, grad_accum, M, ready_ids,
                       ready_grads, w, status);
  else if (plan.local.parts)
    hipLaunchKernelGGL((k_accumulate_wgrad<float, true>), grid, dim3(threads), 0, s, plan, (const float *)dx_dfv, D, grad_accum, M, ready_ids,
                       ready_grads, w, status);
  else
    hipLaunchKernelGGL((k_accumulate_wgrad<float, false>), grid, dim3(threads), 0, s, plan, (const float *)dx_dfv, D, grad_accum, M, ready_ids,
                       ready_grads, w, status);
  return hipGetLastError();
}

}  // namespace gear
