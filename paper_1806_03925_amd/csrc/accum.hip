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
#include "embedding_common.hpp"
#include "tn_tile.hpp"

namespace gear {
namespace {

// A thread owns kCols<GT> consecutive columns: 16 bytes of a dLoss/dx row (4 fp32 or 8 bf16 values),
// kept as loaded until they are added.
template <typename GT> struct Cols;
template <> struct Cols<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void widen(const uint4 &t, float (&v)[4]) {
    v[0] = __uint_as_float(t.x), v[1] = __uint_as_float(t.y), v[2] = __uint_as_float(t.z), v[3] = __uint_as_float(t.w);
  }
};
template <> struct Cols<bf16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void widen(const uint4 &t, float (&v)[8]) {
    v[0] = __uint_as_float(t.x << 16), v[1] = __uint_as_float(t.x & 0xffff0000u);
    v[2] = __uint_as_float(t.y << 16), v[3] = __uint_as_float(t.y & 0xffff0000u);
    v[4] = __uint_as_float(t.z << 16), v[5] = __uint_as_float(t.z & 0xffff0000u);
    v[6] = __uint_as_float(t.w << 16), v[7] = __uint_as_float(t.w & 0xffff0000u);
  }
};

template <int N> __device__ __forceinline__ void load_f32(const float *p, float (&v)[N]) {
#pragma unroll
  for (int k = 0; k < N; k += 4) {
    const float4 t = *reinterpret_cast<const float4 *>(p + k);
    v[k] = t.x, v[k + 1] = t.y, v[k + 2] = t.z, v[k + 3] = t.w;
  }
}
template <int N> __device__ __forceinline__ void store_f32(float *p, const float (&v)[N], float scale) {
#pragma unroll
  for (int k = 0; k < N; k += 4)
    *reinterpret_cast<float4 *>(p + k) = make_float4(v[k] * scale, v[k + 1] * scale, v[k + 2] * scale, v[k + 3] * scale);
}
template <int N> __device__ __forceinline__ void store_div(float *p, const float (&v)[N], float by) {
#pragma unroll
  for (int k = 0; k < N; k += 4)
    *reinterpret_cast<float4 *>(p + k) = make_float4(v[k] / by, v[k + 1] / by, v[k + 2] / by, v[k + 3] / by);
}

// Rows a thread has in flight.  Six keep the kernel within 48 registers per lane, so that three of
// its wavefronts (not two) fit on a SIMD beside the two of a weight-gradient product; alone on the
// device it is as fast with six as with eight.
constexpr int kRowsInFlight = 6;

// acc += sum over sorted positions [qa, qb) of dx[view(q)][col ..] / n_view, in order; kRowsInFlight rows in flight
template <typename GT>
__device__ __forceinline__ void add_rows(float (&acc)[Cols<GT>::N], const int32_t *__restrict__ row_view,
                                         const float *__restrict__ row_scale, const GT *__restrict__ col, int D,
                                         int qa, int qb) {
  constexpr int N = Cols<GT>::N;
  for (int q = qa; q < qb; q += kRowsInFlight) {
    int view[kRowsInFlight];
    float scale[kRowsInFlight];
#pragma unroll
    for (int i = 0; i < kRowsInFlight; ++i) {
      const bool in = q + i < qb;
      view[i] = in ? row_view[q + i] : -1;
      scale[i] = in ? row_scale[q + i] : 0.0f;
    }
    uint4 raw[kRowsInFlight];
#pragma unroll
    for (int i = 0; i < kRowsInFlight; ++i)
      raw[i] = view[i] >= 0 ? *reinterpret_cast<const uint4 *>(col + (size_t)view[i] * D) : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int i = 0; i < kRowsInFlight; ++i) {
      float v[N];
      Cols<GT>::widen(raw[i], v);
#pragma unroll
      for (int k = 0; k < N; ++k) acc[k] += v[k] * scale[i];
    }
  }
}

// The same where the sorted order only says which position of the batch comes next (AccumPlan::row_at): a chain of three
// loads.  The places are fetched two batches of rows ahead and the views one, so that a long group waits for its rows only
// (one image in most of 17 000 occurrences: a step of 2000 views took 97 us with the loads one after the other).
template <typename GT>
__device__ __forceinline__ void add_rows_at(float (&acc)[Cols<GT>::N], const AccumPlan &plan, const GT *__restrict__ col, int D, int qa,
                                            int qb) {
  constexpr int N = Cols<GT>::N, R = kRowsInFlight;
  if (qa >= qb) return;
  int at[R], view[R];
  float scale[R];
#pragma unroll
  for (int i = 0; i < R; ++i) at[i] = plan.row_at[min(qa + i, qb - 1)];
#pragma unroll
  for (int i = 0; i < R; ++i) view[i] = plan.row_view[at[i]], scale[i] = plan.row_scale[at[i]];
#pragma unroll
  for (int i = 0; i < R; ++i) at[i] = plan.row_at[min(qa + R + i, qb - 1)];
  for (int q = qa; q < qb; q += R) {
    uint4 raw[R];
    float by[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      raw[i] = *reinterpret_cast<const uint4 *>(col + (size_t)view[i] * D);
      by[i] = scale[i];
    }
    if (q + R < qb) {
#pragma unroll
      for (int i = 0; i < R; ++i) view[i] = plan.row_view[at[i]], scale[i] = plan.row_scale[at[i]];
#pragma unroll
      for (int i = 0; i < R; ++i) at[i] = plan.row_at[min(q + 2 * R + i, qb - 1)];
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (q + i < qb) {
        float v[N];
        Cols<GT>::widen(raw[i], v);
#pragma unroll
        for (int k = 0; k < N; ++k) acc[k] += v[k] * by[i];
      }
  }
}

// The units u, u + stride, ..., one after the other, by `threads` threads of which this is number t.
template <typename GT, bool AT>
__device__ __forceinline__ void accumulate_units(const AccumPlan &plan, const GT *__restrict__ dx, int D, float *__restrict__ accum,
                                                 int M, int32_t *__restrict__ ready_ids, float *__restrict__ ready_grads, int u,
                                                 int stride, int t, int threads) {
  constexpr int N = Cols<GT>::N;
  const int n_units = *plan.n_units;
  const int DC = D / N;
  const float fM = (float)M;
  if (u >= n_units) return;
  UnitDesc d = plan.units[u];
  while (true) {
    const int u_next = u + stride;
    UnitDesc d_next = d;
    if (u_next < n_units) d_next = plan.units[u_next];  // in flight while this unit is summed
    float *arow = accum + (size_t)d.image * D;
    for (int cg = t; cg < DC; cg += threads) {
      const GT *col = dx + N * cg;
      auto add = [&](float (&to)[N], int qa, int qb) {
        if constexpr (AT)
          add_rows_at<GT>(to, plan, col, D, qa, qb);
        else
          add_rows<GT>(to, plan.row_view, plan.row_scale, col, D, qa, qb);
      };
      float acc[N];
#pragma unroll
      for (int k = 0; k < N; ++k) acc[k] = 0.0f;
      if (d.q0 == d.s0) {
        // first group of this image in this step: continues what earlier steps left
        const int p = d.phase;
        const int len0 = min(M - p, d.s1 - d.s0);
        if (p != 0) load_f32<N>(arow + N * cg, acc);
        add(acc, d.s0, d.s0 + len0);
        const bool complete = (p + len0 == M);
        if (complete) {
          store_div<N>(ready_grads + (size_t)d.slot * D + N * cg, acc, fM);
          if (cg == 0) ready_ids[d.slot] = d.image;
        }
        const int tail = (d.s1 - d.s0 - len0) % M;  // rows of the image's unfinished last group
        if (!complete) {
          store_f32<N>(arow + N * cg, acc, 1.0f);
        } else if (tail == 0) {
          if (p != 0) {
            float zero[N];
#pragma unroll
            for (int k = 0; k < N; ++k) zero[k] = 0.0f;
            store_f32<N>(arow + N * cg, zero, 1.0f);
          }
        } else {
          float rest[N];
#pragma unroll
          for (int k = 0; k < N; ++k) rest[k] = 0.0f;
          add(rest, d.s1 - tail, d.s1);
          store_f32<N>(arow + N * cg, rest, 1.0f);
        }
      } else {
        // a complete middle group of M rows
        add(acc, d.q0, d.q0 + M);
        store_div<N>(ready_grads + (size_t)d.slot * D + N * cg, acc, fM);
        if (cg == 0) ready_ids[d.slot] = d.image;
      }
    }
    if (u_next >= n_units) break;
    u = u_next;
    d = d_next;
  }
}

// What the launch's first workgroups do of the embedding update: nothing (a divided step has it done), its second level
// (two streams: level 1 and the image counters are the launch before), or level 1 and the counters (one stream: level 2
// rides with the parameter update).  Level 1 ahead of the units on two streams held their wavefronts down to three a SIMD
// beside a product that needs the rest (16 384 views: 187 us a step against 180).
enum EmbRide { kNoRide, kSpans, kChunks };
struct RideWork {
  EmbeddingWork w;
  int blocks, count_blocks, lanes;   // workgroups per table and for the counters; lanes of a worker of level 1
};
struct NoWork {};

// level 1 and the counters, if workgroup `block` is one of theirs
__device__ __forceinline__ bool chunks_ride(const AccumPlan &plan, const RideWork &emb, int block) {
  if (block < 2 * emb.blocks) {
    const int second = block >= emb.blocks ? 1 : 0;
    const int tid = (block - second * emb.blocks) * blockDim.x + threadIdx.x;
    if (emb.w.bf16)
      embedding_chunk<bf16_t, 8>(emb.w.table[second], tid, emb.w.dx, 2 * emb.w.d, emb.w.d, emb.lanes, emb.w.opt);
    else
      embedding_chunk<float, 8>(emb.w.table[second], tid, emb.w.dx, 2 * emb.w.d, emb.w.d, emb.lanes, emb.w.opt);
    return true;
  }
  block -= 2 * emb.blocks;
  if (block >= emb.count_blocks) return false;
  count_images(plan, emb.w.counts, block * blockDim.x + threadIdx.x, emb.count_blocks * blockDim.x);
  return true;
}

// dx: the DFV slot of dLoss/dx, [B x D].  One workgroup per unit, D / Cols<GT>::N threads.
// kChunks needs 132 registers where the units alone take 44: three wavefronts a SIMD, which still have 72 KB of rows in
// flight on a CU, as much as a memory latency asks for.  kSpans has eight partials of a long run in flight: 59 (with 32
// in flight 138).
template <typename GT, int RIDE, bool AT>
__global__ void __launch_bounds__(256, RIDE == kChunks ? 3 : 1)
k_accumulate(AccumPlan plan, const GT *__restrict__ dx, int D, float *__restrict__ accum, int M,
             int32_t *__restrict__ ready_ids, float *__restrict__ ready_grads, std::conditional_t<RIDE == kNoRide, NoWork, RideWork> emb,
             const int32_t *__restrict__ status) {
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
  if constexpr (RIDE == kChunks) {
    if (chunks_ride(plan, emb, block)) return;
    block -= 2 * emb.blocks + emb.count_blocks;
    blocks -= 2 * emb.blocks + emb.count_blocks;
  }
  accumulate_units<GT, AT>(plan, dx, D, accum, M, ready_ids, ready_grads, block, blocks, threadIdx.x, blockDim.x);
}

// The same beside the weight-gradient products, for a step in blocks of views whose products all go on small tiles: neither
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
template <typename GT>
__global__ void __launch_bounds__(256, 3)
k_accumulate_wgrad(AccumPlan plan, const GT *__restrict__ dx, int D, float *__restrict__ accum, int M, int32_t *__restrict__ ready_ids,
                   float *__restrict__ ready_grads, BesideWork w, const int32_t *__restrict__ status) {
  using C = typename BesideTile<GT>::C;
  static_assert(C::THREADS == 256, "one size of workgroup");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[C::STAGES * C::STAGE_BYTES];
  int block = blockIdx.x, blocks = gridDim.x;
  if (block < w.tn_blocks) return tn_tile<C>(w.tn, w.K, w.splits, nullptr, xcd_remap(block, w.tn_blocks), lds);   // into the workspace only
  if (*status != 0) return;
  block -= w.tn_blocks;
  blocks -= w.tn_blocks;
  if (chunks_ride(plan, w.ride, block)) return;
  block -= 2 * w.ride.blocks + w.ride.count_blocks;
  blocks -= 2 * w.ride.blocks + w.ride.count_blocks;
  const int side = 256 / w.unit_threads, which = __builtin_amdgcn_readfirstlane((int)threadIdx.x / w.unit_threads);
  accumulate_units<GT, true>(plan, dx, D, accum, M, ready_ids, ready_grads, block * side + which, blocks * side,
                             (int)threadIdx.x - which * w.unit_threads, w.unit_threads);
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
                             float *ready_grads, const EmbeddingWork *emb, bool level2, const int32_t *status, hipStream_t s) {
  if (img.n <= 0 && !emb) return hipSuccess;
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
    blocks += 2 * work.blocks + work.count_blocks;
  }
#define GEAR_ACC(T, R, AT, EMB)                                                                                            \
  hipLaunchKernelGGL((k_accumulate<T, R, AT>), dim3(blocks), dim3(threads), 0, s, plan, (const T *)dx_dfv, D, grad_accum, M, \
                     ready_ids, ready_grads, EMB, status)
#define GEAR_ACC_T(T)              \
  if (!emb)                        \
    GEAR_ACC(T, kNoRide, false, NoWork{}); \
  else if (level2)                 \
    GEAR_ACC(T, kSpans, false, work); \
  else if (plan.row_at)            \
    GEAR_ACC(T, kChunks, true, work); \
  else                             \
    GEAR_ACC(T, kChunks, false, work)
  if (cfg.mlp_dtype == GEAR_BF16) {
    GEAR_ACC_T(bf16_t);
  } else {
    GEAR_ACC_T(float);
  }
#undef GEAR_ACC_T
#undef GEAR_ACC
  return hipGetLastError();
}

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
  if (bf16)
    hipLaunchKernelGGL(k_accumulate_wgrad<bf16_t>, grid, dim3(threads), 0, s, plan, (const bf16_t *)dx_dfv, D, grad_accum, M, ready_ids,
                       ready_grads, w, status);
  else
    hipLaunchKernelGGL(k_accumulate_wgrad<float>, grid, dim3(threads), 0, s, plan, (const float *)dx_dfv, D, grad_accum, M, ready_ids,
                       ready_grads, w, status);
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
