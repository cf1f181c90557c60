// The end of a step's parameter updates (Section 3, step 4), one launch: the weight gradients' partial sums of all hidden
// layers, the logit layer's weights and bias, the hidden layers' biases, each followed by its update, and the loss; on a step that does not
// divide dLoss/dx also the second level of the embedding update (update.hip).
// They are small and wait for nothing but their partials: bound by a launch's own 4 us, which a launch per bias, one for
// the logit layer and one for the weights each paid.  (A step of 4096 views on one stream: 150 us with those and the
// second level of the embedding update in launches of their own, 136 without.)
#include "embedding_common.hpp"

namespace gear {
namespace {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// W <- update(W, sum_z partial[z]), z ascending; a thread owns four consecutive elements (count is a
// multiple of 4 because layer widths are multiples of 8) and keeps eight partials in flight
__device__ __forceinline__ void splitk_sgd_at(const float *__restrict__ partial, int splits, int64_t count,
                                              float *__restrict__ w, const Optim &opt, const Moments &mom, int64_t i) {
  if (i >= count) return;
  float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
  int z = 0;
  for (; z + 8 <= splits; z += 8) {
    float4 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = *reinterpret_cast<const float4 *>(partial + (size_t)(z + k) * count + i);
#pragma unroll
    for (int k = 0; k < 8; ++k) g.x += v[k].x, g.y += v[k].y, g.z += v[k].z, g.w += v[k].w;
  }
  for (; z < splits; ++z) {
    const float4 v = *reinterpret_cast<const float4 *>(partial + (size_t)z * count + i);
    g.x += v.x, g.y += v.y, g.z += v.z, g.w += v.w;
  }
  float4 cur = *reinterpret_cast<float4 *>(w + i);
  if (!opt.adam) {
    cur.x -= opt.lr * g.x, cur.y -= opt.lr * g.y, cur.z -= opt.lr * g.z, cur.w -= opt.lr * g.w;
  } else {
    float4 m = *reinterpret_cast<float4 *>(mom.m + i), v = *reinterpret_cast<float4 *>(mom.v + i);
    cur.x = optim_apply(opt, cur.x, g.x, &m.x, &v.x);
    cur.y = optim_apply(opt, cur.y, g.y, &m.y, &v.y);
    cur.z = optim_apply(opt, cur.z, g.z, &m.z, &v.z);
    cur.w = optim_apply(opt, cur.w, g.w, &m.w, &v.w);
    *reinterpret_cast<float4 *>(mom.m + i) = m;
    *reinterpret_cast<float4 *>(mom.v + i) = v;
  }
  *reinterpret_cast<float4 *>(w + i) = cur;
}

// loss = (sum of the workgroups' partial sums) / B, by one wavefront, in a fixed shape
__device__ __forceinline__ void loss_final(const float *__restrict__ loss_partial, int n, int B,
                                           float *__restrict__ loss) {
  float part[kLossBlocks / kWave];
#pragma unroll
  for (int k = 0; k < kLossBlocks / kWave; ++k) {
    const int i = threadIdx.x + k * kWave;
    part[k] = i < n ? loss_partial[i] : 0.0f;
  }
  float v = 0.0f;
#pragma unroll
  for (int k = 0; k < kLossBlocks / kWave; ++k) v += part[k];
  v = wave_sum(v);
  if (threadIdx.x == 0) *loss = v / (float)B;
}

// dst[j] -= lr * sum_p partial[p][j].  Eight columns per workgroup and 32 row lanes, each adding
// every 32nd partial in order (eight loads in flight); then the 32 lanes are added in order.
__device__ __forceinline__ void partial_sgd(const float *__restrict__ partial, int P, int H, float *__restrict__ dst,
                                            const Optim &opt, const Moments &mom, int block) {
  __shared__ float s[32][8];
  const int c = threadIdx.x & 7, g = threadIdx.x >> 3;
  const int j = block * 8 + c;
  float acc = 0.0f;
  if (j < H) {
    int p = g;
    for (; p + 32 * 7 < P; p += 32 * 8) {
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = partial[(size_t)(p + 32 * i) * H + j];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc += v[i];
    }
    for (; p < P; p += 32) acc += partial[(size_t)p * H + j];
  }
  s[g][c] = acc;
  __syncthreads();
  if (g == 0 && j < H) {
    float t = 0.0f;
#pragma unroll
    for (int k = 0; k < 32; ++k) t += s[k][c];
    dst[j] = optim_apply(opt, dst[j], t, mom.m + j, mom.v + j);
  }
}

struct ParamArgs {
  int count, n_columns, splits;
  SplitkProblem p[GEAR_MAX_LAYERS];
  int first_block[GEAR_MAX_LAYERS];
  ColumnSum c[kMaxColumnSums];
  int first_column_block[kMaxColumnSums];
  int columns_at, loss_at;      // first workgroup of the column sums, and the loss's
  LossSum loss;
  LocalOutputs local;
};
struct SpanWork {
  EmbeddingWork w;
  int blocks;                   // workgroups per table, ahead of all others: the longest run is the longest chain
};
struct NoSpans {};

template <bool SPANS>
__global__ void __launch_bounds__(256) k_param_update(ParamArgs args, std::conditional_t<SPANS, SpanWork, NoSpans> spans,
                                                      Optim opt, const int32_t *__restrict__ status) {
  if (args.local.local.parts) {
    const LocalState local = local_state(args.local.local, blockIdx.x == 0);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      if (local.code)
        atomicCAS(args.local.status, 0, local.code);
      else
        *args.local.n_ready = local.emits;
    }
    if (local.code) return;
  } else if (*status != 0) {
    if (blockIdx.x == 0 && threadIdx.x == 0 && args.local.n_ready) *args.local.n_ready = 0;
    return;
  }
  int block = blockIdx.x;
  if constexpr (SPANS) {
    if (block < 2 * spans.blocks) {
      const int second = block >= spans.blocks ? 1 : 0;
      const int chunk = (block - second * spans.blocks) * (256 / kWave) + threadIdx.x / kWave;
      if (spans.w.bf16)
        embedding_span<bf16_t, 16>(spans.w.table[second], chunk, spans.w.d, spans.w.opt);
      else
        embedding_span<float, 16>(spans.w.table[second], chunk, spans.w.d, spans.w.opt);
      return;
    }
    block -= 2 * spans.blocks;
  }
  if (block >= args.loss_at) {
    if (threadIdx.x < kWave) loss_final(args.loss.partial, args.loss.parts, args.loss.B, args.loss.loss);
  } else if (block >= args.columns_at) {
    int which = 0;
    for (int i = 1; i < args.n_columns; ++i)
      if (block >= args.first_column_block[i]) which = i;
    const ColumnSum &c = args.c[which];
    partial_sgd(c.partial, c.parts, c.width, c.dst, opt, c.mom, block - args.first_column_block[which]);
  } else {
    int which = 0;
    for (int i = 1; i < args.count; ++i)
      if (block >= args.first_block[i]) which = i;
    const SplitkProblem &q = args.p[which];
    splitk_sgd_at(q.partial, args.splits, q.count, q.w, opt, q.mom,
                  ((int64_t)(block - args.first_block[which]) * blockDim.x + threadIdx.x) * 4);
  }
}

}  // namespace

hipError_t launch_param_update(const SplitkProblem *p, int count, int splits, const ColumnSum *c, int n_columns,
                               const LossSum &loss, const EmbeddingWork *emb, const LocalOutputs &local, const Optim &opt,
                               const int32_t *status, hipStream_t s, hipEvent_t stop) {
  if (count < 0 || count > GEAR_MAX_LAYERS || splits < 1 || n_columns < 0 || n_columns > kMaxColumnSums)
    return hipErrorInvalidValue;
  ParamArgs args;
  args.count = count;
  args.n_columns = n_columns;
  args.splits = splits;
  args.loss = loss;
  args.local = local;
  int blocks = 0;
  for (int i = 0; i < GEAR_MAX_LAYERS; ++i) {
    args.p[i] = i < count ? p[i] : SplitkProblem{nullptr, nullptr, Moments{nullptr, nullptr}, 0};
    args.first_block[i] = blocks;
    if (i < count) blocks += (int)((p[i].count / 4 + 255) / 256);
  }
  args.columns_at = blocks;
  for (int i = 0; i < kMaxColumnSums; ++i) {
    args.c[i] = i < n_columns ? c[i] : ColumnSum{nullptr, nullptr, Moments{nullptr, nullptr}, 0, 0};
    args.first_column_block[i] = blocks;
    if (i < n_columns) blocks += (c[i].width + 7) / 8;
  }
  args.loss_at = blocks;
  if (loss.parts > 0) ++blocks;
  if (emb) {
    SpanWork spans;
    spans.w = *emb;
    spans.blocks = (embedding_chunks(*emb) + 256 / kWave - 1) / (256 / kWave);
    launch_leaving(stop, k_param_update<true>, dim3(blocks + 2 * spans.blocks), 256, 0, s, args, spans, opt, status);
    return hipGetLastError();
  }
  if (blocks == 0) return leave(stop, s);
  launch_leaving(stop, k_param_update<false>, dim3(blocks), 256, 0, s, args, NoSpans{}, opt, status);
  return hipGetLastError();
}

}  // namespace gear
