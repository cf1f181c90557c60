// Batch sums of the network (logit layer, biases, loss) in the shape in which blocks of views leave them (rows.hip), from what
// launches layer by layer have written: device code, carried by the accumulation (accum.hip).
//
// A long step on one stream goes layer by layer, because the launches of its layers carry the grouping, and the same step on
// two streams in blocks of views.  Every value of a view has the same bits either way; so that the sums over views have them
// too, they are added here in the blocks' order: a block's rows in parts, a part's rows one after the other, then the parts.
#pragma once

#include "gear_internal.hpp"
#include "rows.hpp"

namespace gear {
namespace {

template <typename T> using Raw4 = std::conditional_t<sizeof(T) == 2, uint2, float4>;   // four neighbouring values
__device__ __forceinline__ void widen4(float (&v)[4], const uint2 &t) {
  v[0] = __uint_as_float(t.x << 16), v[1] = __uint_as_float(t.x & 0xffff0000u);
  v[2] = __uint_as_float(t.y << 16), v[3] = __uint_as_float(t.y & 0xffff0000u);
}
__device__ __forceinline__ void widen4(float (&v)[4], const float4 &t) { v[0] = t.x, v[1] = t.y, v[2] = t.z, v[3] = t.w; }

// Four columns of one block, by one thread: `FLIGHT` rows requested together.  LOGIT: also the sums of dz h.
template <typename T, bool LOGIT, int FLIGHT>
__device__ __forceinline__ void block_columns(const BlockSums &w, const BlockSums::Columns &c, int block, int col) {
  const int row0 = block * w.rows, n = min(w.rows, w.B - row0), N = c.width, len = w.rows / rows_split(w.rows, N / 4);
  const T *delta = static_cast<const T *>(c.delta) + (size_t)row0 * N + col, *h = static_cast<const T *>(w.h) + (size_t)row0 * N + col;
  const float *dz = w.dz + row0;
  float d[4] = {0.f, 0.f, 0.f, 0.f}, g[4] = {0.f, 0.f, 0.f, 0.f}, part_d[4] = {0.f, 0.f, 0.f, 0.f}, part_g[4] = {0.f, 0.f, 0.f, 0.f};
  auto add_part = [&]() {
#pragma unroll
    for (int e = 0; e < 4; ++e) d[e] += part_d[e], g[e] += part_g[e], part_d[e] = part_g[e] = 0.0f;
  };
  for (int r0 = 0; r0 < n; r0 += FLIGHT) {
    Raw4<T> rd[FLIGHT], rh[FLIGHT];
    float z[FLIGHT];
#pragma unroll
    for (int i = 0; i < FLIGHT; ++i) {
      const int r = min(r0 + i, n - 1);
      rd[i] = *reinterpret_cast<const Raw4<T> *>(delta + (size_t)r * N);
      if constexpr (LOGIT) rh[i] = *reinterpret_cast<const Raw4<T> *>(h + (size_t)r * N), z[i] = dz[r];
    }
#pragma unroll
    for (int i = 0; i < FLIGHT; ++i)
      if (r0 + i < n) {
        if (((r0 + i) & (len - 1)) == 0 && r0 + i > 0) add_part();
        float v[4];
        if constexpr (LOGIT) {
          widen4(v, rh[i]);
#pragma unroll
          for (int e = 0; e < 4; ++e) part_g[e] += z[i] * v[e];
        }
        widen4(v, rd[i]);
#pragma unroll
        for (int e = 0; e < 4; ++e) part_d[e] += v[e];
      }
  }
  add_part();
  const size_t at = (size_t)block * N + col;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    c.part[at + e] = d[e];
    if constexpr (LOGIT) w.part_w[at + e] = g[e];
  }
}

// loss and dLoss/dz of one block, by one wavefront: a lane per view, kRowsWaves groups of lanes
__device__ __forceinline__ void block_loss(const BlockSums &w, int block, int lane) {
  const int per = w.rows / kRowsWaves, view = block * w.rows + lane;
  float loss = 0.0f, dz = 0.0f;
  if (lane < w.rows && view < w.B) {
    const float z = w.logits[view], y = w.label[view], ex = expf(-fabsf(z));
    loss = fmaxf(z, 0.0f) - z * y + log1pf(ex);
    dz = w.dz[view];
  }
  for (int off = per / 2; off > 0; off >>= 1) {
    loss += __shfl_xor(loss, off, kWave);
    dz += __shfl_xor(dz, off, kWave);
  }
  float all_loss = 0.0f, all_dz = 0.0f;
#pragma unroll
  for (int g = 0; g < kRowsWaves; ++g) {
    all_loss += __shfl(loss, g * per, kWave);
    all_dz += __shfl(dz, g * per, kWave);
  }
  if (lane == 0) {
    w.part_loss[block] = all_loss;
    w.part_b[block] = all_dz;
  }
}

// thread `tid` of those that block_sums_threads asks for, in whole wavefronts
template <typename T> __device__ __forceinline__ void block_sums(const BlockSums &w, int tid) {
  if (tid < w.blocks * kWave) return block_loss(w, tid / kWave, tid % kWave);
  tid -= w.blocks * kWave;
  for (int l = 0; l < w.layers; ++l) {
    const int owners = w.layer[l].width / 4;
    if (tid < w.blocks * owners)
      return l == 0 ? block_columns<T, true, 8>(w, w.layer[l], tid / owners, tid % owners * 4)
                    : block_columns<T, false, 16>(w, w.layer[l], tid / owners, tid % owners * 4);
    tid -= w.blocks * owners;
  }
}

}  // namespace

inline long long block_sums_threads(const BlockSums &w) {
  long long n = (long long)w.blocks * kWave;
  for (int l = 0; l < w.layers; ++l) n += (long long)w.blocks * (w.layer[l].width / 4);
  return n;
}

}  // namespace gear
