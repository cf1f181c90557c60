// Device code of the accumulation (accum.hip), which a step in blocks of views runs beside its weight gradients
// (accum_wgrad.hip).
#pragma once

#include "embedding_common.hpp"

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

// The units u, u + stride, ..., one after the other, by `threads` threads of which this is number t.  AT: the lists were sorted in LDS;
// PARTS: the plan lies in parts, and the counters of the images go with their first units (as in count_images, which has one thread for each
// of them and would have to look for its part).
template <typename GT, bool AT, bool PARTS>
__device__ __forceinline__ void accumulate_units(const AccumPlan &plan, const LocalState &local, const GT *__restrict__ dx, int D, float *__restrict__ accum,
                                                 int32_t *__restrict__ counts, int M, int32_t *__restrict__ ready_ids,
                                                 float *__restrict__ ready_grads, int u, int stride, int t, int threads) {
  constexpr int N = Cols<GT>::N;
  const int n_units = PARTS ? local.units : *plan.n_units;
  int slot = 0, slot_next = 0;   // emissions of lower parts
  auto unit = [&](int i, int &below) {
    if constexpr (PARTS) {
      const int part = part_of_unit(local, i);
      below = __builtin_amdgcn_readlane(local.slot, part);
      i += __builtin_amdgcn_readlane(local.place, part);
    }
    return plan.units[i];
  };
  const int DC = D / N;
  const float fM = (float)M;
  if (u >= n_units) return;
  UnitDesc d = unit(u, slot);
  while (true) {
    const int u_next = u + stride;
    UnitDesc d_next = d;
    if (u_next < n_units) d_next = unit(u_next, slot_next);  // in flight while this unit is summed
    float *arow = accum + (size_t)d.image * D;
    if constexpr (PARTS) {
      d.slot += slot;
      if (t == 0 && d.q0 == d.s0) counts[d.image] = d.collected;
    }
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
    slot = slot_next;
  }
}

// What the launch's first workgroups do of the embedding update: nothing (a divided step has it done), its second level
// (two streams: level 1 and the image counters are the launch before), or level 1 and the counters (one stream: level 2
// rides with the parameter update).  Level 1 ahead of the units on two streams held their wavefronts down to three a SIMD
// beside a product that needs the rest (16 384 views: 187 us a step against 180).
enum EmbRide { kNoRide, kSpans, kChunks, kChunksAndSums };   // the last: and the batch sums of the network (block_sums.hpp)
struct RideWork {
  EmbeddingWork w;
  int blocks, count_blocks, lanes;   // workgroups per table and for the counters; lanes of a worker of level 1
  int sum_blocks;                    // workgroups of the batch sums
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

}  // namespace
}  // namespace gear
