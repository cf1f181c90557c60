// Device code of the embedding update (update.hip), whose two levels run in launches of their own beside a long product, or
// in workgroups of the accumulation (level 1) and of the parameter update (level 2).
#pragma once

#include "gear_internal.hpp"
#include "local_parts.hpp"

#include <type_traits>

namespace gear {
namespace {

// four values of a row in its storage type
template <typename ET> using RowCell = typename std::conditional<sizeof(ET) == 4, float4, uint2>::type;
__device__ __forceinline__ float4 widen_cell(const float4 &w) { return w; }
__device__ __forceinline__ float4 widen_cell(const uint2 &w) {
  return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                     __uint_as_float(w.y & 0xffff0000u));
}
__device__ __forceinline__ void narrow_cell(float4 &dst, const float4 &v) { dst = v; }
__device__ __forceinline__ void narrow_cell(uint2 &dst, const float4 &v) {
  dst = make_uint2((uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16),
                   (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16));
}

__device__ __forceinline__ void add4(float4 &a, const float4 &b) {
  a.x += b.x;
  a.y += b.y;
  a.z += b.z;
  a.w += b.w;
}

// level 1: one worker per chunk of sorted positions; tid: the thread's number among those of the table
template <typename ET, int AHEAD>
__device__ __forceinline__ void embedding_chunk(const EmbeddingTable &t, int tid, const float *__restrict__ dx, int F, int d,
                                                int lanes_per_worker, const Optim &opt) {
  const int chunk = tid / lanes_per_worker, c4 = tid % lanes_per_worker;
  const int q_begin = chunk * kChunk;
  if (q_begin >= t.n || c4 >= d / 4) return;
  const int q_end = min(t.n, q_begin + kChunk);
  const float *col = dx + t.col0 + 4 * c4;

  // ids, batch positions and rows of the whole chunk first, so that all loads are in flight at once
  int keys[kChunk + 1], pos[kChunk];
  if (q_begin + kChunk <= t.n) {
#pragma unroll
    for (int i = 0; i < kChunk; i += 4) {
      const int4 k = *reinterpret_cast<const int4 *>(t.keys + q_begin + i), p = *reinterpret_cast<const int4 *>(t.perm + q_begin + i);
      keys[i] = k.x, keys[i + 1] = k.y, keys[i + 2] = k.z, keys[i + 3] = k.w;
      pos[i] = p.x, pos[i + 1] = p.y, pos[i + 2] = p.z, pos[i + 3] = p.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kChunk; ++i) {
      const int q = q_begin + i;
      keys[i] = q < t.n ? t.keys[q] : -1;
      pos[i] = q < t.n ? t.perm[q] : 0;
    }
  }
  keys[kChunk] = q_begin + kChunk < t.n ? t.keys[q_begin + kChunk] : -1;
  float4 row[kChunk];
#pragma unroll
  for (int i = 0; i < kChunk; ++i)
    row[i] = q_begin + i < q_end ? *reinterpret_cast<const float4 *>(col + (size_t)pos[i] * F)
                                 : make_float4(0.f, 0.f, 0.f, 0.f);

  // running sums inside each run, in place and in order: row[i] becomes the sum of its run so far
#pragma unroll
  for (int i = 1; i < kChunk; ++i)
    if (q_begin + i < q_end && keys[i] == keys[i - 1]) {
      float4 sum = row[i - 1];
      add4(sum, row[i]);
      row[i] = sum;
    }
  // A run is complete here when it starts and ends inside the chunk; the first run may have begun in
  // an earlier chunk, the last one may go on into the next.
  const bool first_starts_here = q_begin == 0 || t.keys[q_begin - 1] != keys[0];
  bool whole[kChunk];
#pragma unroll
  for (int i = 0; i < kChunk; ++i) {
    const bool in = q_begin + i < q_end;
    const bool ends_here = keys[i + 1] != keys[i];
    const bool starts_here = keys[i] != keys[0] || first_starts_here;
    whole[i] = in && ends_here && starts_here;
    if (in && !whole[i] && (ends_here || q_begin + i + 1 == q_end)) {
      float *dst = (starts_here ? t.part_last : t.part_first) + (size_t)chunk * d;
      *reinterpret_cast<float4 *>(dst + 4 * c4) = row[i];
    }
  }
  // The cells of AHEAD complete runs (a quarter as many with Adam, which has three cells to a run) are requested together,
  // then updated and written back (ids in a sorted chunk are distinct per run, so no two of these cells are the same).  One
  // after the other, each waiting for its own load, sixteen rows cost sixteen memory latencies.
  using Cell = RowCell<ET>;
  if (opt.adam) {
    constexpr int G = AHEAD / 4;
#pragma unroll
    for (int i0 = 0; i0 < kChunk; i0 += G) {
      Cell w[G];
      float4 m[G], v[G];
#pragma unroll
      for (int i = 0; i < G; ++i)
        if (whole[i0 + i]) {
          const size_t at = (size_t)keys[i0 + i] * d;
          w[i] = reinterpret_cast<const Cell *>(static_cast<const ET *>(t.rows) + at)[c4];
          m[i] = reinterpret_cast<const float4 *>(t.mom.m + at)[c4];
          v[i] = reinterpret_cast<const float4 *>(t.mom.v + at)[c4];
        }
#pragma unroll
      for (int i = 0; i < G; ++i)
        if (whole[i0 + i]) {
          const size_t at = (size_t)keys[i0 + i] * d;
          const float4 g = row[i0 + i];
          float4 x = widen_cell(w[i]);
          x.x = optim_apply(opt, x.x, g.x, &m[i].x, &v[i].x);
          x.y = optim_apply(opt, x.y, g.y, &m[i].y, &v[i].y);
          x.z = optim_apply(opt, x.z, g.z, &m[i].z, &v[i].z);
          x.w = optim_apply(opt, x.w, g.w, &m[i].w, &v[i].w);
          narrow_cell(reinterpret_cast<Cell *>(static_cast<ET *>(t.rows) + at)[c4], x);
          reinterpret_cast<float4 *>(t.mom.m + at)[c4] = m[i];
          reinterpret_cast<float4 *>(t.mom.v + at)[c4] = v[i];
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    return;
  }
#pragma unroll
  for (int i0 = 0; i0 < kChunk; i0 += AHEAD) {
    Cell w[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
      if (whole[i0 + i])
        w[i] = reinterpret_cast<const Cell *>(static_cast<const ET *>(t.rows) + (size_t)keys[i0 + i] * d)[c4];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
      if (whole[i0 + i]) {
        const float4 g = row[i0 + i];
        float4 x = widen_cell(w[i]);
        x.x -= opt.lr * g.x, x.y -= opt.lr * g.y, x.z -= opt.lr * g.z, x.w -= opt.lr * g.w;
        narrow_cell(reinterpret_cast<Cell *>(static_cast<ET *>(t.rows) + (size_t)keys[i0 + i] * d)[c4], x);
      }
    if (AHEAD < kChunk) __builtin_amdgcn_sched_barrier(0);
  }
}

// counts[image] += occurrences of the image in this step (Section 1, third point), by the image's first unit; thread `at`
// of `stride`
__device__ __forceinline__ void count_images(const AccumPlan &plan, int32_t *__restrict__ counts, int at, int stride) {
  const int n = *plan.n_units;
  for (int u = at; u < n; u += stride) {
    const UnitDesc d = plan.units[u];
    if (d.q0 == d.s0) counts[d.image] = d.collected;
  }
}

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

inline int embedding_lanes(int d) {   // power of two so that workers do not straddle wavefronts
  int lanes = 1;
  while (lanes < d / 4) lanes <<= 1;
  return lanes;
}
inline int embedding_chunks(const EmbeddingWork &w) { return (w.table[0].n + kChunk - 1) / kChunk; }   // one id of either list per view

}  // namespace gear
