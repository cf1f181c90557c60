// The grouping of short lists of ids in LDS (device code; rows.hip carries it in its first workgroups).
//
// A list that fits into a workgroup's LDS needs no pass over memory: one workgroup reads it, sorts it and writes the result,
// so the chain of a short step has one link for the whole grouping where passes over memory have five, each with the
// latencies of a launch or of words between workgroups.  A list is cut by ranges of its ids into 2^parts_log2 parts, one
// workgroup each: every part reads the whole list and keeps its own ids, in order, so that none of them has to wait for
// another.  An item is 32 bits, the id without its range above its position in the list.
//
// All loops are rolled: a workgroup runs this code once, and what bounded a form with its items in registers, forty times
// unrolled, was the fetch of instructions (26 us for the two passes over a part of 157 ids, now 4).  The three lists of 4096
// views (18 400 images) take 38 us beside the rows' 37, of which the longest part, that of the most popular image (2906 ids,
// 2450 of them that one), needs 8 for reading the list, 14 for sorting and 15 for the plan.
#pragma once

#include "group_device.hpp"

namespace gear {
namespace {

#define GEAR_ROLLED _Pragma("clang loop unroll(disable)")
constexpr int kLocalThreads = 512, kLocalWaves = kLocalThreads / kWave;
constexpr int kLocalDigitBits = 8, kLocalRadix = 1 << kLocalDigitBits;

// exclusive scan over the workgroup's threads; smem: one word per wavefront
__device__ __forceinline__ unsigned long long local_scan(unsigned long long v, unsigned long long *total, unsigned long long *smem) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned long long inc = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const unsigned long long t = __shfl_up(inc, off, kWave);
    if (lane >= off) inc += t;
  }
  __syncthreads();   // smem may still be read
  if (lane == 63) smem[wave] = inc;
  __syncthreads();
  unsigned long long base = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < kLocalWaves; ++w) {
    const unsigned long long t = smem[w];
    if (w < wave) base += t;
    sum += t;
  }
  *total = sum;
  return base + inc - v;
}

__device__ __forceinline__ int lower_lanes(unsigned long long mask, int lane) { return __popcll(mask & ((1ull << lane) - 1ull)); }

// One stable LSD pass from src[0 .. m) to dst: a wavefront owns a contiguous share, counts its digits, and when it knows where
// each of them begins, ranks and moves its share round by round (ballots, in lane order).
__device__ __forceinline__ void local_pass(const uint32_t *src, uint32_t *dst, uint16_t *count /* [waves][radix] */, int m, int shift,
                                           int digit_bits, unsigned long long *smem) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int radix = 1 << digit_bits, share = (m + kLocalThreads - 1) / kLocalThreads * kWave;
  const int begin = wave * share, end = min(m, begin + share);
  uint32_t *words = reinterpret_cast<uint32_t *>(count);   // two counts a word: no carry, a share has fewer than 65 536 items
  GEAR_ROLLED for (int i = tid; i < kLocalWaves * radix / 2; i += kLocalThreads) words[i] = 0u;
  __syncthreads();
  GEAR_ROLLED for (int i = begin + lane; i < end; i += kWave) {
    const int digit = (int)(src[i] >> shift) & (radix - 1);
    // lanes that share the first one's digit add as one: of a popular image all would, to one word, one after the other
    const bool leads = digit == __builtin_amdgcn_readfirstlane(digit);
    const unsigned long long same = __ballot(leads);
    if (!leads || lower_lanes(same, lane) == 0)
      atomicAdd(&words[(wave * radix + digit) >> 1], (leads ? (uint32_t)__popcll(same) : 1u) << (16 * (digit & 1)));
  }
  __syncthreads();
  int total = 0;
  if (tid < radix)
#pragma unroll
    for (int w = 0; w < kLocalWaves; ++w) total += count[w * radix + tid];
  unsigned long long all;
  int base = (int)local_scan((unsigned long long)total, &all, smem);
  if (tid < radix)
#pragma unroll
    for (int w = 0; w < kLocalWaves; ++w) {
      const int c = count[w * radix + tid];
      count[w * radix + tid] = (uint16_t)base;   // at most 65 535 items
      base += c;
    }
  __syncthreads();
  uint16_t *mine = count + wave * radix;
  constexpr int U = 2;   // rounds side by side
  GEAR_ROLLED for (int i = begin; i < end; i += U * kWave) {
    uint32_t item[U];
    unsigned lo[U], hi[U];
    int digit[U];
    bool valid[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      valid[k] = i + k * kWave + lane < end;
      item[k] = valid[k] ? src[i + k * kWave + lane] : 0u;
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      digit[k] = (int)(item[k] >> shift) & (radix - 1);
      const unsigned long long v = __ballot(valid[k]);
      lo[k] = (unsigned)v, hi[k] = (unsigned)(v >> 32);
    }
#pragma unroll
    for (int b = 0; b < kLocalDigitBits; ++b)   // bits that a narrower digit does not have are 0 in all lanes
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const unsigned unset = ~(unsigned)((int)((unsigned)digit[k] << (31 - b)) >> 31);
        const unsigned long long v = __ballot(unset == 0u);
        lo[k] &= (unsigned)v ^ unset;
        hi[k] &= (unsigned)(v >> 32) ^ unset;
      }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const unsigned long long peers = (unsigned long long)hi[k] << 32 | lo[k];
      const int lower = lower_lanes(peers, lane);
      const int at = mine[digit[k]];   // a wavefront's LDS accesses complete in order: all read, then the first of each digit adds
      __builtin_amdgcn_wave_barrier();
      if (valid[k] && lower == 0) mine[digit[k]] = (uint16_t)(at + __popcll(peers));
      __builtin_amdgcn_wave_barrier();
      if (valid[k]) dst[at + lower] = item[k];
    }
  }
  __syncthreads();
}

// A part most of which is one id (a popular image, a user that stands for all unknown ones): those are in order as they are.
// Their positions go to their place in the list at once, the others are sorted by themselves behind the part's items and put
// around them; items[0 .. m) is then in order, but for the positions of the popular id, and p.perm is written.  False: no such
// id, or no room, and nothing has changed.  (us of the sort, 19 000 ids, in passes / like this: 45 % of them one image 19 / 10, 60 % 28 /
// 11, all 42 / 14.)
constexpr int kPopularLeast = 2048;   // items of a part (2048 of one image 39.4 us a step so, 41.6 in passes)
__device__ __forceinline__ bool local_popular(const LocalList &p, uint32_t *items, uint16_t *count, int m, int below, int room,
                                              unsigned long long *smem) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, vb = p.value_bits;
  // the most frequent of up to six of 64 items, the same in every wavefront
  const uint32_t sample = items[(int)((long long)lane * m / kWave)] >> vb;
  unsigned long long left = ~0ull;
  uint32_t id = 0u;
  int votes = 0;
  GEAR_ROLLED for (int k = 0; k < 6 && left; ++k) {
    const uint32_t candidate = __shfl(sample, __builtin_ctzll(left), kWave);
    const unsigned long long same = __ballot(sample == candidate);
    if (__popcll(same) > votes) votes = __popcll(same), id = candidate;
    left &= ~same;
  }
  if (votes < kWave / 2) return false;
  const int share = (m + kLocalThreads - 1) / kLocalThreads * kWave, begin = min(m, wave * share), end = min(m, begin + share);
  int lower = 0, equal = 0;   // of the wavefront's share
  GEAR_ROLLED for (int i = begin; i < end; i += kWave) {
    const uint32_t k = i + lane < end ? items[i + lane] >> vb : ~0u;
    lower += __popcll(__ballot(k < id));
    equal += __popcll(__ballot(k == id));
  }
  unsigned long long all;   // by all threads of a wavefront, of which the first one's counts
  const unsigned long long before = local_scan(lane == 0 ? (unsigned long long)lower | (unsigned long long)equal << 32 : 0ull, &all, smem);
  const int n_lower = (int)(uint32_t)all, n_equal = (int)(all >> 32), others = m - n_equal;
  if (m + others > room) return false;
  const int equal_before = (int)(__shfl(before, 0, kWave) >> 32);
  uint32_t *apart = items + m + (begin - equal_before);
  int32_t *place = p.perm + below + n_lower + equal_before;
  const uint32_t mask = (1u << vb) - 1u;
  GEAR_ROLLED for (int i = begin; i < end; i += kWave) {
    const bool in = i + lane < end;
    const uint32_t item = in ? items[i + lane] : 0u;
    const bool is = in && item >> vb == id;
    const unsigned long long same = __ballot(is), rest = __ballot(in && !is);
    if (is) place[lower_lanes(same, lane)] = (int)(item & mask);
    if (in && !is) apart[lower_lanes(rest, lane)] = item;
    place += __popcll(same);
    apart += __popcll(rest);
  }
  __syncthreads();
  const int bits = p.bits - p.parts_log2, passes = (bits + kLocalDigitBits - 1) / kLocalDigitBits;
  int a = m;   // others <= m: they have room below
  GEAR_ROLLED for (int pass = 0; pass < passes; ++pass) {
    const int from = pass * bits / passes, to = (pass + 1) * bits / passes;
    local_pass(items + a, items + (m - a), count, others, vb + from, to - from, smem);
    a = m - a;
  }
  if (a == 0) {
    GEAR_ROLLED for (int q = tid; q < others; q += kLocalThreads) items[m + q] = items[q];
    __syncthreads();
  }
  GEAR_ROLLED for (int q = tid; q < others; q += kLocalThreads) {
    const uint32_t item = items[m + q];
    const int at = q < n_lower ? q : q + n_equal;
    items[at] = item;
    p.perm[below + at] = (int)(item & mask);
  }
  GEAR_ROLLED for (int q = tid; q < n_equal; q += kLocalThreads) items[n_lower + q] = id << vb;
  __syncthreads();
  return true;
}

// The part's ids, in order, into items[0 .. m).  Returns m; *below = ids of the list in lower ranges.
// A thread owns `per` consecutive positions, a multiple of four: it counts its own, and writes them when it knows where.
// Loads go out in batches whose addresses are clamped instead of branched around: the ids are cold.
__device__ __forceinline__ int local_select(const LocalList &p, int part, uint32_t *items, unsigned long long *smem, int *below, bool *bad_ids) {
  constexpr int U = 5;   // quadruples of ids in flight
  const int tid = threadIdx.x, n = p.n, low_bits = p.bits - p.parts_log2;
  const int per = (n + 4 * kLocalThreads - 1) / (4 * kLocalThreads) * 4, p0 = min(n, tid * per), p1 = min(n, p0 + per);
  const int quads = ((uintptr_t)p.keys_in & 15u) == 0 ? n & ~3 : 0;   // positions that are read four at a time
  const int q1 = min(p1, quads), rest = max(p0, quads);
  unsigned mine = 0, lower = 0;
  bool bad = *bad_ids;
  auto count = [&](int32_t key) {
    const int range = (int)((uint32_t)key >> low_bits);
    bad |= key < 0 || (int64_t)key >= p.range;
    mine += range == part ? 1u : 0u;
    lower += range < part ? 1u : 0u;
  };
  if (quads > 0)
    GEAR_ROLLED for (int i = 0; i < per; i += 4 * U) {
      int4 key[U];
#pragma unroll
      for (int k = 0; k < U; ++k) key[k] = *reinterpret_cast<const int4 *>(p.keys_in + min(p0 + i + 4 * k, quads - 4));
#pragma unroll
      for (int k = 0; k < U; ++k)
        if (i + 4 * k < per && p0 + i + 4 * k < q1) count(key[k].x), count(key[k].y), count(key[k].z), count(key[k].w);
    }
  GEAR_ROLLED for (int q = rest; q < p1; ++q) count(p.keys_in[q]);
  unsigned long long all;   // a list has less than 65 536 ids
  int at = (int)(uint32_t)local_scan((unsigned long long)mine | (unsigned long long)lower << 32 | (unsigned long long)(bad ? 1 : 0) << 48, &all, smem);
  const int m = (int)(uint32_t)all;
  *below = (int)(all >> 32) & 0xffff;
  *bad_ids = (all >> 48) != 0ull;
  auto keep = [&](int32_t key, int q) {
    if ((int)((uint32_t)key >> low_bits) == part) {
      items[at] = ((uint32_t)key & ((1u << low_bits) - 1u)) << p.value_bits | (uint32_t)q;
      ++at;
    }
  };
  if (mine > 0) {
    if (quads > 0)
      GEAR_ROLLED for (int i = 0; i < per; i += 4 * U) {
        int4 key[U];
#pragma unroll
        for (int k = 0; k < U; ++k) key[k] = *reinterpret_cast<const int4 *>(p.keys_in + min(p0 + i + 4 * k, quads - 4));
#pragma unroll
        for (int k = 0; k < U; ++k) {
          const int q = p0 + i + 4 * k;
          if (i + 4 * k < per && q < q1) keep(key[k].x, q), keep(key[k].y, q + 1), keep(key[k].z, q + 2), keep(key[k].w, q + 3);
        }
      }
    GEAR_ROLLED for (int q = rest; q < p1; ++q) keep(p.keys_in[q], q);
  }
  __syncthreads();
  return m;
}

// Segments of the part's ids and the plan of the accumulation (group_device.hpp has the rules): a thread owns `per`
// consecutive positions, at most 64.  cnt: room for the counters of the items' images.
// FITS: the counters too are in LDS.  PARTS: the part leaves what it counts to those who read the plan.
template <bool FITS, bool PARTS>
__device__ __forceinline__ void local_plan(const LocalTask &t, const LocalList &p, int part, const uint32_t *items, int32_t *cnt, int m,
                                           int below, unsigned long long *smem, int (*edge)[kLocalWaves], int *s_base) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const PlanArgs &args = t.plan;
  const AccumPlan &plan = args.plan;
  const int M = args.M, per = ((m + kLocalThreads - 1) / kLocalThreads) | 1, p0 = tid * per, vb = p.value_bits;   // odd: LDS banks
  const int high = part << (p.bits - p.parts_log2), mine = min(max(m - p0, 0), per);
#define GEAR_ID(q) (high | (int)(items[q] >> vb))
  if constexpr (FITS)
#pragma clang loop unroll_count(8)
    for (int q = tid; q < m; q += kLocalThreads) cnt[q] = args.counts[min((int64_t)GEAR_ID(q), p.range - 1)];
  // heads, bit by bit; last head at or before and first head behind the thread's positions
  unsigned long long heads = 0;
  uint32_t before_key = p0 > 0 && p0 < m ? items[p0 - 1] >> vb : ~0u;
  GEAR_ROLLED for (int i = 0; i < mine; ++i) {
    const uint32_t k = items[p0 + i] >> vb;
    if (p0 + i == 0 || k != before_key) heads |= 1ull << i;
    before_key = k;
  }
  int run_last = heads ? p0 + 63 - __builtin_clzll(heads) : -1, run_first = heads ? p0 + __builtin_ctzll(heads) : INT32_MAX;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int a = __shfl_up(run_last, off, kWave), b = __shfl_down(run_first, off, kWave);
    if (lane >= off) run_last = max(run_last, a);
    if (lane + off < kWave) run_first = min(run_first, b);
  }
  if (lane == 63) edge[0][wave] = run_last;
  if (lane == 0) edge[1][wave] = run_first;
  int seg0 = __shfl_up(run_last, 1, kWave), seg1 = __shfl_down(run_first, 1, kWave);
  if (lane == 0) seg0 = -1;
  if (lane == 63) seg1 = INT32_MAX;
  __syncthreads();   // also of cnt
#pragma unroll
  for (int w = 0; w < kLocalWaves; ++w) {
    if (w < wave) seg0 = max(seg0, edge[0][w]);
    if (w > wave) seg1 = min(seg1, edge[1][w]);
  }
  if (seg1 == INT32_MAX) seg1 = m;
  unsigned long long units = 0, emits = 0;
  int seg = seg0;
  // Counters that are not in LDS come four positions at a time, whether it is a head or not: one by one, at the heads, each was
  // a memory latency (a part of 11 500 ids 25 us here, now 19).
  constexpr int U = FITS ? 1 : 4;
  auto counters = [&](int i, int (&c)[U]) {
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int q = min(p0 + min(i + k, mine - 1), m - 1);
      if constexpr (FITS)
        c[k] = cnt[q];
      else
        c[k] = args.counts[min((int64_t)GEAR_ID(q), p.range - 1)];
    }
  };
  GEAR_ROLLED for (int i0 = 0; i0 < mine; i0 += U) {
    int c[U];
    counters(i0, c);
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int i = i0 + k, q = p0 + i;
      if (i >= mine) break;
      const bool head = (heads >> i) & 1ull;
      if (head) seg = q;
      const int ph = (c[k] + (q - seg)) % M;
      if (head || (ph == 0 && M <= m - q && items[q + M - 1] >> vb == items[q] >> vb)) units |= 1ull << i;
      if (ph == M - 1) emits |= 1ull << i;
    }
  }
  // heads, units and emissions, 21 bits each
  unsigned long long all;
  const unsigned long long before = local_scan((unsigned long long)__popcll(heads) | (unsigned long long)__popcll(units) << 21 |
                                                   (unsigned long long)__popcll(emits) << 42, &all, smem);
  constexpr int kMask = (1 << 21) - 1;
  int h = (int)(before & kMask), u = (int)((before >> 21) & kMask), e = (int)(before >> 42);
  if constexpr (PARTS) {
    if (tid == 0) plan.local.parts[part] = PartCounts{below, (int)(all & kMask), (int)((all >> 21) & kMask), (int)(all >> 42)};
    h += below, u += below;
  } else {
    // What the parts below count: each publishes its own before it looks, and parts are numbered by a ticket, so those below
    // are running.  Whether ids are bad or not: a part does not know what another finds.
    if (tid < 3) publish(t.state + 3 * part + tid, 1u + (uint32_t)((all >> (21 * tid)) & kMask));
    if (wave == 0) {
      int v[3] = {0, 0, 0};
      if (lane < part)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          uint32_t w;
          while ((w = published(t.state + 3 * lane + c)) == 0u) __builtin_amdgcn_s_sleep(2);
          v[c] = (int)w - 1;
        }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[c] += __shfl_xor(v[c], off, kWave);
        if (lane == 0) s_base[c] = v[c];
      }
    }
    __syncthreads();
    h += s_base[0], u += s_base[1], e += s_base[2];
  }
  seg = seg0;
  GEAR_ROLLED for (int i0 = 0; i0 < mine; i0 += U) {
    int c[U];
    counters(i0, c);
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int i = i0 + k, q = p0 + i;
      if (i >= mine) break;
      const bool head = (heads >> i) & 1ull;
      if (head) seg = q;
      if (head && t.unique) {
        t.unique[h] = GEAR_ID(q);
        t.segoff[h] = below + q;
      }
      h += head ? 1 : 0;
      if ((units >> i) & 1ull) {
        const unsigned long long behind = i < 63 ? heads >> (i + 1) : 0ull;   // next head of this thread, or what follows it
        const int end = behind ? q + 1 + __builtin_ctzll(behind) : seg1;
        UnitDesc d;
        d.q0 = below + q;
        d.image = GEAR_ID(q);
        d.slot = e;
        d.s0 = below + seg;
        d.s1 = below + end;
        d.phase = c[k] % M;
        d.collected = c[k] + (end - seg);
        d.pad = 0;
        plan.units[u] = d;
        ++u;
      }
      e += (emits >> i) & 1ull ? 1 : 0;
    }
  }
  if (!PARTS && part == (1 << p.parts_log2) - 1 && tid == 0) {
    const int n_heads = s_base[0] + (int)(all & kMask), n_emits = s_base[2] + (int)(all >> 42);
    *t.n_unique = n_heads;
    if (t.unique) t.segoff[n_heads] = p.n;
    *plan.n_units = s_base[1] + (int)((all >> 21) & kMask);
    *args.n_ready = n_emits > args.ready_cap ? 0 : n_emits;
    if (n_emits > args.ready_cap) flag(t.failed, args.status, GEAR_ERR_CAPACITY);
  }
#undef GEAR_ID
}

// the part's place in the sorted list, and what hangs on the images
template <bool FITS, bool PARTS>
__device__ __forceinline__ void local_finish(const LocalTask &t, const LocalList &p, bool last, bool placed, int part, const uint32_t *sorted,
                                             uint32_t *spare, int m, int below, unsigned long long *smem,
                                             int (*edge)[kLocalWaves], int *s_base) {
  const int high = part << (p.bits - p.parts_log2);
  GEAR_ROLLED for (int q = threadIdx.x; q < m; q += kLocalThreads) {
    const uint32_t item = sorted[q];
    if (!last) p.sorted_keys[below + q] = high | (int)(item >> p.value_bits);   // the images' are in the plan
    if (!placed) p.perm[below + q] = (int)(item & ((1u << p.value_bits) - 1u));
  }
  if (last) local_plan<FITS, PARTS>(t, p, part, sorted, reinterpret_cast<int32_t *>(spare), m, below, smem, edge, s_base);
}

// Two sets of the part's items are in LDS (INSIDE), or one is and the other in the workspace: a part is that long only where
// one image is very popular.
template <bool INSIDE, bool PARTS>
__device__ __forceinline__ void local_sorted(const LocalTask &t, const LocalList &p, bool last, bool placed, int part, uint32_t *items, uint16_t *count,
                                             int m, int below, unsigned long long *smem, int (*edge)[kLocalWaves], int *s_base) {
  const int bits = p.bits - p.parts_log2, passes = placed ? 0 : (bits + kLocalDigitBits - 1) / kLocalDigitBits;
  uint32_t *spare = p.spare + below;
  int a = 0;   // offsets and not pointers that change places: the compiler then knows what is LDS
  GEAR_ROLLED for (int pass = 0; pass < passes; ++pass) {
    const int from = pass * bits / passes, to = (pass + 1) * bits / passes, shift = p.value_bits + from;
    if constexpr (INSIDE) {
      local_pass(items + a, items + (m - a), count, m, shift, to - from, smem);
      a = m - a;
    } else {
      local_pass(items, spare, count, m, shift, to - from, smem);
#pragma clang loop unroll_count(8)
      for (int q = threadIdx.x; q < m; q += kLocalThreads) items[q] = spare[q];
      __syncthreads();
    }
  }
  if constexpr (INSIDE)
    local_finish<true, PARTS>(t, p, last, placed, part, items + a, items + (m - a), m, below, smem, edge, s_base);
  else
    local_finish<false, PARTS>(t, p, last, placed, part, items, nullptr, m, below, smem, edge, s_base);
}

// Workgroup `block` of t.blocks, with kLocalThreads threads.  lds: kLocalWaves * kLocalRadix counts and t.room items.
template <bool PARTS> __device__ __forceinline__ void local_group(const LocalTask &t, int block, unsigned char *lds) {
  __shared__ unsigned long long smem[kLocalWaves];
  __shared__ int edge[2][kLocalWaves], s_base[3], s_part;
  // by selection and not by an index, with which the arguments would be copied to memory
  static_assert(kMaxProblems == 3, "users, URLs, images");
  const int first = 1 << t.list[0].parts_log2, second = first + (1 << t.list[1].parts_log2);
  const bool last = block >= second;
  const int word = block;
  // Past the L2, from which they would be written back when the launch ends, over what another call has reported meanwhile.
  if (PARTS && block == 0 && threadIdx.x == 0) {
    __hip_atomic_store(t.plan.status, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(t.plan.n_ready, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(t.loss, 0.0f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  LocalList p = t.list[0];
  if (last)
    p = t.list[2], block -= second;
  else if (block >= first)
    p = t.list[1], block -= first;
  int part = block;
  if (!PARTS && last) {
    if (threadIdx.x == 0) s_part = draw_ticket(t.ticket);
    __syncthreads();
    part = s_part;
  }
  bool bad = false;
  if (word < first) {   // the offsets with the first list
    int32_t lo, hi;
    GEAR_ROLLED for (int i = word * kLocalThreads + threadIdx.x; i < t.views.B; i += first * kLocalThreads)
      bad |= !view_ok(t.views, i, lo, hi);
  }
  uint32_t *items = reinterpret_cast<uint32_t *>(lds + kLocalWaves * kLocalRadix * sizeof(uint16_t));
  uint16_t *count = reinterpret_cast<uint16_t *>(lds);
  int below;
  const int m = local_select(p, part, items, smem, &below, &bad);
  if constexpr (PARTS) {
    const LocalResult &result = t.plan.plan.local;
    if (threadIdx.x == 0) result.codes[word] = bad ? 1 : 0;
    if (word == 0 && (int)threadIdx.x < (kCodeGroup - t.blocks % kCodeGroup) % kCodeGroup) result.codes[t.blocks + threadIdx.x] = 0;
  } else {
    if (bad && threadIdx.x == 0) flag(t.failed, t.plan.status, GEAR_ERR_RANGE);
  }
  const bool placed = m >= kPopularLeast && local_popular(p, items, count, m, below, t.room, smem);
  if (2 * m <= t.room)
    local_sorted<true, PARTS>(t, p, last, placed, part, items, count, m, below, smem, edge, s_base);
  else
    local_sorted<false, PARTS>(t, p, last, placed, part, items, count, m, below, smem, edge, s_base);
}

}  // namespace
}  // namespace gear
