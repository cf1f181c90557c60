// Device code of the grouping of a step's ids (group.hip), which runs in launches of its own or in workgroups that the
// launches of the forward pass carry along.
#pragma once

#include "gear_internal.hpp"

namespace gear {
namespace {

__device__ __forceinline__ int wave_inclusive_scan(int v, int lane) {
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int t = __shfl_up(v, off, kWave);
    if (lane >= off) v += t;
  }
  return v;
}

// exclusive scan of one int per thread over a workgroup of WAVES wavefronts; *total = sum of all
template <int WAVES = 4>
__device__ __forceinline__ int block_exclusive_scan(int v, int *total, int *smem /* >= WAVES ints */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int inc = wave_inclusive_scan(v, lane);
  __syncthreads();  // smem may still be read from a previous call
  if (lane == 63) smem[wave] = inc;
  __syncthreads();
  int base = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    const int t = smem[w];
    if (w < wave) base += t;
    sum += t;
  }
  *total = sum;
  return base + inc - v;
}

// ---- words that tiles publish for the tiles after them -------------------------------------------------
// 0: nothing yet; 1 + c: this tile alone counts c (at most a tile's keys); kPrefix | c: this tile and all before it
// count c.  A word carries its own value, so no order between stores matters and relaxed accesses do; agent scope,
// because the tiles run on several XCDs.  Tiles are numbered by a ticket that a workgroup draws when it starts, not by
// its place in the grid: whoever waits for a word waits for a workgroup that is already running and that publishes its
// own count before it waits for anybody, so every wait ends whatever else occupies the device.  A workgroup that stays idle
// publishes nothing, so all of a launch have to agree on that: they look at `failed`, which no other call writes.
constexpr uint32_t kPrefix = 0x80000000u;
__device__ __forceinline__ void publish(uint32_t *word, uint32_t v) {
  __hip_atomic_store(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t published(const uint32_t *word) {
  return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int draw_ticket(int32_t *counter) {
  return __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- check of the ids and digit counts of all passes ---------------------------------------------------
// A page view is a user id, a URL bucket and
// a list of image ids (Section 1, Table 1); every id later indexes a table, so a bad id must be caught before any
// kernel that changes caller state dereferences it: a violation sets the status word and every later kernel of the
// step returns at once.  Also expands the CSR offsets into occ_view[j] = the view that owns occurrence j.
__device__ __forceinline__ void flag(int32_t *failed, int32_t *status, int code) {
  atomicCAS(failed, 0, code);
  atomicCAS(status, 0, code);
}

// The bounds come by value: read again in a loop that writes occ_view, which for all the compiler knows may be the offsets, they
// are a load for every occurrence.
__device__ __forceinline__ bool view_ok(const ViewCheck &views, int i, int32_t &lo, int32_t &hi) {
  lo = views.img_off[i], hi = views.img_off[i + 1];
  return lo >= 0 && lo <= hi && hi <= views.nnz && (i > 0 || lo == 0) && (i < views.B - 1 || hi == views.nnz);
}

// Workgroup `block` of those that check: list by list, then the views.
__device__ __forceinline__ void check_and_count(const CheckTask &t, int block, int *hist /* [pass][digit] */) {
  const int per = t.tiles_per_block * kSortTile;
  int list = 0;
  for (; list < t.gb.count; ++list) {
    const int blocks = (int)(((int64_t)t.gb.p[list].n + per - 1) / per);
    if (block < blocks) break;
    block -= blocks;
  }
  if (list == t.gb.count) {
    const ViewCheck &views = t.views;
    const int i = block * kSortBlock + threadIdx.x;
    if (i >= views.B) return;
    int32_t lo, hi;
    if (!view_ok(views, i, lo, hi)) return flag(t.failed, t.status, GEAR_ERR_RANGE);
    for (int j = lo; j < hi; ++j) views.occ_view[j] = i;
    return;
  }
  const GroupProblem &p = t.gb.p[list];
  const int64_t begin = (int64_t)block * per;
  const int radix = 1 << p.digit_bits, words = p.passes << p.digit_bits;
  for (int d = threadIdx.x; d < words; d += kSortBlock) hist[d] = 0;
  __syncthreads();
  const int64_t end = min((int64_t)p.n, begin + per);
  for (int64_t q0 = begin + threadIdx.x; q0 < end; q0 += kSortTile) {
    int32_t key[kSortItems];
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) key[i] = q0 + i * kSortBlock < end ? p.keys_in[q0 + i * kSortBlock] : 0;
    bool bad = false;
#pragma unroll
    for (int i = 0; i < kSortItems; ++i)
      if (q0 + i * kSortBlock < end) {
        bad |= key[i] < 0 || (int64_t)key[i] >= p.range;
        for (int pass = 0; pass < p.passes; ++pass)
          atomicAdd(&hist[(pass << p.digit_bits) + ((key[i] >> (pass * p.digit_bits)) & (radix - 1))], 1);
      }
    if (bad && p.range > 0) flag(t.failed, t.status, GEAR_ERR_RANGE);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < words; d += kSortBlock)
    if (hist[d]) atomicAdd(&p.totals[d], hist[d]);
}

__host__ __device__ inline int radix_tiles(int n) { return (int)(((int64_t)n + kSortTile - 1) / kSortTile); }

// ---- radix pass: stable scatter ---------------------------------------------------------------------
// A key's place = start of its digit + keys of that digit in earlier tiles + in earlier waves of the tile + in earlier
// rounds of the wave + its rank among the wave's keys of the round (ballots, in lane order).  A wavefront owns 512
// consecutive keys of the tile and counts its digits as it goes, so LDS holds one 16-bit count per wave and digit:
// 6 KB at nine bits, few enough that a workgroup fits on a CU beside one of the matrix-product kernel.
// A thread owns DPT consecutive digits of the scans and of the look-back.
template <int DPT, int WINDOW>
__device__ __forceinline__ void radix_pass(const GroupProblem &p, int pass, int32_t *ticket, bool idle, unsigned char *lds,
                                           int *scan_smem, int *s_tile) {
  constexpr int WAVES = kSortBlock / kWave;
  const int radix = 1 << p.digit_bits, shift = pass * p.digit_bits;
  int *digit_off = reinterpret_cast<int *>(lds);                                   // [radix]
  uint16_t *wave_cnt = reinterpret_cast<uint16_t *>(lds + radix * sizeof(int));    // [wave][radix]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) *s_tile = draw_ticket(ticket);
  const int d0 = tid * DPT;
  const bool owner = d0 < radix;
  int total[DPT];
#pragma unroll
  for (int j = 0; j < DPT; ++j) total[j] = owner && d0 + j < radix ? p.totals[pass * radix + d0 + j] : 0;
  for (int i = tid; i < WAVES * radix / 2; i += kSortBlock) reinterpret_cast<uint32_t *>(wave_cnt)[i] = 0u;
  if (idle) return;
  __syncthreads();
  const int tile = *s_tile, n_tiles = radix_tiles(p.n);
  const int64_t first = (int64_t)tile * kSortTile + wave * (kWave * kSortItems) + lane;
  const int32_t *keys_in = pass == 0 ? p.keys_in : p.keys[pass & 1];
  const int32_t *vals_in = p.vals[pass & 1];
  int32_t key[kSortItems], val[kSortItems], rank[kSortItems];
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const int64_t q = first + i * kWave;
    key[i] = q < p.n ? keys_in[q] : 0;
    val[i] = q < p.n ? (pass == 0 ? (int32_t)q : vals_in[q]) : 0;
  }
  uint16_t *mine = wave_cnt + wave * radix;
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const bool valid = first + i * kWave < p.n;
    const int digit = (key[i] >> shift) & (radix - 1);
    unsigned long long peers = __ballot(valid);
    for (int b = 0; b < p.digit_bits; ++b) {
      const bool bit = (digit >> b) & 1;
      const unsigned long long m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const int lower = __popcll(peers & ((1ull << lane) - 1ull));
    const int before = mine[digit];   // the wave's LDS accesses complete in order: all lanes read, then the first of each digit adds
    __builtin_amdgcn_wave_barrier();
    if (valid && lower == 0) mine[digit] = (uint16_t)(before + __popcll(peers));
    __builtin_amdgcn_wave_barrier();
    rank[i] = before + lower;
  }
  __syncthreads();
  // counts of the tile's digits: published; per wave they become the keys in earlier waves
  int count[DPT];
  uint32_t *row = p.state + ((size_t)pass * (n_tiles - 1) + tile) * radix + d0;
#pragma unroll
  for (int j = 0; j < DPT; ++j) {
    count[j] = 0;
    if (owner && d0 + j < radix) {
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        const int c = wave_cnt[w * radix + d0 + j];
        wave_cnt[w * radix + d0 + j] = (uint16_t)count[j];
        count[j] += c;
      }
      if (tile < n_tiles - 1) publish(row + j, tile == 0 ? kPrefix | (uint32_t)count[j] : 1u + (uint32_t)count[j]);
    }
  }
  int mine_total = 0;
#pragma unroll
  for (int j = 0; j < DPT; ++j) mine_total += total[j];
  int all;
  int base = block_exclusive_scan<WAVES>(mine_total, &all, scan_smem);
  // Look back, kAhead tiles at a time; where the next tile has not published yet, one word of it per open digit until it
  // has.  (The words come past the caches; whole windows asked for over and over by all tiles of a long list took memory
  // bandwidth from the products beside them.)
  constexpr int kAhead = WINDOW >= 2 * DPT ? WINDOW / DPT : 1;
  int before[DPT], look[DPT];
  int open = 0;
#pragma unroll
  for (int j = 0; j < DPT; ++j) {
    before[j] = 0;
    look[j] = owner && d0 + j < radix ? tile - 1 : -1;
    open += look[j] >= 0 ? 1 : 0;
  }
  bool waits = false;
  while (open > 0) {
    uint32_t w[DPT][kAhead];
#pragma unroll
    for (int j = 0; j < DPT; ++j)
#pragma unroll
      for (int a = 0; a < kAhead; ++a)
        w[j][a] = look[j] - a >= 0 && (a == 0 || !waits) ? published(p.state + ((size_t)pass * (n_tiles - 1) + (look[j] - a)) * radix + d0 + j) : 0u;
    const int window = waits ? 1 : kAhead;
    waits = false;
#pragma unroll
    for (int j = 0; j < DPT; ++j) {
      bool go = look[j] >= 0;
#pragma unroll
      for (int a = 0; a < kAhead; ++a) {
        if (a >= window) go = false;
        if (go && w[j][a] == 0u) {
          go = false;
          waits = true;
        }
        if (go) {
          if (w[j][a] & kPrefix) {
            before[j] += (int)(w[j][a] & ~kPrefix);
            look[j] = -1;
            --open;
            go = false;
          } else {
            before[j] += (int)w[j][a] - 1;
            --look[j];   // tile 0 publishes a prefix, so this never passes it
          }
        }
      }
    }
    if (waits) __builtin_amdgcn_s_sleep(8);   // 512 cycles
  }
#pragma unroll
  for (int j = 0; j < DPT; ++j)
    if (owner && d0 + j < radix) {
      if (tile > 0 && tile < n_tiles - 1) publish(row + j, kPrefix | (uint32_t)(before[j] + count[j]));
      digit_off[d0 + j] = base + before[j];
      base += total[j];
    }
  __syncthreads();
  int32_t *keys_out = p.keys[(pass + 1) & 1];
  int32_t *vals_out = p.vals[(pass + 1) & 1];
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    if (first + i * kWave < p.n) {
      const int digit = (key[i] >> shift) & (radix - 1);
      const int pos = digit_off[digit] + mine[digit] + rank[i];
      keys_out[pos] = key[i];
      vals_out[pos] = val[i];
    }
  }
}

// Digits of up to BITS bits: the wide ones (lists whose keys then take a pass less) need more registers, which would
// keep the narrow form off the CUs that a product occupies.
// WINDOW: words in flight of a thread that looks back.
template <int BITS, int WINDOW>
__device__ __forceinline__ void radix_pass_any(const GroupBatch &gb, int list, int pass, bool idle, unsigned char *lds) {
  const GroupProblem &p = gb.p[list];
  if (pass >= p.passes) return;
  __shared__ int scan_smem[8], s_tile;
  int32_t *ticket = gb.tickets + list * kMaxPasses + pass;
  const int digits = (1 << p.digit_bits) / kSortBlock;   // of a thread, at least one
  constexpr int kMost = (1 << BITS) / kSortBlock;
  if constexpr (kMost >= 16)
    if (digits == 16) return radix_pass<16, WINDOW>(p, pass, ticket, idle, lds, scan_smem, &s_tile);
  if constexpr (kMost >= 8)
    if (digits == 8) return radix_pass<8, WINDOW>(p, pass, ticket, idle, lds, scan_smem, &s_tile);
  if constexpr (kMost >= 4)
    if (digits == 4) return radix_pass<4, WINDOW>(p, pass, ticket, idle, lds, scan_smem, &s_tile);
  if constexpr (kMost >= 2)
    if (digits == 2) return radix_pass<2, WINDOW>(p, pass, ticket, idle, lds, scan_smem, &s_tile);
  return radix_pass<1, WINDOW>(p, pass, ticket, idle, lds, scan_smem, &s_tile);
}

// ---- radix pass with counted tiles --------------------------------------------------------------------
// The same scatter where a launch ahead of it has counted every tile's digits (p.state: [pass][tile][digit]).  A tile adds up
// the counts of the tiles before it, many loads at once, instead of looking back at words that come past the caches one after
// the other, and the sort needs no totals.  For what runs beside blocks of views, which is bound by latency: while the blocks
// gather, a load takes microseconds.  us of the launch alone, 36 tiles of 2048 keys 7 to 9, 68 tiles 9 (looking back 10 and 25),
// its count 3 to 5; in a step, of 106 000 ids 10 to 16 and its count 2.5, of 172 000 6 to 29 and 2.5 to 6 (looking back 13 to 18 and
// 20 to 57).  Digits of ten bits then cost about what narrow ones do, so ids of 20 bits take two passes.  Counted by adds to the next
// pass' words while a pass scatters, the most popular ids' words took 20 us of a pass, one add after the other.
// Waves at the highest priority: blocks of views keep the matrix unit busy, not the others, and wait for nobody here.
__device__ __forceinline__ void count_tile(const GroupProblem &p, int pass, int tile, int *hist /* [radix] */) {
  const int radix = 1 << p.digit_bits, shift = pass * p.digit_bits, lane = threadIdx.x & 63;
  const int32_t *keys = pass == 0 ? p.keys_in : p.keys[pass & 1];
  const int64_t q0 = (int64_t)tile * kSortTile + threadIdx.x;
  int32_t key[kSortItems];
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) key[i] = q0 + i * kSortBlock < p.n ? keys[q0 + i * kSortBlock] : 0;
  for (int d = threadIdx.x; d < radix; d += kSortBlock) hist[d] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const bool valid = q0 + i * kSortBlock < p.n;
    const int digit = (key[i] >> shift) & (radix - 1);
    // lanes that share the first one's digit add as one: of a popular image all would, to one word, one after the other
    const bool leads = valid && digit == __builtin_amdgcn_readfirstlane(digit);
    const unsigned long long same = __ballot(leads);
    if (valid && (!leads || (same & ((1ull << lane) - 1ull)) == 0ull)) atomicAdd(&hist[digit], leads ? __popcll(same) : 1);
  }
  __syncthreads();
  uint32_t *row = p.state + ((size_t)pass * radix_tiles(p.n) + tile) * radix;
  for (int d = threadIdx.x; d < radix; d += kSortBlock) row[d] = (uint32_t)hist[d];
}

// A thread owns DPT consecutive digits: four where there are 1024, two of 512, else one.
// VIEWS: the images' last pass, which also leaves where each occurrence's gradient lives.
template <int DPT, bool VIEWS>
__device__ __forceinline__ void counted_pass(const GroupProblem &p, int pass, int tile, int n_views, const PlanArgs &args, int32_t *failed,
                                             unsigned char *lds, int *scan_smem) {
  constexpr int WAVES = kSortBlock / kWave;
  const int radix = 1 << p.digit_bits, shift = pass * p.digit_bits;
  int *digit_off = reinterpret_cast<int *>(lds);                                   // [radix]
  uint16_t *wave_cnt = reinterpret_cast<uint16_t *>(lds + radix * sizeof(int));    // [wave][radix]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int d0 = tid * DPT, n_tiles = radix_tiles(p.n);
  const bool owner = d0 < radix;
  const int64_t first = (int64_t)tile * kSortTile + wave * (kWave * kSortItems) + lane;
  const int32_t *keys_in = pass == 0 ? p.keys_in : p.keys[pass & 1];
  const int32_t *vals_in = p.vals[pass & 1];
  int32_t key[kSortItems], val[kSortItems], rank[kSortItems];
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const int64_t q = first + i * kWave;
    key[i] = q < p.n ? keys_in[q] : 0;
    val[i] = q < p.n ? (pass == 0 ? (int32_t)q : vals_in[q]) : 0;
  }
  for (int i = tid; i < WAVES * radix / 2; i += kSortBlock) reinterpret_cast<uint32_t *>(wave_cnt)[i] = 0u;
  int view[kSortItems];
  float scale[kSortItems];
  if constexpr (VIEWS) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) view[i] = args.occ_view[val[i]];
    __builtin_amdgcn_sched_barrier(0);
  }
  // counts of the tiles before this one and of all
  int before[DPT] = {}, total[DPT] = {};
  const uint32_t *rows = p.state + (size_t)pass * n_tiles * radix + d0;
  if (owner) {
    constexpr int U = DPT == 4 ? 6 : 12;
    for (int t0 = 0; t0 < n_tiles; t0 += U) {
      uint32_t c[U][DPT];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t *row = rows + (size_t)min(t0 + u, n_tiles - 1) * radix;
        if constexpr (DPT == 4) {
          const uint4 v = *reinterpret_cast<const uint4 *>(row);
          c[u][0] = v.x, c[u][1] = v.y, c[u][2] = v.z, c[u][3] = v.w;
        } else if constexpr (DPT == 2) {
          const uint2 v = *reinterpret_cast<const uint2 *>(row);
          c[u][0] = v.x, c[u][1] = v.y;
        } else {
          c[u][0] = row[0];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < DPT; ++j) {
          total[j] += t0 + u < n_tiles ? (int)c[u][j] : 0;
          before[j] += t0 + u < tile ? (int)c[u][j] : 0;
        }
    }
  }
  if (pass == 0 && p.range > 0) {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) bad |= key[i] < 0 || (int64_t)key[i] >= p.range;
    if (bad) flag(failed, args.status, GEAR_ERR_RANGE);
  }
  if constexpr (VIEWS) {
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
      // Where the offsets are no CSR index, which a workgroup of this very launch may be the one to find, an occurrence can be
      // without a view, and its word has whatever was there before: it must not become an address.
      view[i] = (int)min((uint32_t)view[i], (uint32_t)n_views - 1u);
      const int32_t *off = args.img_off + view[i];
      scale[i] = (float)(off[1] - off[0]);
    }
  }
  __syncthreads();
  uint16_t *mine = wave_cnt + wave * radix;
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const bool valid = first + i * kWave < p.n;
    const int digit = (key[i] >> shift) & (radix - 1);
    unsigned long long peers = __ballot(valid);
    for (int b = 0; b < p.digit_bits; ++b) {
      const bool bit = (digit >> b) & 1;
      const unsigned long long m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const int lower = __popcll(peers & ((1ull << lane) - 1ull));
    const int sofar = mine[digit];   // the wave's LDS accesses complete in order: all lanes read, then the first of each digit adds
    __builtin_amdgcn_wave_barrier();
    if (valid && lower == 0) mine[digit] = (uint16_t)(sofar + __popcll(peers));
    __builtin_amdgcn_wave_barrier();
    rank[i] = sofar + lower;
  }
  int mine_total = 0;
#pragma unroll
  for (int j = 0; j < DPT; ++j) mine_total += total[j];
  int all;
  int base = block_exclusive_scan<WAVES>(mine_total, &all, scan_smem);   // and every wave has counted its digits
#pragma unroll
  for (int j = 0; j < DPT; ++j)
    if (owner) {
      int count = 0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        const int c = wave_cnt[w * radix + d0 + j];
        wave_cnt[w * radix + d0 + j] = (uint16_t)count;
        count += c;
      }
      digit_off[d0 + j] = base + before[j];
      base += total[j];
    }
  __syncthreads();
  int32_t *keys_out = p.keys[(pass + 1) & 1];
  int32_t *vals_out = p.vals[(pass + 1) & 1];
#pragma unroll
  for (int i = 0; i < kSortItems; ++i)
    if (first + i * kWave < p.n) {
      const int digit = (key[i] >> shift) & (radix - 1);
      const int pos = digit_off[digit] + mine[digit] + rank[i];
      keys_out[pos] = key[i];
      vals_out[pos] = val[i];
      if constexpr (VIEWS) {
        args.plan.row_view[pos] = view[i];
        args.plan.row_scale[pos] = 1.0f / scale[i];
      }
    }
}

// ---- segments of the sorted keys and the plan of the windowed accumulation -------------------------------
// Section 1, third point: the gradients of one image are collected until M have arrived, then
// averaged.  With c gradients already collected in earlier steps, the occurrence at in-step rank r
// has ordinal k = c + r; ordinals kM .. kM+M-1 form one group.  A "unit" is the work of one
// workgroup: the first (possibly partial, possibly continuing) group of an image together with its
// unfinished last group, or one complete middle group.  An "emission" is a completed group.

// A thread owns the eight consecutive positions tile0 + 8 t .. + 7.  All loads that do not depend on each other are
// requested together and none is behind a branch; the chain is ticket -> keys -> counters, start and end of the
// segments that cross the tile's borders -> flags -> look-back -> descriptors.
// VIEWS: and where each occurrence's gradient lives, unless the last pass has left that.
template <bool PLAN, bool VIEWS>
__device__ __forceinline__ void segments(const GroupBatch &gb, const PlanArgs &args, int block, int32_t *failed) {
  const bool idle = *failed != 0;
  const GroupProblem &p = gb.p[gb.count - 1];
  const AccumPlan &plan = args.plan;
  uint32_t *state = gb.seg_state;
  const int32_t *__restrict__ occ_view = args.occ_view, *__restrict__ img_off = args.img_off, *__restrict__ counts = args.counts;
  const int M = args.M;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (p.n <= 0) {
    if (!idle && block == 0 && tid == 0) {
      *p.n_unique = 0;
      if (p.segoff) p.segoff[0] = 0;
      if (PLAN) {
        *plan.n_units = 0;
        *args.n_ready = 0;
      }
    }
    return;
  }
  __shared__ int s_tile, s_edge[2], s_last[4], s_first[4];
  __shared__ unsigned long long s_sum[4];
  __shared__ int s_base[3];
  if (tid == 0) s_tile = draw_ticket(gb.tickets + kTickets - 1);
  if (idle) return;
  __syncthreads();
  const int n = p.n, n_tiles = (n + kSortTile - 1) / kSortTile, tile = s_tile;
  const int tile0 = tile * kSortTile, tile1 = min(n - tile0, kSortTile) + tile0;
  const int32_t *__restrict__ sk = p.sorted_keys;
  const int64_t q0 = (int64_t)tile0 + tid * kSortItems;

  int key[kSortItems];
  const bool whole = q0 + kSortItems <= n;
  if (whole) {
    const int4 a = *reinterpret_cast<const int4 *>(sk + q0), b = *reinterpret_cast<const int4 *>(sk + q0 + 4);
    key[0] = a.x, key[1] = a.y, key[2] = a.z, key[3] = a.w, key[4] = b.x, key[5] = b.y, key[6] = b.z, key[7] = b.w;
  } else {
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) key[i] = sk[min(q0 + i, (int64_t)n - 1)];
  }
  const int key_before = q0 > 0 && q0 < n ? sk[q0 - 1] : -1;
  int view[kSortItems], far_key[kSortItems], cnt[kSortItems];
  if constexpr (PLAN && VIEWS) {
    if (whole) {
      const int4 a = *reinterpret_cast<const int4 *>(p.perm + q0), b = *reinterpret_cast<const int4 *>(p.perm + q0 + 4);
      view[0] = a.x, view[1] = a.y, view[2] = a.z, view[3] = a.w, view[4] = b.x, view[5] = b.y, view[6] = b.z, view[7] = b.w;
    } else {
#pragma unroll
      for (int i = 0; i < kSortItems; ++i) view[i] = p.perm[min(q0 + i, (int64_t)n - 1)];
    }
  }
  if constexpr (PLAN) {
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) far_key[i] = sk[min(q0 + i + M - 1, (int64_t)n - 1)];
    __builtin_amdgcn_sched_barrier(0);   // requests stay in flight, their addresses need not
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) cnt[i] = counts[key[i]];
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (PLAN && VIEWS) {
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) view[i] = occ_view[view[i]];
    __builtin_amdgcn_sched_barrier(0);
  }
  // the segments that the tile's first and last keys belong to may begin before the tile and end behind it
  if (wave == 0) {
    const int k = sk[tile0];
    const int s = tile0 > 0 && sk[tile0 - 1] == k ? wave_search(sk, 0, tile0, k, false, lane) : tile0;
    if (lane == 0) s_edge[0] = s;
  } else if (wave == 1) {
    const int k = sk[tile1 - 1];
    const int s = tile1 < n && sk[tile1] == k ? wave_search(sk, tile1, n, k, true, lane) : tile1;
    if (lane == 0) s_edge[1] = s;
  }
  bool head[kSortItems];
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) head[i] = q0 + i < n && (q0 + i == 0 || key[i] != (i == 0 ? key_before : key[i - 1]));

  // last head at or before each position and first head behind it, over the tile
  int last = -1, first = INT32_MAX;
#pragma unroll
  for (int i = 0; i < kSortItems; ++i)
    if (head[i]) {
      last = (int)(q0 + i);
      if (first == INT32_MAX) first = last;
    }
  int run_last = last, run_first = first;   // inclusive scans over the wave, from below and from above
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int a = __shfl_up(run_last, off, kWave), b = __shfl_down(run_first, off, kWave);
    if (lane >= off) run_last = max(run_last, a);
    if (lane + off < kWave) run_first = min(run_first, b);
  }
  if (lane == 63) s_last[wave] = run_last;
  if (lane == 0) s_first[wave] = run_first;
  int seg0 = __shfl_up(run_last, 1, kWave), seg1 = __shfl_down(run_first, 1, kWave);
  if (lane == 0) seg0 = -1;
  if (lane == 63) seg1 = INT32_MAX;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (w < wave) seg0 = max(seg0, s_last[w]);
    if (w > wave) seg1 = min(seg1, s_first[w]);
  }
  if (seg0 < 0) seg0 = s_edge[0];
  if (seg1 == INT32_MAX) seg1 = s_edge[1];

  // flags; heads, units and emissions are counted together, 21 bits each
  bool unit[kSortItems], emit[kSortItems];
  int seg = seg0;   // start of the segment at each position
  unsigned long long sum = 0;
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const int64_t q = q0 + i;
    if (head[i]) seg = (int)q;
    unit[i] = emit[i] = false;
    if constexpr (PLAN) {
      if (q < n) {
        const int ph = (cnt[i] + (int)(q - seg)) % M;
        unit[i] = head[i] || (ph == 0 && M <= n - q && far_key[i] == key[i]);
        emit[i] = ph == M - 1;
      }
    }
    sum += (head[i] ? 1ull : 0ull) + (unit[i] ? 1ull << 21 : 0ull) + (emit[i] ? 1ull << 42 : 0ull);
    if constexpr (PLAN) __builtin_amdgcn_sched_barrier(0);   // one division at a time: registers
  }
  unsigned long long inc = sum;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const unsigned long long t = __shfl_up(inc, off, kWave);
    if (lane >= off) inc += t;
  }
  if (lane == 63) s_sum[wave] = inc;
  __syncthreads();
  unsigned long long below = inc - sum, all = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (w < wave) below += s_sum[w];
    all += s_sum[w];
  }
  constexpr int kMask = (1 << 21) - 1;
  const int own[3] = {(int)(all & kMask), (int)((all >> 21) & kMask), (int)(all >> 42)};
  if (tid == 0 && tile < n_tiles - 1)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      publish(state + 3 * (size_t)tile + c, tile == 0 ? kPrefix | (uint32_t)own[c] : 1u + (uint32_t)own[c]);

  if constexpr (PLAN && VIEWS) {
    // where the occurrence's gradient lives: dLoss/dx of its view, divided by the view's image count
    float scale[kSortItems];
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
      const int32_t *off = img_off + view[i];
      scale[i] = (float)(off[1] - off[0]);
    }
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
      scale[i] = 1.0f / scale[i];
      __builtin_amdgcn_sched_barrier(0);
    }
    if (whole) {
      *reinterpret_cast<int4 *>(plan.row_view + q0) = make_int4(view[0], view[1], view[2], view[3]);
      *reinterpret_cast<int4 *>(plan.row_view + q0 + 4) = make_int4(view[4], view[5], view[6], view[7]);
      *reinterpret_cast<float4 *>(plan.row_scale + q0) = make_float4(scale[0], scale[1], scale[2], scale[3]);
      *reinterpret_cast<float4 *>(plan.row_scale + q0 + 4) = make_float4(scale[4], scale[5], scale[6], scale[7]);
    } else {
#pragma unroll
      for (int i = 0; i < kSortItems; ++i)
        if (q0 + i < n) {
          plan.row_view[q0 + i] = view[i];
          plan.row_scale[q0 + i] = scale[i];
        }
    }
  }

  if (wave == 0) {
    // look back 64 tiles at a time; a tile counts once all three of its words are of one kind
    int before[3] = {0, 0, 0};
    int look = tile - 1;
    while (look >= 0) {
      uint32_t w[3];
      const int at = look - lane;
#pragma unroll
      for (int c = 0; c < 3; ++c) w[c] = at >= 0 ? published(state + 3 * (size_t)at + c) : kPrefix;
      const bool there = w[0] != 0u && w[1] != 0u && w[2] != 0u;
      const bool prefix = (w[0] & w[1] & w[2] & kPrefix) != 0u;
      const bool alone = there && ((w[0] | w[1] | w[2]) & kPrefix) == 0u;
      // lanes before the first that is not a lone count; that one too if it is a prefix
      const unsigned long long stop = ~__ballot(alone), pre = __ballot(prefix);
      const int upto = stop ? __builtin_ctzll(stop) : kWave;
      const bool done = upto < kWave && ((pre >> upto) & 1ull);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        int v = lane < upto ? (int)w[c] - 1 : (done && lane == upto ? (int)(w[c] & ~kPrefix) : 0);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
        before[c] += v;
      }
      if (done) break;
      look -= upto;
      if (upto == 0) __builtin_amdgcn_s_sleep(8);
    }
    if (lane < 3) {
      const int b = lane == 0 ? before[0] : lane == 1 ? before[1] : before[2];
      const int o = lane == 0 ? own[0] : lane == 1 ? own[1] : own[2];
      s_base[lane] = b;
      if (tile > 0 && tile < n_tiles - 1) publish(state + 3 * (size_t)tile + lane, kPrefix | (uint32_t)(b + o));
    }
  }
  __syncthreads();
  int h = s_base[0] + (int)(below & kMask), u = s_base[1] + (int)((below >> 21) & kMask), e = s_base[2] + (int)(below >> 42);
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const int64_t q = q0 + i;
    if (head[i] && p.unique) {
      p.unique[h] = key[i];
      p.segoff[h] = (int)q;
    }
    h += head[i] ? 1 : 0;
    if (head[i]) seg0 = (int)q;
    if constexpr (PLAN) {
      if (unit[i]) {
        int end = seg1;   // of the unit's segment: the next head of this thread, or what follows it
#pragma unroll
        for (int j = kSortItems - 1; j > i; --j)
          if (head[j]) end = (int)(q0 + j);
        UnitDesc d;
        d.q0 = (int)q;
        d.image = key[i];
        d.slot = e;
        d.s0 = seg0;
        d.s1 = end;
        d.phase = cnt[i] % M;
        d.collected = cnt[i] + (end - seg0);
        d.pad = 0;
        plan.units[u] = d;
        ++u;
      }
      e += emit[i] ? 1 : 0;
    }
  }
  if (tile == n_tiles - 1 && tid == 0) {
    *p.n_unique = s_base[0] + own[0];
    if (p.unique) p.segoff[s_base[0] + own[0]] = n;
    if constexpr (PLAN) {
      *plan.n_units = s_base[1] + own[1];
      // a list that does not fit is reported as empty: nobody may read ready_ids past ready_cap.  Every other tile has
      // read `failed` by now: it did so before it published the counts that this one has seen
      const int emits = s_base[2] + own[2];
      *args.n_ready = emits > args.ready_cap ? 0 : emits;
      if (emits > args.ready_cap) flag(failed, args.status, GEAR_ERR_CAPACITY);
    }
  }
}

// ---- the grouping as a passenger ---------------------------------------------------------------------
// A short step has no use for a second stream: the events alone cost more than there is to hide.  Its grouping is a chain
// of small launches that the forward pass does not wait for, nor the other way round, so each link rides in the first
// workgroups of a launch that goes out anyway: the check with the gather, a pass or the segments with a product or the
// logit layer.  Workgroups have kSortBlock threads in all of them.
// lds: 12 bytes per digit of the widest list's radix
__device__ __forceinline__ void side_work(const SideTask &t, int block, unsigned char *lds) {
  if (t.kind == SideTask::kSegments) {
    const int n = t.gb.p[t.gb.count - 1].n;
    if (block < max(1, (int)(((int64_t)n + kSortTile - 1) / kSortTile))) segments<true, true>(t.gb, t.plan, block, t.failed);
    return;
  }
  const bool idle = *t.failed != 0;
  for (int list = 0; list < t.gb.count; ++list) {
    const int tiles = radix_tiles(t.gb.p[list].n);
    if (block < tiles) return radix_pass_any<kSideDigitBits, 16>(t.gb, list, t.pass, idle, lds);
    block -= tiles;
  }
}

}  // namespace
}  // namespace gear
