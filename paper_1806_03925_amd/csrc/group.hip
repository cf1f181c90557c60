// Sort-by-key grouping of a step's ids, and the plan of the per-image accumulation.
//
// The Sparse Part's gradients are applied per embedding row (Section 3, step 4) and the DFV
// gradients are collected per image id (Section 3, steps 5-6).  Both need "all positions that
// carry the same id, in their original order": a stable LSD radix sort of (id, position) pairs, and for the images a
// head-flag scan that gives the segments.  Up to three id lists (users, URLs, images) go through the same launches.
//
// What bounds this is not bytes but the chain: every launch costs its ramp, a fetch of cold arguments and one or two
// memory latencies (4 to 6 us on lists of a few thousand ids) before it has done anything.  So the chain is as short as
// it can be made: one launch checks the ids and counts the digits of all passes (the counts do not depend on the
// order of the keys), a pass is one launch, and the segments and the plan are one.  Where a tile needs what earlier
// tiles counted it looks back at words they publish (below) instead of waiting for another launch.  With three launches
// per pass, two for the segments, two for the plan and one for the counters, lists of 4096 users and URLs and 18 000
// images took 15 launches and 113 us alone on the device; now 4 and 45 us.
//
// Everything here is integer work whose result does not depend on scheduling: digit counts are
// integer sums, ranks come from wave ballots in lane order, scans run in a fixed shape.
#include "group_device.hpp"

namespace gear {
namespace {

// sum of tile_vals[0 .. tile) for tile <= 256 * 4, computed by the whole workgroup
__device__ __forceinline__ int sum_before(const int32_t *tile_vals, int tile, int *smem) {
  int v = 0;
  for (int t = threadIdx.x; t < tile; t += blockDim.x) v += tile_vals[t];
  int total;
  block_exclusive_scan(v, &total, smem);
  return total;
}

// ---- expiry of cached inference results ------------------------------------------------------------
// Every occurrence whose cached row is old writes a 1 into its image's byte of a map over all images
// (a plain store of the same value, whoever comes first; an atomic OR into a bitmap was tried and
// spent 260 us on the thousands of occurrences of the most popular image, all aimed at one word);
// the marked bytes are then counted per tile and written out in ascending order at the tile's
// offset.  No sort is needed: the map is already in id order.
__device__ __forceinline__ bool is_expired(const int32_t *__restrict__ stamp, int64_t n_images, int id, int32_t now,
                                           int32_t expiry, int32_t *status) {
  if (id < 0 || id >= n_images) {
    atomicCAS(status, 0, GEAR_ERR_RANGE);
    return false;
  }
  return (int64_t)now - (int64_t)stamp[id] >= (int64_t)expiry;
}

__global__ void __launch_bounds__(256) k_expired_mark(const int32_t *__restrict__ ids, int n,
                                                      const int32_t *__restrict__ stamp, int64_t n_images, int32_t now,
                                                      int32_t expiry, uint8_t *__restrict__ marks, int32_t *status) {
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < n; r += gridDim.x * blockDim.x) {
    const int id = ids[r];
    if (is_expired(stamp, n_images, id, now, expiry, status)) marks[id] = 1;
  }
}

// The map is read as words of four images; thread t of a tile owns the words tile0 + 8 t .. + 7, so a
// scan keeps id order.  The map is padded with zeros to a whole number of words.
__global__ void __launch_bounds__(kSortBlock) k_expired_count(const uint32_t *__restrict__ marks, int64_t n_words,
                                                              int32_t *__restrict__ tile_counts) {
  const int64_t tile0 = (int64_t)blockIdx.x * kSortTile;
  __shared__ int smem[8];
  int c = 0;
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const int64_t w = tile0 + threadIdx.x * kSortItems + i;
    if (w < n_words) c += __popc(marks[w]);
  }
  int total;
  block_exclusive_scan(c, &total, smem);
  if (threadIdx.x == 0) tile_counts[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kSortBlock) k_expired_scatter(const uint32_t *__restrict__ marks, int64_t n_words,
                                                                const int32_t *__restrict__ tile_counts,
                                                                int32_t *__restrict__ out_ids, int32_t *n_out,
                                                                const int32_t *status) {
  const int64_t tile0 = (int64_t)blockIdx.x * kSortTile;
  __shared__ int smem[8];
  const int base = sum_before(tile_counts, blockIdx.x, smem);
  uint32_t word[kSortItems];
  int c = 0;
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const int64_t w = tile0 + threadIdx.x * kSortItems + i;
    word[i] = w < n_words ? marks[w] : 0u;
    c += __popc(word[i]);
  }
  int total;
  int at = base + block_exclusive_scan(c, &total, smem);
  const bool bad = *status != 0;   // set by the marking pass, which saw every id: the list is then empty
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const int64_t w = tile0 + threadIdx.x * kSortItems + i;
#pragma unroll
    for (int byte = 0; byte < 4; ++byte)
      if (word[i] & (1u << (8 * byte))) {
        if (!bad) out_ids[at] = (int32_t)(w * 4 + byte);
        ++at;
      }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *n_out = bad ? 0 : base + total;
}

__global__ void __launch_bounds__(256) k_stamp(int32_t *__restrict__ stamp, int64_t n_images,
                                               const int32_t *__restrict__ ids, int64_t n, int32_t now, int32_t *status,
                                               const int32_t *__restrict__ n_dev) {
  if (n_dev) n = min((int64_t)max(*n_dev, 0), n);  // the row count is only known on the device
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
    const int64_t id = ids ? (int64_t)ids[r] : r;
    if (id < 0 || id >= n_images) {
      if (status) atomicCAS(status, 0, GEAR_ERR_RANGE);
      continue;
    }
    stamp[id] = now;
  }
}

}  // namespace

hipError_t launch_expired(const int32_t *image_ids, int n, const int32_t *stamp, int64_t n_images, int32_t now,
                          int32_t expiry, uint8_t *marks, int32_t *tile_counts, int32_t *out_ids, int32_t *n_out,
                          int32_t *status, hipStream_t s) {
  const int64_t n_words = expiry_words(n_images);
  hipError_t e = launch_fill_zero(marks, (size_t)n_words * sizeof(uint32_t), s);
  if (e != hipSuccess) return e;
  if (n > 0) {
    int blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_expired_mark, dim3(blocks), dim3(256), 0, s, image_ids, n, stamp, n_images, now, expiry, marks,
                       status);
  }
  const int tiles = (int)expiry_tiles(n_images);
  hipLaunchKernelGGL(k_expired_count, dim3(tiles), dim3(kSortBlock), 0, s, (const uint32_t *)marks, n_words,
                     tile_counts);
  hipLaunchKernelGGL(k_expired_scatter, dim3(tiles), dim3(kSortBlock), 0, s, (const uint32_t *)marks, n_words,
                     tile_counts, out_ids, n_out, status);
  return hipGetLastError();
}

hipError_t launch_stamp(int32_t *stamp, int64_t n_images, const int32_t *ids, int64_t n, int32_t now, int32_t *status,
                        hipStream_t s, const int32_t *n_dev) {
  if (n <= 0) return hipSuccess;
  int64_t want = (n + 255) / 256;
  const int blocks = (int)(want < 4096 ? want : 4096);
  hipLaunchKernelGGL(k_stamp, dim3(blocks), dim3(256), 0, s, stamp, n_images, ids, n, now, status, n_dev);
  return hipGetLastError();
}

namespace {
// by one workgroup: a copy for callers who look at the grouping itself
__global__ void __launch_bounds__(256) k_unique(LocalResult local, const int32_t *unique, const int32_t *segoff, int n, int32_t *out_unique,
                                                int32_t *out_segoff, int32_t *out_n) {
  int at = 0;
  for (int part = 0; part < local.n_parts; ++part) {
    const PartCounts c = local.parts[part];
    for (int i = threadIdx.x; i < c.heads; i += 256) {
      if (out_unique) out_unique[at + i] = unique[c.below + i];
      if (out_segoff) out_segoff[at + i] = segoff[c.below + i];
    }
    at += c.heads;
  }
  if (threadIdx.x == 0) {
    if (out_segoff) out_segoff[at] = n;
    if (out_n) *out_n = at;
  }
}
}  // namespace

hipError_t launch_unique(const LocalResult &local, const int32_t *unique, const int32_t *segoff, int n, int32_t *out_unique, int32_t *out_segoff,
                         int32_t *out_n, hipStream_t s) {
  if ((out_unique && !unique) || (out_segoff && !segoff)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_unique, dim3(1), dim3(256), 0, s, local, unique, segoff, n, out_unique, out_segoff, out_n);
  return hipGetLastError();
}

// What the grouping counts in has to be zero first.
void group_zero_list(const GroupBatch &gb, ZeroList *z) {
  z->count = 0;
  auto add = [&](void *p, int64_t words) {
    if (words > 0) z->p[z->count] = (uint32_t *)p, z->words[z->count++] = words;
  };
  add(gb.tickets, kTickets);
  for (int i = 0; i < gb.count; ++i) {
    const GroupProblem &p = gb.p[i];
    const int64_t words = (int64_t)p.passes << p.digit_bits;
    add(p.totals, words);
    add(p.state, (radix_tiles(p.n) - 1) * words);
  }
  const GroupProblem &last = gb.p[gb.count - 1];
  add(gb.seg_state, 3 * (((int64_t)last.n + kSortTile - 1) / kSortTile - 1));
}

// A workgroup that checks takes one tile of a short list, so that as many CUs as possible work on it, and four tiles of a
// long one, so that fewer workgroups add to the digits' totals (a list of more than 65 536 ids has 32 tiles and more).
CheckTask check_task(const GroupBatch &gb, const int32_t *img_off, int32_t *occ_view, int B, int nnz, int32_t *failed,
                     int32_t *status) {
  CheckTask t;
  t.gb = gb;
  t.views = ViewCheck{img_off, occ_view, B, nnz};
  t.failed = failed;
  t.status = status;
  t.tiles_per_block = 1;
  for (int i = 0; i < gb.count; ++i)
    if (gb.p[i].n > kLongList) t.tiles_per_block = 4;
  t.blocks = (B + kSortBlock - 1) / kSortBlock;
  for (int i = 0; i < gb.count; ++i)
    t.blocks += (int)(((int64_t)gb.p[i].n + t.tiles_per_block * kSortTile - 1) / (t.tiles_per_block * kSortTile));
  return t;
}
int check_lds_bytes(const GroupBatch &gb) {
  int words = 0;
  for (int i = 0; i < gb.count; ++i)
    if (gb.p[i].passes << gb.p[i].digit_bits > words) words = gb.p[i].passes << gb.p[i].digit_bits;
  return words * (int)sizeof(int);
}
int group_passes(const GroupBatch &gb) {
  int passes = 0;
  for (int i = 0; i < gb.count; ++i)
    if (gb.p[i].n > 0 && gb.p[i].passes > passes) passes = gb.p[i].passes;
  return passes;
}
static int widest_radix(const GroupBatch &gb) {
  int radix = 0;
  for (int i = 0; i < gb.count; ++i)
    if (1 << gb.p[i].digit_bits > radix) radix = 1 << gb.p[i].digit_bits;
  return radix;
}
int radix_lds_bytes(const GroupBatch &gb) { return (int)(sizeof(int) + kSortBlock / kWave * sizeof(uint16_t)) * widest_radix(gb); }

SideTask side_task(const GroupBatch &gb, const PlanArgs &plan, int step, int32_t *failed) {
  SideTask t;
  t.kind = step < group_passes(gb) ? SideTask::kPass : SideTask::kSegments;
  t.pass = step;
  t.gb = gb;
  t.plan = plan;
  t.failed = failed;
  t.blocks = 0;
  if (t.kind == SideTask::kPass)
    for (int i = 0; i < gb.count; ++i) t.blocks += radix_tiles(gb.p[i].n);
  else
    t.blocks = (int)(((int64_t)gb.p[gb.count - 1].n + kSortTile - 1) / kSortTile);
  t.blocks = (t.blocks + 7) / 8 * 8;
  if (t.blocks == 0) t.blocks = 8;
  return t;
}

namespace {
__global__ void __launch_bounds__(kSortBlock) k_check_and_count(CheckTask t) {
  extern __shared__ int hist[];
  check_and_count(t, blockIdx.x, hist);
}

// What runs beside the products of a long step has to fit on a CU that one of their workgroups is on: two wavefronts a SIMD
// of 200 registers leave 112 (gemm.hip).  A workgroup that needs more keeps the next tile of a product waiting: a step of
// 65 536 views took 991 us with 114 registers here and 123 in k_segments, 985 with 102 and 116, 973 with 102 and 96 (and a
// dozen spilled).
template <int BITS>
__global__ void __launch_bounds__(kSortBlock) k_radix_pass(GroupBatch gb, int pass, const int32_t *failed) {
  const bool idle = *failed != 0;
  if ((int)blockIdx.x >= radix_tiles(gb.p[blockIdx.y].n)) return;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  radix_pass_any<BITS, BITS <= 9 ? 4 : 16>(gb, blockIdx.y, pass, idle, lds);
}

// 96 registers in the passes and the segments: five waves' worth, which find a place beside four of a block's 96 on a SIMD whatever
// was there before (with 128 the first pass waited 40 us for one to end).
__global__ void __launch_bounds__(kSortBlock) k_count(GroupBatch gb, int pass) {
  const GroupProblem &p = gb.p[blockIdx.y];
  if (pass >= p.passes || (int)blockIdx.x >= radix_tiles(p.n)) return;
  __builtin_amdgcn_s_setprio(3);
  extern __shared__ int hist[];
  count_tile(p, pass, blockIdx.x, hist);
}

__global__ void __launch_bounds__(kSortBlock, 5) k_counted_pass(GroupBatch gb, int pass, ViewCheck views, PlanArgs args, int32_t *failed) {
  if ((int)blockIdx.y == gb.count) {
    int32_t lo, hi;
    for (int i = blockIdx.x * kSortBlock + threadIdx.x; i < views.B; i += gridDim.x * kSortBlock)
      if (!view_ok(views, i, lo, hi)) flag(failed, args.status, GEAR_ERR_RANGE);
    return;
  }
  const GroupProblem &p = gb.p[blockIdx.y];
  if (pass >= p.passes || (int)blockIdx.x >= radix_tiles(p.n)) return;
  __builtin_amdgcn_s_setprio(3);
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  __shared__ int scan_smem[8];
  const bool last = (int)blockIdx.y == gb.count - 1 && pass == p.passes - 1;
#define GEAR_COUNTED(DPT)                                                                  \
  if (last)                                                                                \
    counted_pass<DPT, true>(p, pass, blockIdx.x, views.B, args, failed, lds, scan_smem);   \
  else                                                                                     \
    counted_pass<DPT, false>(p, pass, blockIdx.x, views.B, args, failed, lds, scan_smem)
  if (p.digit_bits == 10) {
    GEAR_COUNTED(4);
  } else if (p.digit_bits == 9) {
    GEAR_COUNTED(2);
  } else {
    GEAR_COUNTED(1);
  }
#undef GEAR_COUNTED
}

template <bool PLAN, bool BESIDE>
__global__ void __launch_bounds__(kSortBlock, BESIDE ? 5 : 1) k_segments(GroupBatch gb, PlanArgs args, int32_t *failed) {
  segments<PLAN, true>(gb, args, blockIdx.x, failed);
}

// behind counted passes, with the counts of the other lists' next pass
__global__ void __launch_bounds__(kSortBlock, 5) k_segments_count(GroupBatch gb, PlanArgs args, int pass, int32_t *failed) {
  __builtin_amdgcn_s_setprio(3);
  if ((int)blockIdx.y == 0) {
    const int tiles = radix_tiles(gb.p[gb.count - 1].n);
    if ((int)blockIdx.x < (tiles < 1 ? 1 : tiles)) segments<true, false>(gb, args, blockIdx.x, failed);
    return;
  }
  const GroupProblem &p = gb.p[blockIdx.y - 1];
  if (pass >= p.passes || (int)blockIdx.x >= radix_tiles(p.n)) return;
  extern __shared__ int hist[];
  count_tile(p, pass, blockIdx.x, hist);
}
}  // namespace

hipError_t launch_check(const GroupBatch &gb, const int32_t *img_off, int32_t *occ_view, int B, int nnz, int32_t *failed,
                        int32_t *status, hipStream_t s) {
  const CheckTask t = check_task(gb, img_off, occ_view, B, nnz, failed, status);
  if (t.blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_check_and_count, dim3(t.blocks), dim3(kSortBlock), check_lds_bytes(gb), s, t);
  return hipGetLastError();
}

hipError_t launch_radix_pass(const GroupBatch &gb, int pass, const int32_t *failed, hipStream_t s) {
  int tiles = 0;
  for (int i = 0; i < gb.count; ++i)
    if (radix_tiles(gb.p[i].n) > tiles) tiles = radix_tiles(gb.p[i].n);
  if (tiles == 0) return hipSuccess;
  if (widest_radix(gb) > 512)
    hipLaunchKernelGGL(k_radix_pass<kMaxDigitBits>, dim3(tiles, gb.count), dim3(kSortBlock), radix_lds_bytes(gb), s, gb, pass, failed);
  else
    hipLaunchKernelGGL(k_radix_pass<9>, dim3(tiles, gb.count), dim3(kSortBlock), radix_lds_bytes(gb), s, gb, pass, failed);
  return hipGetLastError();
}

int counted_passes(int bits, int n, int cap, int widest) {
  const size_t tiles = radix_tiles(n);
  for (int passes = 1; passes <= kMaxPasses; ++passes) {
    const int digit_bits = (bits + passes - 1) / passes;
    if (digit_bits <= widest && (tiles * passes << digit_bits) <= 3 * (size_t)cap) return passes;
  }
  return 0;
}
int counted_lds_bytes(int digit_bits) { return ((int)(sizeof(int) + kSortBlock / kWave * sizeof(uint16_t)) << digit_bits) + 1280; }

static int most_tiles(const GroupBatch &gb, int pass) {
  int tiles = 0;
  for (int i = 0; i < gb.count; ++i)
    if (pass < gb.p[i].passes && radix_tiles(gb.p[i].n) > tiles) tiles = radix_tiles(gb.p[i].n);
  return tiles;
}

static int counted_digits_ok(const GroupBatch &gb) {
  for (int i = 0; i < gb.count; ++i)
    if (gb.p[i].digit_bits > kCountedDigitBits) return 0;   // counted_pass
  return 1;
}

FirstCounts first_counts(const GroupBatch &gb, const ViewCheck &views) {
  FirstCounts f;
  f.gb = gb;
  f.views = views;
  int blocks = 0;
  for (int i = 0; i < kMaxProblems; ++i) {
    f.first_block[i] = blocks;
    if (i < gb.count) blocks += radix_tiles(gb.p[i].n);
  }
  f.first_block[kMaxProblems] = blocks;
  return f;
}

// what the segments publish in
void counted_zero_list(const GroupBatch &gb, ZeroList *z) {
  z->count = 1;
  z->p[0] = (uint32_t *)(gb.tickets + kTickets - 1);
  z->words[0] = 1;
  const int64_t words = 3 * ((int64_t)radix_tiles(gb.p[gb.count - 1].n) - 1);
  if (words > 0) z->p[1] = gb.seg_state, z->words[z->count++] = words;
}

hipError_t launch_count(const GroupBatch &gb, int pass, hipStream_t s) {
  if (!counted_digits_ok(gb)) return hipErrorInvalidValue;
  const int tiles = most_tiles(gb, pass);
  if (tiles == 0) return hipSuccess;
  hipLaunchKernelGGL(k_count, dim3(tiles, gb.count), dim3(kSortBlock), widest_radix(gb) * sizeof(int), s, gb, pass);
  return hipGetLastError();
}

hipError_t launch_counted_pass(const GroupBatch &gb, int pass, const ViewCheck &views, const PlanArgs &args, int32_t *failed, hipStream_t s,
                               hipEvent_t stop) {
  if (!counted_digits_ok(gb)) return hipErrorInvalidValue;
  const int tiles = most_tiles(gb, pass);
  if (tiles == 0) return leave(stop, s);
  launch_leaving(stop, k_counted_pass, dim3(tiles, gb.count + (pass == 0 ? 1 : 0)), kSortBlock, radix_lds_bytes(gb), s, gb, pass, views,
                 args, failed);
  return hipGetLastError();
}

// the plan of the last list, and the counts of the others' pass `next` where they have one
hipError_t launch_segments_count(const GroupBatch &gb, const PlanArgs &args, int next, int32_t *failed, hipStream_t s, hipEvent_t stop) {
  int tiles = radix_tiles(gb.p[gb.count - 1].n), others = 0;
  if (tiles < 1) tiles = 1;
  for (int i = 0; i + 1 < gb.count; ++i)
    if (next < gb.p[i].passes) {
      others = gb.count - 1;
      if (radix_tiles(gb.p[i].n) > tiles) tiles = radix_tiles(gb.p[i].n);
    }
  launch_leaving(stop, k_segments_count, dim3(tiles, 1 + others), kSortBlock, widest_radix(gb) * sizeof(int), s, gb, args, next, failed);
  return hipGetLastError();
}

// segments of the last list; with `args` also the plan of the accumulation
hipError_t launch_segments(const GroupBatch &gb, const PlanArgs *args, int32_t *failed, hipStream_t s, hipEvent_t stop) {
  const int tiles = (int)(((int64_t)gb.p[gb.count - 1].n + kSortTile - 1) / kSortTile);
  // Beside the large products of a long step: few registers (96 instead of 116, of which 14 spill, 60 bytes of scratch), so
  // that a workgroup fits on a product's CU.  The list's length decides, not the products: a long list beside products of
  // moderate size takes as long either way (us a step, few registers / all: 16 384 views in bf16 175.6 / 175.9, 139 000
  // occurrences in fp32 180.1 / 179.2; 65 536 views beside large products 986 / 997).  With a shorter one nothing needs the
  // room.
  const dim3 grid(tiles < 1 ? 1 : tiles);
  if (!args)
    launch_leaving(stop, k_segments<false, false>, grid, kSortBlock, 0, s, gb, PlanArgs{}, failed);
  else if (gb.p[gb.count - 1].n > kLongList)
    launch_leaving(stop, k_segments<true, true>, grid, kSortBlock, 0, s, gb, *args, failed);
  else
    launch_leaving(stop, k_segments<true, false>, grid, kSortBlock, 0, s, gb, *args, failed);
  return hipGetLastError();
}

}  // namespace gear
