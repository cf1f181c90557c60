// Step prologue, one launch: reset the per-step outputs, clear the words that the sorts count in, and make the operand
// copies of the weights.  Ahead of sorts in counted tiles also the counts of their first passes, which a launch of its own on the
// other stream had before: that one began 5 us into the step, behind an event of its own, and now the first pass does.
#include "group_device.hpp"

namespace gear {
namespace {

// wc = W as MLP operands [rows x cols], wct = its transpose [cols x rows]; both from the fp32 master, row-major or `packed`.
// One launch serves all layers: a workgroup owns a 32 x 32 tile of one of them; those behind the tiles clear words.
struct BeginArgs {
  int count, cast_blocks, clear_blocks;
  CastJob job[GEAR_MAX_LAYERS];
  int first_block[GEAR_MAX_LAYERS];
  ZeroList zero;
};

__device__ __forceinline__ void clear_words(const ZeroList &zero, int64_t at, int64_t stride) {
  for (int k = 0; k < zero.count; ++k)
    for (int64_t i = at; i < zero.words[k]; i += stride) zero.p[k][i] = 0u;
}

__global__ void __launch_bounds__(256) k_clear(ZeroList zero) {
  clear_words(zero, (int64_t)blockIdx.x * 256 + threadIdx.x, (int64_t)gridDim.x * 256);
}

// Operand order of rows.hip: all rows' 64 bytes of a k-step lie together, sixteen rows at a time, and of those lane by lane:
// the 16 bytes of row r at q * rows + r hold k = 32 s + 8 q .. + 7 (bf16) or 16 s + q, + 4, + 8, + 12 (fp32).  What is left of
// k is a step of fewer q (bf16) or of 8 bytes (fp32).  As many elements as the matrix has.  `row` counts in the operand,
// get(k) is element (row, k) of the 32 x 32 tile whose first column is k0.
template <typename T, typename Get>
__device__ __forceinline__ void put_packed(T *dst, int N, int K, int row, int k0, int piece, Get get) {
  if (row >= N) return;
  const int first = row & ~15, rows = min(16, N - first), r = row & 15;
  if constexpr (sizeof(T) == 2) {   // piece: of four
    const int k = 8 * piece, s = k0 / 32;
    if (k0 + k >= K) return;
    const int pieces = min(4, K / 8 - 4 * s);
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = (uint32_t)from_f32<T>(get(k + 2 * e)) | ((uint32_t)from_f32<T>(get(k + 2 * e + 1)) << 16);
    *reinterpret_cast<uint4 *>(dst + (size_t)32 * s * N + ((size_t)first * pieces + piece * rows + r) * 8) = make_uint4(w[0], w[1], w[2], w[3]);
  } else {                          // piece: of eight
    const int q = piece & 3, k = 16 * (piece >> 2), s = (k0 + k) / 16;
    T *step = dst + (size_t)16 * s * N;
    if (k0 + k + 16 <= K)
      *reinterpret_cast<float4 *>(step + ((size_t)first * 4 + q * rows + r) * 4) = make_float4(get(k + q), get(k + 4 + q), get(k + 8 + q), get(k + 12 + q));
    else if (k0 + k < K)
      *reinterpret_cast<float2 *>(step + ((size_t)first * 4 + q * rows + r) * 2) = make_float2(get(k + q), get(k + 4 + q));
  }
}

// Operand order of the large tiles (gemm.hip): 1 KB for every 32 rows and 16 k, of which lane (g, r) has the 16 bytes of row r, k = 8 g .. + 7.
// `piece`: eight of the 32 k from k0 on.
template <typename Get>
__device__ __forceinline__ void put_tiles(bf16_t *dst, int K, int row0, int r, int k0, int piece, Get get) {
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
    w[e] = (uint32_t)from_f32<bf16_t>(get(8 * piece + 2 * e)) | ((uint32_t)from_f32<bf16_t>(get(8 * piece + 2 * e + 1)) << 16);
  *reinterpret_cast<uint4 *>(dst + (size_t)row0 * K + (k0 / 16 + piece / 2) * 512 + ((piece & 1) * 32 + r) * 8) = make_uint4(w[0], w[1], w[2], w[3]);
}

struct NoCounts {};
template <typename T, bool PACKED, bool COUNT>
__global__ void __launch_bounds__(256) k_begin(BeginArgs args, std::conditional_t<COUNT, FirstCounts, NoCounts> first, int32_t *status,
                                               int32_t *failed, int32_t *n_ready, float *loss) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *status = 0;
    *failed = 0;
    *n_ready = 0;
    *loss = 0.0f;
  }
  int block = blockIdx.x;
  if constexpr (COUNT) {   // ahead of the rest: they are the longest
    extern __shared__ int hist[];
    static_assert(kSortBlock == 256, "one size of workgroup");
    const int counts = first.first_block[kMaxProblems], views = (first.views.B + 255) / 256;
    if (block < counts) {
      int list = 0;
      for (int i = 1; i < kMaxProblems; ++i)
        if (block >= first.first_block[i]) list = i;
      return count_tile(first.gb.p[list], 0, block - first.first_block[list], hist);
    }
    block -= counts;
    if (block < views) {
      // the views of the occurrences; a list that is no list is noted by the next launch, since this one clears the word for it
      const int i = block * 256 + threadIdx.x;
      int32_t lo, hi;
      if (i < first.views.B && view_ok(first.views, i, lo, hi))
        for (int j = lo; j < hi; ++j) first.views.occ_view[j] = i;
      return;
    }
    block -= views;
  }
  if (block >= args.cast_blocks) {
    clear_words(args.zero, (int64_t)(block - args.cast_blocks) * 256 + threadIdx.x, (int64_t)args.clear_blocks * 256);
    return;
  }
  __shared__ float tile[32][33];
  int which = 0;
  for (int i = 1; i < args.count; ++i)
    if (block >= args.first_block[i]) which = i;
  const int rows = args.job[which].rows, cols = args.job[which].cols;
  const float *__restrict__ w = args.job[which].w;
  T *__restrict__ wc = static_cast<T *>(args.job[which].wc);
  T *__restrict__ wct = static_cast<T *>(args.job[which].wct);
  const int local = block - args.first_block[which], col_tiles = (cols + 31) / 32;
  const int c0 = (local % col_tiles) * 32, r0 = (local / col_tiles) * 32;
  const bool tiles = !PACKED && args.job[which].tiles, tiles_t = !PACKED && c0 >= args.job[which].tiles_from;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
#pragma unroll
  for (int rr = ty; rr < 32; rr += 8) {
    const int r = r0 + rr, c = c0 + tx;
    float v = 0.0f;
    if (r < rows && c < cols) {
      v = w[(size_t)r * cols + c];
      if constexpr (!PACKED)
        if (!tiles) wc[(size_t)r * cols + c] = from_f32<T>(v);
    }
    tile[rr][tx] = v;
  }
  __syncthreads();
  if constexpr (PACKED) {
    const int at = threadIdx.x & 31, piece = threadIdx.x >> 5;
    auto of_row = [&](int k) { return tile[at][k]; };
    auto of_col = [&](int k) { return tile[k][at]; };
    if (sizeof(T) == 4 || piece < 4) put_packed(wc, rows, cols, r0 + at, c0, piece, of_row);
    if (sizeof(T) == 4 || piece >= 4) put_packed(wct, cols, rows, c0 + at, r0, sizeof(T) == 4 ? piece : piece - 4, of_col);
    return;
  }
  if constexpr (sizeof(T) == 2) {   // whole 32 x 32 tiles: the host asks for them of such matrices alone
    const int piece = ty & 3;
    if (tiles && ty < 4) put_tiles(wc, cols, r0, tx, c0, piece, [&](int k) { return tile[tx][k]; });
    if (tiles_t && ty >= 4) put_tiles(wct, rows, c0, tx, r0, piece, [&](int k) { return tile[k][tx]; });
  }
  if (tiles_t) return;
#pragma unroll
  for (int cc = ty; cc < 32; cc += 8) {
    const int c = c0 + cc, r = r0 + tx;
    if (r < rows && c < cols) wct[(size_t)c * rows + r] = from_f32<T>(tile[tx][cc]);
  }
}

}  // namespace

static int clear_blocks(const ZeroList &zero) {   // four words a thread, then more
  int64_t words = 0;
  for (int k = 0; k < zero.count; ++k) words += zero.words[k];
  const int64_t blocks = (words + 1023) / 1024;
  return blocks > 256 ? 256 : blocks < 1 ? 1 : (int)blocks;
}

hipError_t launch_clear(const ZeroList &zero, hipStream_t s) {
  hipLaunchKernelGGL(k_clear, dim3(clear_blocks(zero)), dim3(256), 0, s, zero);
  return hipGetLastError();
}

hipError_t launch_begin(int32_t *status, int32_t *failed, int32_t *n_ready, float *loss, const ZeroList &zero, int dtype, const CastJob *jobs,
                        int count, bool packed, const FirstCounts *first, hipStream_t s, hipEvent_t stop) {
  if (count < 0 || count > GEAR_MAX_LAYERS || (first && !packed)) return hipErrorInvalidValue;
  BeginArgs args;
  args.count = count;
  args.zero = zero;
  args.cast_blocks = 0;
  for (int i = 0; i < GEAR_MAX_LAYERS; ++i) {
    args.job[i] = i < count ? jobs[i] : CastJob{nullptr, nullptr, nullptr, 0, 0, false, INT32_MAX};
    if (!packed && i < count && (jobs[i].tiles || jobs[i].tiles_from < jobs[i].cols) &&
        (dtype != GEAR_BF16 || jobs[i].rows % 32 || jobs[i].cols % 32 || (jobs[i].tiles_from < jobs[i].cols && jobs[i].tiles_from % 32)))
      return hipErrorInvalidValue;
    args.first_block[i] = args.cast_blocks;
    if (i < count) args.cast_blocks += ((jobs[i].cols + 31) / 32) * ((jobs[i].rows + 31) / 32);
  }
  args.clear_blocks = clear_blocks(zero);
  int blocks = args.cast_blocks + args.clear_blocks;
  size_t lds = 0;
  if (first) {
    blocks += first->first_block[kMaxProblems] + (first->views.B + 255) / 256;
    for (int i = 0; i < first->gb.count; ++i) lds = max(lds, sizeof(int) << first->gb.p[i].digit_bits);
  }
#define GEAR_BEGIN(T, P, C, FIRST) \
  launch_leaving(stop, k_begin<T, P, C>, dim3((unsigned)blocks), 256, lds, s, args, FIRST, status, failed, n_ready, loss)
  if (dtype == GEAR_BF16) {
    if (first)
      GEAR_BEGIN(bf16_t, true, true, *first);
    else if (packed)
      GEAR_BEGIN(bf16_t, true, false, NoCounts{});
    else
      GEAR_BEGIN(bf16_t, false, false, NoCounts{});
  } else {
    if (first)
      GEAR_BEGIN(float, true, true, *first);
    else if (packed)
      GEAR_BEGIN(float, true, false, NoCounts{});
    else
      GEAR_BEGIN(float, false, false, NoCounts{});
  }
#undef GEAR_BEGIN
  return hipGetLastError();
}

}  // namespace gear
