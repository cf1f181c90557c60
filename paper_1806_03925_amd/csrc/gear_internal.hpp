// Internal declarations shared by the libgear translation units (gfx950 only).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "gear.h"

namespace gear {

// ------------------------------------------------------------------------------------------------
// storage types
// ------------------------------------------------------------------------------------------------
using bf16_t = uint16_t;  // raw bfloat16 bits: sign, 8 exponent bits, 7 fraction bits

__host__ __device__ inline size_t dtype_bytes(int dt) { return dt == GEAR_BF16 ? 2 : 4; }

__device__ __forceinline__ float bf16_to_f32(bf16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// round to nearest, ties to even
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40u);  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

// two floats -> two bf16 in one word (round to nearest even, one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// How a gradient changes a parameter (Section 3, step 4 applies the Sparse Part's gradients every
// step; Section 4.1 trains with Adam).  SGD: w -= lr g.  Adam (Kingma & Ba, Algorithm 1):
// m = b1 m + (1 - b1) g, v = b2 v + (1 - b2) g^2, w -= lr / (1 - b1^t) * m / (sqrt(v) / sqrt(1 - b2^t) + eps);
// the two factors that depend on t are computed by the host.
struct Optim {
  float lr;        // SGD: the rate.  Adam: lr / (1 - beta1^t)
  float beta1, beta2, eps;
  float inv_bc2;   // Adam: 1 / sqrt(1 - beta2^t)
  int32_t adam;    // 0 = SGD
};
struct Moments {   // first and second moment arrays of the same shape as the parameters; null for SGD
  float *m, *v;
};
__host__ __device__ __forceinline__ Moments moments_at(const Moments &base, ptrdiff_t offset) {
  Moments r = {base.m ? base.m + offset : nullptr, base.v ? base.v + offset : nullptr};
  return r;
}
__device__ __forceinline__ float optim_apply(const Optim &o, float w, float g, float *m, float *v) {
  if (!o.adam) return w - o.lr * g;
  const float mn = o.beta1 * *m + (1.0f - o.beta1) * g;
  const float vn = o.beta2 * *v + (1.0f - o.beta2) * g * g;
  *m = mn;
  *v = vn;
  return w - o.lr * mn / (sqrtf(vn) * o.inv_bc2 + o.eps);
}

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t v) { return bf16_to_f32(v); }

template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return f32_to_bf16(v); }

// 16-byte vector of T
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int N = 4;
  float4 v;
  __device__ __forceinline__ float get(int i) const { return (&v.x)[i]; }
  __device__ __forceinline__ void set(int i, float f) { (&v.x)[i] = f; }
};
template <> struct Vec16<bf16_t> {
  static constexpr int N = 8;
  uint4 v;
  __device__ __forceinline__ float get(int i) const {
    uint32_t w = (&v.x)[i >> 1];
    return __uint_as_float((i & 1) ? (w & 0xffff0000u) : (w << 16));
  }
  __device__ __forceinline__ void set(int i, float f) {
    uint32_t b = f32_to_bf16(f);
    uint32_t &w = (&v.x)[i >> 1];
    w = (i & 1) ? ((w & 0x0000ffffu) | (b << 16)) : ((w & 0xffff0000u) | b);
  }
};

constexpr int kWave = 64;

// first index of the ascending keys[lo .. hi) whose key is >= key (> key with `after`), hi if there is none;
// by one wavefront, 64 probes at a time
__device__ __forceinline__ int wave_search(const int32_t *__restrict__ keys, int lo, int hi, int key, bool after, int lane) {
  while (lo < hi) {
    const int step = (hi - lo - 1) / kWave + 1;
    const int64_t at = (int64_t)lo + (int64_t)lane * step;
    const int probe = at < hi ? keys[at] : 0;
    const unsigned long long m = __ballot(at >= hi || (after ? probe > key : probe >= key));
    const int first = m ? __builtin_ctzll(m) : kWave;
    const int64_t up = (int64_t)lo + (int64_t)first * step;
    if (first < kWave && up < hi) hi = (int)up;
    if (first > 0) lo = (int)min((int64_t)hi, (int64_t)lo + (int64_t)(first - 1) * step + 1);
  }
  return lo;
}

// ------------------------------------------------------------------------------------------------
// grouping (sort by key + segments) problem descriptors
// ------------------------------------------------------------------------------------------------
constexpr int kSortBlock = 256;                       // threads
constexpr int kSortItems = 8;                         // keys per thread
constexpr int kSortTile = kSortBlock * kSortItems;    // keys per workgroup
constexpr int kMaxProblems = 3;
constexpr int kMaxPasses = 4;
constexpr int kMaxRides = 3;                          // passes that other launches are asked to carry, if it is up to us
constexpr int kMaxDigitBits = 12;
constexpr int kSideDigitBits = 11;                    // of passes that other launches carry
constexpr int kBesideDigitBits = 9;                   // of passes that look back beside workgroups that fill their CU
constexpr int kCountedDigitBits = 10;                 // of passes whose tiles are counted ahead of them
// ids from which a workgroup of the check takes several tiles and the segments take few registers
constexpr int kLongList = 65536;
// Counts a tile publishes over all passes, at most.  A pass costs a launch and two memory latencies whatever its
// radix, so a list takes as few passes as its keys allow within this (one up to 12 bits, two up to 22, then three);
// it is what the regions that hold the counts have room for (24 KB per tile of 2048 keys).
constexpr int kStateWords = 6144;
constexpr int kTickets = kMaxProblems * kMaxPasses + 1;   // one per list and pass, the last one for the segments

struct GroupProblem {
  const int32_t *keys_in;  // [n] original keys (read by the first pass)
  int64_t range;           // keys have to be below this; 0: not checked
  int32_t n;
  int32_t passes;          // radix passes
  int32_t digit_bits;      // bits per pass
  int32_t *keys[2];        // ping-pong key buffers [n]
  int32_t *vals[2];        // ping-pong position buffers [n]
  int32_t *totals;         // [passes][radix] keys of a digit in the whole list
  uint32_t *state;         // [passes][tiles - 1][radix] what tiles publish for those after them; counted: [passes][tiles][radix]
  int32_t *sorted_keys;    // = keys[passes & 1]
  int32_t *perm;           // = vals[passes & 1]
  int32_t *unique;         // [n]   distinct keys ascending (NULL: not wanted)
  int32_t *segoff;         // [n+1] segment offsets (with `unique`)
  int32_t *n_unique;       // [1]
};

struct GroupBatch {
  GroupProblem p[kMaxProblems];   // segments are made of the last one
  int32_t count;
  int32_t *tickets;               // [kTickets]
  uint32_t *seg_state;            // [tiles - 1][3] heads, units and emissions, published like `state`
};

// The widest digits a list of n ids is sorted by in launches of their own: a wide digit saves a pass of a short list, but a
// tile looks back at up to all before it for every digit (139 000 ids, 22 bits: two passes of eleven bits 39 and 43 us
// beside a product, three of eight bits 12 us each; 600 000 ids of 31 bits alone, three of eleven 289 us in all, four of
// eight 139).
inline int widest_digit(int n) { return n > 16 * kSortTile ? 9 : kMaxDigitBits; }

inline int bits_for(int64_t range) {
  int b = 1;
  while (b < 31 && ((int64_t)1 << b) < range) ++b;
  return b;
}

// fewest passes over keys of `bits` bits in digits of up to `widest` bits
inline int radix_passes(int bits, int most_words, int widest) {
  int passes = 1;
  for (; passes < kMaxPasses; ++passes) {
    const int digit_bits = (bits + passes - 1) / passes;
    if (digit_bits <= widest && (passes << digit_bits) <= most_words) break;
  }
  return passes;
}

// plan of the windowed accumulation over the sorted image occurrences
struct UnitDesc {         // one workgroup's share of the accumulation (32 bytes)
  int32_t q0;             // first sorted position of the unit
  int32_t image;          // image id
  int32_t slot;           // ready-list slot of the unit's (first) emission
  int32_t s0, s1;         // the image's range of sorted positions
  int32_t phase;          // gradients already collected for the image before this step, modulo M
  int32_t collected;      // gradients collected for the image after this step
  int32_t pad;
};

// What the workgroups that sort short lists in LDS (local_group.hpp) leave where a step has no prologue: none of them looks at what another
// one does, so that nothing has to be cleared ahead of their launch.  Who reads their plan adds up what the parts of the images count
// (local_parts.hpp).
struct PartCounts {
  int32_t below;          // ids of the list in lower parts: the part's units begin at that place
  int32_t heads, units, emits;
};
constexpr int kMaxParts = 32;
constexpr int kCodeGroup = 64;
struct LocalResult {
  PartCounts *parts;      // [n_parts], 16-byte aligned; NULL: not so
  uint8_t *codes;         // [n_codes up to a whole group, 64-byte aligned] whether a workgroup has found ids or offsets that are wrong
  int n_parts, n_codes;
  int ready_cap;          // -1: more emissions than there is room for cannot be
};

struct AccumPlan {
  UnitDesc *units;       // [nnz]
  int32_t *row_view;     // [nnz] view that owns the occurrence at each sorted position
  float *row_scale;      // [nnz] 1 / (images of that view): backward of the mean
  const int32_t *row_at; // [nnz] where the two are by position in the batch: that of each sorted one (else NULL)
  int32_t *n_units;      // [1]
  LocalResult local;     // with it units lie part by part, their slots count from the part's first emission, and n_units is not there
};

// ---- tasks of the grouping (group.hip) ----
// What goes wrong in a step is noted twice: in the caller's status word, and in a word of the step's own workspace
// (`failed`), which is the one that later kernels look at before they do anything.  The caller's may be written by other
// calls while a step runs (a refresh on another stream reports its ids there), and workgroups of one launch that read it at
// different times would not agree on whether to work: those that do wait for what the others publish (group_device.hpp).
// Only launches of the step write `failed`, and a launch that reads it begins after the last one that may set it, but for
// the tile that finds the ready list too long when all others have read it.
struct ViewCheck {
  const int32_t *img_off;
  int32_t *occ_view;
  int32_t B, nnz;   // B = 0: no views to check
};
struct CheckTask {
  GroupBatch gb;
  ViewCheck views;
  int blocks, tiles_per_block;
  int32_t *failed, *status;
};
struct PlanArgs {
  AccumPlan plan;
  const int32_t *occ_view, *img_off, *counts;
  int32_t M, ready_cap;
  int32_t *n_ready, *status;
};
// one link of the grouping that a launch of the forward pass carries (group_device.hpp)
struct SideTask {
  enum Kind { kPass, kSegments };
  int kind, pass;
  int blocks;       // workgroups, a multiple of the XCDs' number so that the products' stay on the XCDs they share operands on
  GroupBatch gb;
  PlanArgs plan;
  int32_t *failed;
};
struct NoTask {};
// the grouping of short lists in LDS (local_group.hpp)
constexpr int kLocalMost = 19200;                    // ids of a list: a part, which may be all of it, fits in half a CU's LDS (rows.hip)
struct LocalList {
  const int32_t *keys_in;
  int64_t range;
  int n, bits, parts_log2, value_bits;   // of an id, of the number of parts, of a position
  int32_t *sorted_keys, *perm;
  uint32_t *spare;                       // [n]
};
struct LocalTask {
  LocalList list[kMaxProblems];          // segments are made of the last one
  PlanArgs plan;
  ViewCheck views;
  int32_t *unique, *segoff, *n_unique;   // of the last list; the first two may be NULL
  // where the step has a prologue, which clears them: what the parts of the last list publish ([parts][3]), and their ticket
  uint32_t *state;
  int32_t *ticket, *failed;
  float *loss;                           // where it has none the first workgroup clears the step's outputs: this, and the plan's
  int blocks, room;                      // workgroups; items that LDS has room for
};
// the distinct ids and their segments from where the parts have left them to where one after the other belongs (each may be NULL)
hipError_t launch_unique(const LocalResult &local, const int32_t *unique, const int32_t *segoff, int n, int32_t *out_unique, int32_t *out_segoff,
                         int32_t *out_n, hipStream_t s);

// ------------------------------------------------------------------------------------------------
// workspace layout (byte offsets from a 256-byte aligned base)
// ------------------------------------------------------------------------------------------------
struct Layout {
  int32_t F;                         // MLP input width
  int32_t L;                         // layers
  int32_t in_dim[GEAR_MAX_LAYERS];   // input width of each layer
  int32_t out_dim[GEAR_MAX_LAYERS];
  int64_t w_off[GEAR_MAX_LAYERS];    // float offsets into mlp_params
  int64_t b_off[GEAR_MAX_LAYERS];
  int64_t n_params;
  bool colsum_coarse;                // the partials only fit with at least kColsumRows rows each
  size_t act_bytes;                  // sizeof(mlp_dtype)

  size_t x, h[GEAR_MAX_LAYERS], delta[GEAR_MAX_LAYERS], logits, dz, loss_partial, dx_emb, dx_dfv;
  size_t relu_bits[GEAR_MAX_LAYERS];  // [B x out/8] sign bitmaps of the hidden activations
  size_t wc[GEAR_MAX_LAYERS], wct[GEAR_MAX_LAYERS], wgrad_partial, colsum_partial, emb_partial;
  size_t colsum_at[GEAR_MAX_LAYERS]; // floats before the column-sum partials that layer l's masked product leaves
  size_t wgrad_partial_bytes;        // size of the split-K partial region
  size_t occ_view, failed;
  struct G {
    size_t keys[2], vals[2], totals, state, unique, segoff, n_unique;
    int32_t total_words;             // room for `totals`
  } g[kMaxProblems];
  size_t pool_bytes, pool_rest;       // the region of sums that begins at loss_partial; what follows its digit totals
  size_t tickets, seg_state, units, row_view, row_scale, n_units;
  size_t expiry_marks, expiry_tiles;  // gear_expired_ids: byte map over the images, marked bytes per tile
  size_t total;
};

bool make_layout(const gear_config &cfg, Layout *lay);
bool config_ok(const gear_config &cfg);

constexpr int kColsumRows = 128;     // rows per partial of a column sum that the region of partials is sized for
constexpr int kLossBlocks = 2048;    // most workgroups (and partial sums) of the logit/loss kernel

// ------------------------------------------------------------------------------------------------
// kernel launchers (each defined next to its kernel)
// ------------------------------------------------------------------------------------------------
// `stop` (may be NULL) is an event that the launch itself leaves when it ends.  Recorded behind the launch, an event is a packet
// of its own, which what follows on the stream waits for.
inline hipError_t leave(hipEvent_t stop, hipStream_t s) { return stop ? hipEventRecord(stop, s) : hipSuccess; }   // no launch to leave it
template <typename Kernel, typename... Args>
inline void launch_leaving(hipEvent_t stop, Kernel kernel, dim3 grid, int threads, size_t lds, hipStream_t s, const Args &...args) {
  if (stop)
    hipExtLaunchKernelGGL(kernel, grid, dim3((unsigned)threads), (uint32_t)lds, s, nullptr, stop, 0, args...);
  else
    hipLaunchKernelGGL(kernel, grid, dim3((unsigned)threads), (uint32_t)lds, s, args...);
}
hipError_t launch_fill_normal(void *dst, int dtype, int64_t n_elems, uint64_t seed, uint32_t stream_id,
                              float std, hipStream_t s);
hipError_t launch_fill_zero(void *dst, size_t bytes, hipStream_t s);

// words that a launch clears on the way
struct ZeroList {
  static constexpr int kMax = 2 * kMaxProblems + 3;
  int count;
  uint32_t *p[kMax];
  int64_t words[kMax];
};
// launch_begin clears the step's outputs and `zero`, and makes the operand copies of `count` layers' weights
struct CastJob {
  const float *w;
  void *wc, *wct;
  int rows, cols;
  // bf16, not `packed`: W in the operand order of the large tiles (gemm.hip), and so its transpose from that row on (a multiple of
  // 32; INT32_MAX: row-major)
  bool tiles;
  int tiles_from;
};
hipError_t launch_clear(const ZeroList &zero, hipStream_t s);
struct FirstCounts {
  GroupBatch gb;
  ViewCheck views;
  int first_block[kMaxProblems + 1];   // of each list, then of the views
};
FirstCounts first_counts(const GroupBatch &gb, const ViewCheck &views);
void counted_zero_list(const GroupBatch &gb, ZeroList *z);
// `first` (may be NULL; packed weights only): and what the first passes over lists in counted tiles need, the counts and the views
hipError_t launch_begin(int32_t *status, int32_t *failed, int32_t *n_ready, float *loss, const ZeroList &zero, int dtype, const CastJob *jobs,
                        int count, bool packed, const FirstCounts *first, hipStream_t s, hipEvent_t stop);
void group_zero_list(const GroupBatch &gb, ZeroList *z);
CheckTask check_task(const GroupBatch &gb, const int32_t *img_off, int32_t *occ_view, int B, int nnz, int32_t *failed,
                     int32_t *status);
int check_lds_bytes(const GroupBatch &gb);
int group_passes(const GroupBatch &gb);
SideTask side_task(const GroupBatch &gb, const PlanArgs &plan, int step, int32_t *failed);   // step: a pass, or the segments behind them
int radix_lds_bytes(const GroupBatch &gb);
hipError_t launch_check(const GroupBatch &gb, const int32_t *img_off, int32_t *occ_view, int B, int nnz, int32_t *failed,
                        int32_t *status, hipStream_t s);
hipError_t launch_radix_pass(const GroupBatch &gb, int pass, const int32_t *failed, hipStream_t s);
// passes of a list whose tiles are counted, in digits of up to `widest` bits: the fewest whose counts fit where the list's
// unique ids and their offsets go (of `cap` ids at most); 0: they do not
int counted_passes(int bits, int n, int cap, int widest);
int counted_lds_bytes(int digit_bits);
hipError_t launch_count(const GroupBatch &gb, int pass, hipStream_t s);   // the first passes' counts are the prologue's
hipError_t launch_counted_pass(const GroupBatch &gb, int pass, const ViewCheck &views, const PlanArgs &args, int32_t *failed, hipStream_t s,
                               hipEvent_t stop);
hipError_t launch_segments_count(const GroupBatch &gb, const PlanArgs &args, int next, int32_t *failed, hipStream_t s, hipEvent_t stop);
hipError_t launch_segments(const GroupBatch &gb, const PlanArgs *args, int32_t *failed, hipStream_t s, hipEvent_t stop = nullptr);
// distinct ids of a grouped list whose cache entry is older than `expiry`, ascending
// words (four images each) of the byte map over all images that the expiry filter marks, and tiles
// of kSortTile words
inline int64_t expiry_words(int64_t n_images) { return (n_images + 3) / 4; }
inline int64_t expiry_tiles(int64_t n_images) { return (expiry_words(n_images) + kSortTile - 1) / kSortTile; }
hipError_t launch_expired(const int32_t *image_ids, int n, const int32_t *stamp, int64_t n_images, int32_t now,
                          int32_t expiry, uint8_t *marks, int32_t *tile_counts, int32_t *out_ids, int32_t *n_out,
                          int32_t *status, hipStream_t s);
hipError_t launch_stamp(int32_t *stamp, int64_t n_images, const int32_t *ids, int64_t n, int32_t now, int32_t *status,
                        hipStream_t s, const int32_t *n_dev = nullptr);
hipError_t launch_gather_pool(const gear_config &cfg, const gear_batch &b, const gear_tables &t,
                              const void *dfv_cache, void *x, hipStream_t s, const CheckTask *check = nullptr);

enum GemmEpilogue {
  EPI_BIAS_RELU = 0,  // out(T)   = max(acc + bias[n], 0)
  EPI_MASK = 1,       // out(T)   = aux[m,n] > 0 ? acc : 0
  EPI_F32 = 2,        // out(f32) = acc
  EPI_DX = 3,         // columns < split: out(f32)[M x split] = acc; others: aux(T)[M x (N - split)] = acc
  EPI_MASK_BITS = 4,  // EPI_MASK with aux = the bitmap [M x N/8] an EPI_BIAS_RELU product left in `relu_bits`
};
// C[M x N] = A[M x K] * B[N x K]^T, both operands K-contiguous, type `dtype`.
// relu_bits (bf16 and EPI_BIAS_RELU only, may be NULL): bit (n % 8) of byte [m][n / 8] = (out[m][n] > 0), which is
// what EPI_MASK_BITS (bf16 only) masks with.  colpart (masked products, may be NULL): [parts x N] column sums of
// what is stored, per row tile; `coarse` keeps row tiles at kColsumRows rows or more.  status may be NULL (the product
// then always runs).
hipError_t launch_gemm_nt(int dtype, const void *A, const void *B, int M, int N, int K, int epilogue,
                          const float *bias, const void *aux, void *out, int split, float *colpart,
                          uint8_t *relu_bits, const int32_t *status, hipStream_t s, bool coarse = false,
                          const SideTask *side = nullptr, bool tiles = false, hipEvent_t stop = nullptr);
// whether such a product without a SideTask takes B in the operand order of the large tiles (`tiles`)
bool gemm_nt_takes_tiles(int dtype, int M, int N, int K, int epilogue);
bool gemm_nt_carries(int dtype, int M, int N, int K);   // whether a bias + ReLU or dLoss/dx product of this shape takes a SideTask
int gemm_nt_colsum_parts(int dtype, int M, int N, int K, bool coarse);
// partial_i[z][M_i x N_i] = sum over the z-th of `splits` ranges of the K rows of A_i[K x M_i]^T * B_i[K x N_i], for
// all problems in one launch (operands M-/N-contiguous).  k_dev (may be NULL): device word holding the real
// contraction length, at most K; it is then split into ranges on the device.
struct TnProblem {
  const void *A, *B;
  float *partial;
  int M, N;
};
// `large`: on 256 x 256 tiles (bf16, K a multiple of 32 and no k_dev), as gemm_tn_choice says.
hipError_t launch_gemm_tn(int dtype, const TnProblem *p, int count, int K, int splits, bool large, bool pairs, const int32_t *status,
                          hipStream_t s, const int32_t *k_dev = nullptr);
// how to go about several of them (looks at M and N only): the first `layers` in one launch, on which tiles, in how many ranges
struct TnChoice {
  int layers;
  bool large;
};
TnChoice gemm_tn_choice(int dtype, const TnProblem *p, int count, int K);
// *pairs: whether it may be of workgroups that walk two halves of a range (in a launch of their own and of known length, gemm_tile.hip);
// then whether it is
int gemm_tn_splits(int dtype, const TnProblem *p, int count, int K, bool large, bool *pairs);
// w_i <- update(w_i, sum_z partial_i[z]) for the results of such a launch
struct SplitkProblem {
  const float *partial;
  float *w;
  Moments mom;
  int64_t count;
};
// dst[j] <- update(dst[j], sum_p partial[p][j]), p < parts and j < width, in a fixed two-level shape
struct ColumnSum {
  const float *partial;
  float *dst;
  Moments mom;
  int parts, width;
};
struct LossSum {   // *loss = (sum of the partial sums) / B; parts = 0: not wanted
  const float *partial;
  float *loss;
  int parts, B;
};
constexpr int kMaxColumnSums = GEAR_MAX_LAYERS + 2;
// n_ready (may be NULL) is cleared if the step has failed; with local.parts, it and what has gone wrong are written here, and the status
// word is left alone otherwise: what another call has reported there meanwhile stays.
struct LocalOutputs {
  LocalResult local;
  int32_t *status, *n_ready;
};
// all of that in one launch, and level 2 of an embedding update (may be NULL)
struct EmbeddingWork;
hipError_t launch_param_update(const SplitkProblem *p, int count, int splits, const ColumnSum *c, int n_columns,
                               const LossSum &loss, const EmbeddingWork *emb, const LocalOutputs &local, const Optim &opt,
                               const int32_t *status, hipStream_t s, hipEvent_t stop = nullptr);
// the same products on tiles of moderate size (gemm_tile.hip)
hipError_t launch_gemm_nt_tile(int dtype, const void *A, const void *B, int M, int N, int K, int epilogue,
                               const float *bias, const void *aux, void *out, int split, float *colpart,
                               uint8_t *relu_bits, const int32_t *status, hipStream_t s, bool coarse, const SideTask *side, hipEvent_t stop);
int nt_tile_colsum_parts(int dtype, int M, int N, bool coarse);
hipError_t launch_gemm_tn_tile(int dtype, const TnProblem *p, int count, int K, int splits, bool pairs, const int32_t *status,
                               hipStream_t s, const int32_t *k_dev);
int tn_tile_splits(int dtype, const TnProblem *p, int count, int K, bool *pairs);
long long tn_tile_rows(int dtype, const TnProblem *p, int count, int K);   // that a CU walks, two ranges at a time

hipError_t launch_logit_loss(int dtype, const void *h, const void *wc_last, const float *bias_last, const float *label,
                             int B, int H, float *logits, float *dz, void *delta, float *partials,
                             const int32_t *status, hipStream_t s, const SideTask *side = nullptr);
// where launch_logit_loss leaves its sums, one row per workgroup
struct LogitSums {
  const float *w, *delta, *bias, *loss;   // [parts x H], [parts x H], [parts], [parts]
  int parts;
};
LogitSums logit_sums(const float *partials, int B, int H);
size_t logit_partial_floats(int H, int B);

constexpr int kChunk = 16;

struct EmbeddingTable {
  const int32_t *keys;   // sorted ids
  const int32_t *perm;   // batch position of each sorted position
  int n;
  void *rows;            // embedding table
  int col0;              // first column of this table's slice inside a dx row
  float *part_first;     // [chunks x d] partial of a run that began in an earlier chunk
  float *part_last;      // [chunks x d] partial of a run that begins here and goes on
  Moments mom;           // Adam: fp32 moment tables of the same shape as `rows` (only touched rows move)
};
struct EmbeddingWork {
  EmbeddingTable table[2];   // users, URLs
  const float *dx;           // the embedding slots of dLoss/dx, [B x 2 d]
  int32_t d, bf16;           // width and type of a row
  Optim opt;
  AccumPlan plan;            // of the images, for
  int32_t *counts;           // their counters
};
EmbeddingWork embedding_work(const gear_config &cfg, const GroupProblem &users, const GroupProblem &urls, const float *dx,
                             void *user_emb, void *url_emb, float *partials, const Optim &opt, const Moments &mom_user,
                             const Moments &mom_url, const AccumPlan &plan, int32_t *counts);
hipError_t launch_embedding_update(const EmbeddingWork &w, bool both_levels, const int32_t *status, hipStream_t s);
size_t embedding_partial_floats(const gear_config &cfg);

// batch sums of a step layer by layer, in the shape in which blocks of views leave them (block_sums.hpp)
struct BlockSums {
  struct Columns {
    const void *delta;   // [B x width]
    float *part;         // [blocks x width]
    int width;
  };
  int B, rows, blocks, layers;             // rows of a block
  const float *dz, *logits, *label;
  const void *h;                           // activations of the last hidden layer, whose delta is layer[0]'s
  float *part_w, *part_b, *part_loss;
  Columns layer[GEAR_MAX_LAYERS - 1];
};
// `sums` (may be NULL; one stream only) ride along
hipError_t launch_accumulate(const gear_config &cfg, const GroupProblem &img, const AccumPlan &plan,
                             const void *dx_dfv, float *grad_accum, int32_t M, int32_t *ready_ids,
                             float *ready_grads, const EmbeddingWork *emb, bool level2, const BlockSums *sums, const int32_t *status,
                             hipStream_t s, hipEvent_t stop);

// with level 1 and the counters, beside `count` weight-gradient products on tiles of moderate size
hipError_t launch_accumulate_wgrad(const gear_config &cfg, const GroupProblem &img, const AccumPlan &plan, const void *dx_dfv,
                                   float *grad_accum, int32_t M, int32_t *ready_ids, float *ready_grads, const EmbeddingWork &emb,
                                   const TnProblem *p, int count, int K, int splits, const int32_t *status, hipStream_t s);

// n_dev (may be NULL): device word holding the real row count, at most n
hipError_t launch_refresh(int dtype, void *dfv_cache, int64_t n_images, int dim, const int32_t *ids,
                          const void *rows, int64_t n, int32_t *status, hipStream_t s, const int32_t *n_dev = nullptr);

}  // namespace gear
