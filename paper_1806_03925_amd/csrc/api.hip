// C ABI of libgear: argument checks, workspace layout and the launch sequence of one step.
#include "gear_internal.hpp"
#include "rows.hpp"

#include <math.h>
#include <string.h>

#include <mutex>
#include <new>

namespace gear {

namespace {

constexpr size_t kAlign = 256;

size_t take(size_t *cursor, size_t bytes) {
  const size_t at = *cursor;
  *cursor = (at + bytes + kAlign - 1) / kAlign * kAlign;
  return at;
}

// `bits`: what the keys have at most
GroupProblem make_problem(const Layout &lay, char *ws, int slot, const int32_t *keys, int n, int64_t range, int passes, int bits) {
  GroupProblem p;
  memset(&p, 0, sizeof(p));
  p.keys_in = keys;
  p.n = n;
  p.range = range;
  p.passes = passes;
  p.digit_bits = (bits + passes - 1) / passes;
  const Layout::G &g = lay.g[slot];
  for (int i = 0; i < 2; ++i) {
    p.keys[i] = (int32_t *)(ws + g.keys[i]);
    p.vals[i] = (int32_t *)(ws + g.vals[i]);
  }
  p.totals = (int32_t *)(ws + g.totals);
  p.state = (uint32_t *)(ws + g.state);
  p.sorted_keys = p.keys[p.passes & 1];
  p.perm = p.vals[p.passes & 1];
  p.unique = (int32_t *)(ws + g.unique);
  p.segoff = (int32_t *)(ws + g.segoff);
  p.n_unique = (int32_t *)(ws + g.n_unique);
  return p;
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace

}  // namespace gear

// HIP-event pool for per-launch timing of a step
struct gear_profile {
  static constexpr int kMaxSpans = 96;
  hipEvent_t start[kMaxSpans], stop[kMaxSpans];
  const char *name[kMaxSpans];
  int used;
};

namespace gear {
namespace {

struct Span {
  gear_profile *p;
  hipStream_t s;
  int slot;
  Span(gear_profile *prof, const char *name, hipStream_t stream) : p(prof), s(stream), slot(-1) {
    if (p && p->used < gear_profile::kMaxSpans) {
      slot = p->used++;
      p->name[slot] = name;
      (void)hipEventRecord(p->start[slot], s);
    }
  }
  ~Span() {
    if (slot >= 0) (void)hipEventRecord(p->stop[slot], s);
  }
};

}  // namespace

bool config_ok(const gear_config &c) {
  if (c.n_users < 1 || c.n_urls < 1 || c.n_images < 1) return false;
  if (c.n_users > INT32_MAX || c.n_urls > INT32_MAX || c.n_images > INT32_MAX) return false;
  if (c.emb_dim < 8 || c.emb_dim % 8 || c.dfv_dim < 8 || c.dfv_dim % 8) return false;
  if (c.n_layers < 2 || c.n_layers > GEAR_MAX_LAYERS) return false;
  for (int l = 0; l < c.n_layers - 1; ++l)
    if (c.layer_out[l] < 8 || c.layer_out[l] % 8) return false;
  if (c.layer_out[c.n_layers - 1] != 1) return false;
  if (c.layer_out[c.n_layers - 2] > 1024) return false;  // the logit kernel keeps a hidden row in one wavefront
  for (int dt : {c.emb_dtype, c.dfv_dtype, c.mlp_dtype})
    if (dt != GEAR_F32 && dt != GEAR_BF16) return false;
  if (c.max_batch < 1 || c.max_nnz < 1) return false;
  if (!(c.emb_init_std >= 0.0f) || !isfinite(c.emb_init_std)) return false;
  return true;
}

// Bytes of the region that holds the weight gradients' partial results.  Callers allocate a workspace once and keep it,
// and which configurations the static scratch array takes depends on its size, so this is a fixed rule of the
// configuration; how many ranges a step cuts its batch into follows from it and not the other way round.
static size_t wgrad_region_bytes(int dtype, const int32_t *rows, const int32_t *cols, int layers, int K) {
  auto ranges = [](int tiles, int cap) {
    int s = 256 / tiles;
    if (cap < 1) cap = 1;
    if (s > cap) s = cap;
    return s < 1 ? 1 : (s > 64 ? 64 : s);
  };
  auto tiles_of = [](int m, int n, int bn) { return ((m + 255) / 256) * ((n + bn - 1) / bn); };
  size_t most = 0, all = 0;
  int tiles = 0;
  for (int l = 0; l < layers; ++l) {
    int s = ranges(tiles_of(rows[l], cols[l], 128), K / 128);
    if (dtype == GEAR_BF16) {
      const int t = ranges(tiles_of(rows[l], cols[l], 256), K / 512);
      if (t > s) s = t;
    }
    const size_t n = (size_t)rows[l] * cols[l];
    if (s * n > most) most = s * n;
    all += n;
    tiles += tiles_of(rows[l], cols[l], 256);
  }
  // the layers of a bf16 model together, for batches of whole 32-row tiles
  if (dtype == GEAR_BF16 && layers >= 2 && K >= 32 && tiles <= 128) {
    const size_t together = ranges(tiles, K / 32 * 32 / 512) * all;
    if (together > most) most = together;
  }
  return most * sizeof(float);
}

bool make_layout(const gear_config &c, Layout *lay) {
  if (!config_ok(c)) return false;
  memset(lay, 0, sizeof(*lay));
  const int L = c.n_layers, F = 2 * c.emb_dim + c.dfv_dim;
  const size_t B = (size_t)c.max_batch, NNZ = (size_t)c.max_nnz;
  lay->F = F;
  lay->L = L;
  lay->act_bytes = dtype_bytes(c.mlp_dtype);
  int64_t off = 0;
  for (int l = 0; l < L; ++l) {
    lay->in_dim[l] = l == 0 ? F : c.layer_out[l - 1];
    lay->out_dim[l] = c.layer_out[l];
    lay->w_off[l] = off;
    off += (int64_t)lay->in_dim[l] * lay->out_dim[l];
    lay->b_off[l] = off;
    off += lay->out_dim[l];
  }
  lay->n_params = off;

  size_t cur = 0;
  const size_t ab = lay->act_bytes;
  lay->x = take(&cur, B * F * ab);
  size_t max_partial = 0, max_h = 1;
  for (int l = 0; l < L; ++l) {
    const size_t wn = (size_t)lay->in_dim[l] * lay->out_dim[l];
    lay->wc[l] = take(&cur, wn * ab);
    lay->wct[l] = take(&cur, wn * ab);
    if (l < L - 1) {
      lay->h[l] = take(&cur, B * lay->out_dim[l] * ab);
      lay->relu_bits[l] = take(&cur, B * lay->out_dim[l] / 8);
      lay->delta[l] = take(&cur, B * lay->out_dim[l] * ab);
    }
    if ((size_t)lay->out_dim[l] > max_h) max_h = lay->out_dim[l];
    if ((size_t)lay->in_dim[l] > max_h) max_h = lay->in_dim[l];
  }
  lay->logits = take(&cur, B * sizeof(float));
  lay->dz = take(&cur, B * sizeof(float));
  // The sums of the logit kernel and the digit totals of the sorts share a region: a batch of B views has one row of
  // sums per 32 views, which leaves most of a region of kLossBlocks rows to the totals of a short batch; a long one has
  // more tiles, whose share (one row of 512 per tile and list) is enough.
  const size_t sums = logit_partial_floats(lay->in_dim[L - 1], c.max_batch);
  size_t pool = logit_partial_floats(lay->in_dim[L - 1], 32 * kLossBlocks);
  for (int s = 0; s < kMaxProblems; ++s) pool += ((s == 2 ? NNZ : B) + kSortTile - 1) / kSortTile * 512 + 512;
  lay->loss_partial = take(&cur, pool * sizeof(float));
  lay->tickets = lay->loss_partial + sums * sizeof(float);
  size_t room = (pool - sums - kTickets) / kMaxProblems;
  if (room > (size_t)kStateWords) room = kStateWords;
  for (int s = 0; s < kMaxProblems; ++s) {
    lay->g[s].totals = lay->tickets + (kTickets + s * room) * sizeof(float);
    lay->g[s].total_words = (int32_t)room;
  }
  lay->pool_bytes = pool * sizeof(float);
  lay->pool_rest = lay->tickets + (kTickets + kMaxProblems * room) * sizeof(float);
  lay->dx_emb = take(&cur, B * 2 * c.emb_dim * sizeof(float));
  lay->dx_dfv = take(&cur, B * c.dfv_dim * ab);
  max_partial = wgrad_region_bytes(c.mlp_dtype, lay->out_dim, lay->in_dim, L - 1, c.max_batch);
  lay->wgrad_partial = take(&cur, max_partial);
  lay->wgrad_partial_bytes = max_partial;
  // column-sum partials of all masked products (they are reduced at the end of a step): one block of rows per
  // kColsumRows rows and layer is what the region holds; products of 64-row tiles leave up to twice as many
  const size_t blocks = (B + kColsumRows - 1) / kColsumRows;
  size_t fine = 0;
  for (int l = 1; l < L - 1; ++l) fine += 2 * blocks * lay->in_dim[l];
  lay->colsum_coarse = fine > blocks * max_h * (size_t)(L - 1);
  size_t at = 0;
  for (int l = 1; l < L - 1; ++l) {
    lay->colsum_at[l] = at;
    at += (lay->colsum_coarse ? 1 : 2) * blocks * lay->in_dim[l];
  }
  lay->colsum_partial = take(&cur, blocks * max_h * (size_t)(L - 1) * sizeof(float));
  lay->emb_partial = take(&cur, embedding_partial_floats(c) * sizeof(float));
  lay->occ_view = take(&cur, NNZ * sizeof(int32_t));
  for (int s = 0; s < kMaxProblems; ++s) {
    const size_t n = s == 2 ? NNZ : B;
    const size_t tiles = (n + kSortTile - 1) / kSortTile;
    Layout::G &g = lay->g[s];
    for (int i = 0; i < 2; ++i) {
      g.keys[i] = take(&cur, n * sizeof(int32_t));
      g.vals[i] = take(&cur, n * sizeof(int32_t));
    }
    // what the tiles of a pass publish (at most 24 KB for each tile but the last) lies where nothing is kept until
    // the sorts are done
    if (s < 2) take(&cur, tiles * sizeof(int32_t));
    g.unique = take(&cur, n * sizeof(int32_t));
    g.segoff = take(&cur, (n + 1) * sizeof(int32_t));
    take(&cur, n * sizeof(int32_t));
    g.n_unique = take(&cur, sizeof(int32_t));
    g.state = g.unique;
  }
  const size_t tiles = (NNZ + kSortTile - 1) / kSortTile;
  lay->seg_state = take(&cur, tiles * sizeof(int32_t));   // three words a tile
  take(&cur, tiles * sizeof(int32_t));
  take(&cur, tiles * sizeof(int32_t));
  lay->units = take(&cur, NNZ * sizeof(UnitDesc));
  lay->row_view = take(&cur, NNZ * sizeof(int32_t));
  lay->row_scale = take(&cur, NNZ * sizeof(float));
  lay->n_units = take(&cur, sizeof(int32_t));
  lay->failed = lay->n_units + kAlign / 2;   // in the same line of kAlign bytes
  lay->expiry_marks = take(&cur, (size_t)expiry_words(c.n_images) * sizeof(uint32_t));
  lay->expiry_tiles = take(&cur, (size_t)expiry_tiles(c.n_images) * sizeof(int32_t));
  lay->total = cur;
  return true;
}

}  // namespace gear

using namespace gear;

// Scratch memory of gear_step_static: one array per device, inside the code object, so that the call
// needs no allocation.  In host code the array's name only stands for the symbol; the address of a
// device's copy comes from hipGetSymbolAddress with that device current, and that address is what
// the kernels are given.
#define GEAR_STATIC_SCRATCH_BYTES (64u << 20)
static __device__ __align__(256) unsigned char scratch[GEAR_STATIC_SCRATCH_BYTES];

namespace {
void *g_scratch_ptr[64];
std::mutex g_scratch_mutex;

// address of the current device's copy of `scratch` (looked up once per device); nullptr on failure
void *static_scratch() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
    if ((uintptr_t)ptr & 255u) return nullptr;
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

// One helper stream and five events per device, created on first use and kept for the life of the
// process: the integer grouping of a long step runs beside its gather and forward pass.
namespace {
struct SideLane {
  hipStream_t stream = nullptr;
  hipEvent_t fork = nullptr, join = nullptr, join_captured = nullptr, checked = nullptr;
  bool ready = false;
  // Two programs that step on streams of their own may collect gradients in one store, so what steps do to it has to happen
  // in the order in which they were issued, whichever form each takes.  Long steps do it on the helper stream; a short one
  // does it on its caller's, waits for what the last step left, and leaves this event.
  hipEvent_t done = nullptr;
  hipEvent_t *last = nullptr;   // what the last step left: `done`, or `join` of a long one (nullptr before the first)
  std::mutex busy;  // held while a step enqueues: two host threads never interleave their forks and joins
};
SideLane g_side[64];
std::mutex g_side_mutex;

// multiply-adds of the DFV-slot part of the dLoss/dx product from which it is worth an extra launch
// and event to let the embedding update run beside it (about 10 us of work on the device)
constexpr double kSplitDxMacs = 5e9;

// Ids of a batch (users, URLs and images) from which a step uses the helper stream.  Its events cost the host 65 us a step
// and the device four idle gaps; a shorter step has less than that to hide.  Layer by layer, on one stream with the grouping
// carried by other launches against two streams: 2 300 ids 53 / 99 us, 15 000 82 / 119, 27 000 106 / 128, 63 000 154 / 178 (the
// slowest host seen), 65 000 143 .. 152 / 144; from there on 89 000 169 / 153, 106 000 187 / 172, 172 000 198 / 182.
// Steps that go in blocks of views (rows.hip) have other forms on either side.  Their lists of ids in LDS or in launches beside
// them, one image a view: 16 383 and 16 384 views of 192 -> 128 bf16 68 / 108, 320 -> 256 bf16 75 / 113, 320 -> 256 fp32 137 / 162, so
// that this line is below where it would be for them alone.  Grouping carried or blocks on two streams: 576 -> 512 -> 256 bf16, 58 000
// ids 134 / 123, 106 000 184 / 152; narrow networks would carry on (192 -> 128 bf16, 64 000 ids 97 / 110, 106 000 114 / 117; 96 -> 64
// fp32, 106 000 106 / 119).
constexpr long long kOneStreamIds = 49152;
// ... and the multiply-adds of its forward products, in bf16; four times that of fp32.  Weight gradients that long are worth
// hiding the accumulation behind however few ids there are.  Layer by layer, one stream / two, us, of steps of 12 000 to 48 000
// ids: bf16, 5.2e9 126 / 132, 5.9e9 138 / 137, 6.8e9 154 / 149, 7.2e9 169 / 151, 8.9e9 197 / 167, 23e9 311 / 256; fp32, 0.9e9
// 131 / 129, 1.2e9 148 / 149, 1.4e9 179 / 183, 1.7e9 191 / 183, 2.4e9 225 / 214, 2.9e9 311 / 288.
constexpr double kOneStreamMacs = 6.8e9;

// The lane of the current device, with the helper stream if it is wanted; nullptr when one of its objects cannot be created
// (nothing half-made is kept: the next call starts over).
SideLane *side_lane(bool helper) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lock(g_side_mutex);
  SideLane &l = g_side[dev];
  // no fence beyond the device: only its streams wait for this event, and the fence was half of its price
  if (!l.done && hipEventCreateWithFlags(&l.done, hipEventDisableTiming | hipEventDisableSystemFence) != hipSuccess) {
    l.done = nullptr;
    return nullptr;
  }
  if (helper && !l.ready) {
    hipStream_t stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr, join_captured = nullptr, checked = nullptr;
    bool ok = hipStreamCreateWithFlags(&stream, hipStreamNonBlocking) == hipSuccess;
    // Those that only streams of this device wait for go without a fence beyond it, as `done` does (a step of 65 536 views with all
    // of them so 950 us against 958).  `join` keeps it: without, the helper stream is reported as busy after it has ended.
    ok = ok && hipEventCreateWithFlags(&fork, hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&join, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&join_captured, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&checked, hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess;
    if (!ok) {
      if (checked) (void)hipEventDestroy(checked);
      if (join_captured) (void)hipEventDestroy(join_captured);
      if (join) (void)hipEventDestroy(join);
      if (fork) (void)hipEventDestroy(fork);
      if (stream) (void)hipStreamDestroy(stream);
      return nullptr;
    }
    l.stream = stream;
    l.fork = fork;
    l.join = join;
    l.join_captured = join_captured;
    l.checked = checked;
    l.ready = true;
  }
  return &l;
}

bool capturing(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

// A step's use of the lane, with the helper stream or for its place in the order alone.  Holds the lane for the whole
// enqueue, so that steps issued from
// several host threads on one device use the lane's events one after the other, and makes sure
// that whatever was forked to the helper stream is joined back into the caller's stream however the
// enqueue ends: after an early return (a failed launch) the next call on the caller's stream must
// not run beside kernels this call left on the helper stream.
class LaneScope {
 public:
  // books: what the step does to the store of gradients, it does on the helper stream
  LaneScope(SideLane *lane, bool helper, bool books, bool captured, hipStream_t caller)
      : lane_(lane), side_(helper ? lane : nullptr), s_(caller), captured_(captured), books_(helper && books),
        join_(!helper ? nullptr : captured ? lane->join_captured : lane->join) {
    if (lane_) lane_->busy.lock();
  }
  ~LaneScope() {
    if (!lane_) return;
    if (side_ && forked_ && !joined_) {
      if (hipEventRecord(join_, side_->stream) == hipSuccess) (void)hipStreamWaitEvent(s_, join_, 0);
    }
    if (entered_ && !captured_) {
      if (books_) {
        if (forked_) lane_->last = &lane_->join;   // else it ended before it gave the helper anything
      } else if (done_left_ || hipEventRecord(lane_->done, s_) == hipSuccess) {
        lane_->last = &lane_->done;
      }
    }
    lane_->busy.unlock();
  }
  LaneScope(const LaneScope &) = delete;
  LaneScope &operator=(const LaneScope &) = delete;
  // The step takes its place behind the last one.  Of two long steps the helper stream keeps the order by itself; behind or
  // ahead of a short one it takes an event.  (In an earlier form a short step paid 2 us for one recorded behind it, 49.7 -> 51.8, 78.6 ->
  // 80.5 and 104.9 -> 106.6 us on the three smallest workloads, and for one left by its last launch itself 0.3 us where the device was the
  // slower side and 4 us where the host was.  Now the latter is the cheaper one on either side: done_by.)
  // A step that is being captured has the place its graph is launched in; it leaves the events of the others alone.
  // `on`: the stream that first looks at the store; what the step gives to its streams before this call, or to others than this
  // one, runs beside the steps ahead of it (us for a step of each of two programs on streams of their own, with the whole step
  // behind the other's / so: 16 384 views bf16 334 / 267, 192 -> 128 bf16 244 / 198, 320 -> 256 fp32 361 / 277; 32 768 views of
  // 1152 -> 1024 -> 256 beside 16 384 of 576 -> 512 -> 256 642 / 602).
  hipError_t enter(hipStream_t on) {
    if (!lane_) return hipSuccess;
    hipError_t e = hipSuccess;
    const bool in_order = side_ && on == side_->stream && lane_->last == &lane_->join;
    if (!captured_ && lane_->last && !in_order) e = hipStreamWaitEvent(on, *lane_->last, 0);
    entered_ = e == hipSuccess;
    return e;
  }
  // The launches that an event is to come behind leave it themselves where they can: what follows on the stream then waits for no
  // event's packet (us between the ends of a launch and the start of the next one on its stream, with the packet / without: 8 to 10 / 3;
  // from a launch on one stream to one on the other that waits for it 10 to 12 / 6 to 8).  us a step, all events recorded / left: 512 views
  // 26.4 / 25.4, 4096 fp32 74.3 / 72.7, 16 384 fp32 164.4 / 159.6, bf16 151.5 / 149.4, 65 536 936.5 / 930.6.  The host issues a step of 512
  // views in 18.6 / 18.2 us (23.5 / 22.7 on a slower core), of 16 384 in 70 / 64 (85 / 90), and one that is waited for takes 47 / 46 and
  // 173 / 174; first passes on a new state differ by no more than two of one build (58 / 57, 230 / 241, 1112 / 1104).  Not while they are
  // being captured.  `left`: the launch ahead was given the event.
  hipEvent_t fork_by() const { return side_ && !captured_ ? side_->fork : nullptr; }
  hipEvent_t mark_by() const { return side_ && !captured_ ? join_ : nullptr; }
  hipEvent_t mark_checked_by() const { return side_ && !captured_ ? side_->checked : nullptr; }
  hipEvent_t done_by() const { return lane_ && !captured_ && !books_ ? lane_->done : nullptr; }
  void done_left() { done_left_ = done_by() != nullptr; }   // it was the step's last launch
  // what the caller's stream has done so far happens before whatever the helper stream is given next
  hipError_t fork(bool left) {
    if (!side_) return hipSuccess;
    if (!left || captured_)
      if (hipError_t e = hipEventRecord(side_->fork, s_)) return e;
    forked_ = true;
    joined_ = false;
    return hipStreamWaitEvent(side_->stream, side_->fork, 0);
  }
  // marks the point of the helper stream that a later wait() refers to
  hipError_t mark(bool left) { return side_ && (!left || captured_) ? hipEventRecord(join_, side_->stream) : hipSuccess; }
  // the same for the end of the helper's first part (ids checked, plan made): the status word is final
  hipError_t mark_checked(bool left) { return side_ && (!left || captured_) ? hipEventRecord(side_->checked, side_->stream) : hipSuccess; }
  hipError_t wait_checked() { return side_ ? hipStreamWaitEvent(s_, side_->checked, 0) : hipSuccess; }
  // the caller's stream continues after the last mark(); final = nothing is given to the helper after it
  hipError_t wait(bool final) {
    if (!side_) return hipSuccess;
    hipError_t e = hipStreamWaitEvent(s_, join_, 0);
    if (e == hipSuccess && final) joined_ = true;
    return e;
  }

 private:
  SideLane *lane_, *side_;   // side_: the lane if the helper stream is used
  hipStream_t s_;
  const bool captured_, books_;
  const hipEvent_t join_;
  bool entered_ = false, forked_ = false, joined_ = false, done_left_ = false;
};
}  // namespace

// Test hook: the n-th launch of this thread's next steps reports failure instead of being enqueued
// (0 = off).  Lets a test walk the error paths of a step without a failing device.
thread_local int g_fail_at = 0;
inline bool fail_injected() { return g_fail_at > 0 && --g_fail_at == 0; }

#define GEAR_HIP(expr)                             \
  do {                                             \
    if ((expr) != hipSuccess) return GEAR_ERR_HIP; \
  } while (0)
// a launch bracketed by profile events (when a profile is attached)
#define GEAR_RUN(name, expr)    \
  do {                          \
    if (fail_injected()) return GEAR_ERR_HIP; \
    Span span_(prof, name, s);  \
    GEAR_HIP(expr);             \
  } while (0)

extern "C" {

size_t gear_workspace_bytes(const gear_config *cfg) {
  Layout lay;
  if (!cfg || !make_layout(*cfg, &lay)) return 0;
  return lay.total;
}

int64_t gear_mlp_param_count(const gear_config *cfg) {
  Layout lay;
  if (!cfg || !make_layout(*cfg, &lay)) return -1;
  return lay.n_params;
}

int64_t gear_mlp_param_offset(const gear_config *cfg, int32_t layer, int32_t which) {
  Layout lay;
  if (!cfg || !make_layout(*cfg, &lay) || layer < 0 || layer >= lay.L || which < 0 || which > 1) return -1;
  return which == 0 ? lay.w_off[layer] : lay.b_off[layer];
}

gear_status gear_workspace_region(const gear_config *cfg, const char *name, size_t *offset, size_t *bytes) {
  Layout lay;
  if (!cfg || !name || !offset || !bytes || !make_layout(*cfg, &lay)) return GEAR_ERR_INVALID;
  const size_t B = (size_t)cfg->max_batch;
  if (!strcmp(name, "x")) {
    *offset = lay.x;
    *bytes = B * lay.F * lay.act_bytes;
  } else if (!strcmp(name, "logits")) {
    *offset = lay.logits;
    *bytes = B * sizeof(float);
  } else if (!strcmp(name, "dx_emb")) {
    *offset = lay.dx_emb;
    *bytes = B * 2 * cfg->emb_dim * sizeof(float);
  } else if (!strcmp(name, "dx_dfv")) {
    *offset = lay.dx_dfv;
    *bytes = B * cfg->dfv_dim * lay.act_bytes;
  } else if (name[0] == 'h' && name[1] >= '0' && name[1] < '0' + GEAR_MAX_LAYERS && !name[2] &&
             name[1] - '0' < lay.L - 1) {
    const int l = name[1] - '0';
    *offset = lay.h[l];
    *bytes = B * lay.out_dim[l] * lay.act_bytes;
  } else {
    return GEAR_ERR_INVALID;
  }
  return GEAR_OK;
}

gear_status gear_fill_normal(void *dst, int32_t dtype, int64_t n_rows, int32_t dim, uint64_t seed,
                             uint32_t stream_id, float std, void *stream) {
  if (!dst || n_rows < 0 || dim < 1 || (dtype != GEAR_F32 && dtype != GEAR_BF16) || !(std >= 0.0f) || !isfinite(std))
    return GEAR_ERR_INVALID;
  GEAR_HIP(launch_fill_normal(dst, dtype, n_rows * dim, seed, stream_id, std, (hipStream_t)stream));
  return GEAR_OK;
}

gear_status gear_init_tables(const gear_config *cfg, gear_tables *t, float *grad_accum, int32_t *counts,
                             void *stream) {
  Layout lay;
  if (!cfg || !t || !t->user_emb || !t->url_emb || !t->mlp_params || !grad_accum || !counts) return GEAR_ERR_INVALID;
  if (!make_layout(*cfg, &lay) || !aligned16(grad_accum) || !aligned16(counts) || !aligned16(t->mlp_params))
    return GEAR_ERR_INVALID;
  hipStream_t s = (hipStream_t)stream;
  if (!static_scratch()) return GEAR_ERR_HIP;  // looked up here so that a later gear_step_static need not
  GEAR_HIP(launch_fill_normal(t->user_emb, cfg->emb_dtype, cfg->n_users * cfg->emb_dim, cfg->seed, 1u,
                              cfg->emb_init_std, s));
  GEAR_HIP(launch_fill_normal(t->url_emb, cfg->emb_dtype, cfg->n_urls * cfg->emb_dim, cfg->seed, 2u,
                              cfg->emb_init_std, s));
  GEAR_HIP(launch_fill_zero(t->mlp_params, (size_t)lay.n_params * sizeof(float), s));
  for (int l = 0; l < lay.L; ++l)
    GEAR_HIP(launch_fill_normal(t->mlp_params + lay.w_off[l], GEAR_F32, (int64_t)lay.in_dim[l] * lay.out_dim[l],
                                cfg->seed, 16u + (uint32_t)l, sqrtf(2.0f / (float)lay.in_dim[l]), s));
  GEAR_HIP(launch_fill_zero(grad_accum, (size_t)cfg->n_images * cfg->dfv_dim * sizeof(float), s));
  GEAR_HIP(launch_fill_zero(counts, (size_t)cfg->n_images * sizeof(int32_t), s));
  return GEAR_OK;
}

gear_status gear_step(const gear_config *cfg, const gear_batch *b, gear_tables *t, const void *dfv_cache,
                      float *grad_accum, int32_t *counts, int32_t M, float lr, void *workspace,
                      size_t workspace_bytes, gear_step_out *out, void *stream) {
  return gear_step_adam(cfg, b, t, dfv_cache, grad_accum, counts, M, lr, nullptr, workspace, workspace_bytes, out,
                        stream);
}

gear_status gear_step_static(const gear_config *cfg, const gear_batch *b, gear_tables *t, const void *dfv_cache,
                             float *grad_accum, int32_t *counts, int32_t M, float lr, gear_step_out *out,
                             void *stream) {
  Layout lay;
  if (!cfg || !out || !make_layout(*cfg, &lay)) return GEAR_ERR_INVALID;
  if (lay.total > GEAR_STATIC_SCRATCH_BYTES) return GEAR_ERR_CAPACITY;
  void *ws = static_scratch();
  if (!ws) return GEAR_ERR_HIP;
  // every kernel on the caller's stream: no helper stream or event has to exist
  gear_step_out o = *out;
  o.one_stream = 1;
  return gear_step_adam(cfg, b, t, dfv_cache, grad_accum, counts, M, lr, nullptr, ws, GEAR_STATIC_SCRATCH_BYTES, &o,
                        stream);
}

gear_status gear_step_adam(const gear_config *cfg, const gear_batch *b, gear_tables *t, const void *dfv_cache,
                           float *grad_accum, int32_t *counts, int32_t M, float lr, const gear_adam *adam,
                           void *workspace, size_t workspace_bytes, gear_step_out *out, void *stream) {
  Layout lay;
  if (!cfg || !b || !t || !dfv_cache || !grad_accum || !counts || !workspace || !out) return GEAR_ERR_INVALID;
  if (!make_layout(*cfg, &lay)) return GEAR_ERR_INVALID;
  if (!t->user_emb || !t->url_emb || !t->mlp_params) return GEAR_ERR_INVALID;
  if (!out->loss || !out->n_ready || !out->ready_ids || !out->ready_grads || !out->status || out->ready_cap < 0)
    return GEAR_ERR_INVALID;
  if (M < 1 || !isfinite(lr)) return GEAR_ERR_INVALID;
  if (b->B < 0 || b->nnz < 0 || b->B > cfg->max_batch || b->nnz > cfg->max_nnz) return GEAR_ERR_INVALID;
  if (b->B > 0 && (!b->user_id || !b->url_id || !b->img_off || !b->label)) return GEAR_ERR_INVALID;
  if (b->nnz > 0 && (!b->img_id || b->B == 0)) return GEAR_ERR_INVALID;
  if (((uintptr_t)workspace & (kAlign - 1)) || !aligned16(grad_accum) || !aligned16(out->ready_grads) ||
      !aligned16(dfv_cache) || !aligned16(t->user_emb) || !aligned16(t->url_emb) || !aligned16(t->mlp_params))
    return GEAR_ERR_INVALID;
  if (workspace_bytes < lay.total) return GEAR_ERR_CAPACITY;

  // the update rule and where each parameter array keeps its moments
  Optim opt = {lr, 0.0f, 0.0f, 0.0f, 1.0f, 0};
  Moments mom_mlp = {nullptr, nullptr}, mom_user = {nullptr, nullptr}, mom_url = {nullptr, nullptr};
  if (adam) {
    if (!(adam->beta1 >= 0.0f && adam->beta1 < 1.0f) || !(adam->beta2 >= 0.0f && adam->beta2 < 1.0f) ||
        !(adam->eps > 0.0f) || adam->t < 1)
      return GEAR_ERR_INVALID;
    if (!adam->user_m || !adam->user_v || !adam->url_m || !adam->url_v || !adam->mlp_m || !adam->mlp_v)
      return GEAR_ERR_INVALID;
    if (!aligned16(adam->user_m) || !aligned16(adam->user_v) || !aligned16(adam->url_m) || !aligned16(adam->url_v) ||
        !aligned16(adam->mlp_m) || !aligned16(adam->mlp_v))
      return GEAR_ERR_INVALID;
    opt.adam = 1;
    opt.beta1 = adam->beta1;
    opt.beta2 = adam->beta2;
    opt.eps = adam->eps;
    opt.lr = (float)((double)lr / (1.0 - pow((double)adam->beta1, (double)adam->t)));
    opt.inv_bc2 = (float)(1.0 / sqrt(1.0 - pow((double)adam->beta2, (double)adam->t)));
    mom_mlp = {adam->mlp_m, adam->mlp_v};
    mom_user = {adam->user_m, adam->user_v};
    mom_url = {adam->url_m, adam->url_v};
  }

  hipStream_t s = (hipStream_t)stream;
  char *ws = (char *)workspace;
  const int B = b->B, L = lay.L, F = lay.F, dt = cfg->mlp_dtype;
  int32_t *failed = (int32_t *)(ws + lay.failed);   // what the step's kernels look at; out->status is told as well

  gear_profile *prof = (gear_profile *)out->profile;
  if (prof) prof->used = 0;
  static const char *const kFwd[GEAR_MAX_LAYERS] = {"fwd_gemm_l0", "fwd_gemm_l1", "fwd_gemm_l2", "fwd_gemm_l3",
                                                    "fwd_gemm_l4", "fwd_gemm_l5", "fwd_gemm_l6", "fwd_gemm_l7"};
  static const char *const kDgrad[GEAR_MAX_LAYERS] = {"dgrad_gemm_l0", "dgrad_gemm_l1", "dgrad_gemm_l2",
                                                      "dgrad_gemm_l3", "dgrad_gemm_l4", "dgrad_gemm_l5",
                                                      "dgrad_gemm_l6", "dgrad_gemm_l7"};
  if (B == 0) {
    GEAR_RUN("begin", launch_begin(out->status, failed, out->n_ready, out->loss, ZeroList{}, dt, nullptr, 0, false, nullptr, s, nullptr));
    return GEAR_OK;
  }
  int32_t *occ_view = (int32_t *)(ws + lay.occ_view);
  const int E2 = 2 * cfg->emb_dim;   // columns of the embedding slots

  // On one stream the launches of the forward pass carry the grouping along where they can (gemm_tile.hip); with two, the
  // helper stream has it.
  bool moderate = true;
  for (int l = 0; l < L - 1; ++l) moderate = moderate && gemm_nt_carries(dt, B, lay.out_dim[l], lay.in_dim[l]);
  double macs = 0.0;
  for (int l = 0; l < L - 1; ++l) macs += (double)B * lay.in_dim[l] * lay.out_dim[l];
  const bool is_short = (long long)2 * B + b->nnz < kOneStreamIds && macs * (dt == GEAR_BF16 ? 1 : 4) < kOneStreamMacs;
  // In blocks of views: the whole network in one launch (rows.hip), of a short step with the grouping of the ids in its first
  // workgroups.  A longer one has the grouping on the other stream, by tiles that are counted ahead of every pass
  // (group_device.hpp), from the prologue on, which counts the first pass, so that it is done when the weight gradients are, and the bookkeeping
  // follows those on the caller's (accumulation beside weight gradients, in one launch or on two streams, took as long as one
  // behind the other, and the wait for the blocks 10 us more).  us a step, tiles that look back / counted: 16 384 views of 576 ->
  // 512 -> 256 bf16, 106 000 ids, 170 / 158; of 320 -> 256 fp32, 172 000 ids, 178 / 166.
  RowsPlan rows;
  const bool long_dx = (double)B * (F - 2 * cfg->emb_dim) * lay.out_dim[0] >= kSplitDxMacs;
  TnProblem widths[GEAR_MAX_LAYERS];   // of the weight-gradient products
  size_t all_partials = 0;
  for (int l = L - 2; l >= 0; --l) {
    widths[L - 2 - l] = TnProblem{nullptr, nullptr, nullptr, lay.out_dim[l], lay.in_dim[l]};
    all_partials += (size_t)lay.out_dim[l] * lay.in_dim[l];
  }
  const TnChoice first_choice = gemm_tn_choice(dt, widths, L - 1, B);
  const bool one_group = first_choice.layers == L - 1 && all_partials * sizeof(float) <= lay.wgrad_partial_bytes;
  const bool planned = (is_short || (!long_dx && one_group)) && plan_rows(*cfg, lay, B, b->nnz, is_short, &rows);
  const int key_bits[kMaxProblems] = {bits_for(cfg->n_users), bits_for(cfg->n_urls), bits_for(cfg->n_images)};
  int own_passes[kMaxProblems];   // of a longer step's lists, where their tiles' counts have room: hardly any image, and they have not
  bool fit = true;
  for (int i = 0; planned && !is_short && i < kMaxProblems; ++i) {
    const bool last = i == kMaxProblems - 1;
    own_passes[i] = counted_passes(key_bits[i], last ? b->nnz : B, last ? cfg->max_nnz : cfg->max_batch, rows.digit_bits);
    fit = fit && own_passes[i] > 0;
  }
  // On one stream nothing runs beside the blocks of a longer step, while the launches of its layers carry the grouping: it goes
  // layer by layer, with its batch sums in the shape the blocks would leave (block_sums.hpp), so that both forms have the same
  // bits.  us a step on one stream, layers / blocks, 576 -> 512 -> 256 bf16: 9001 views 134 / 154, 12 288 148 / 165, 16 384 184 / 188;
  // 192 -> 128, 10 000 views 97 / 110; 96 -> 64 fp32, 16 384 106 / 127.  The sums are 1 to 4 of it.
  const bool by_rows = planned && (is_short || !out->one_stream), as_rows = planned && !by_rows;
  const bool local_sort = by_rows && is_short, long_rows = by_rows && !is_short;
  const bool beside = local_sort && !first_choice.large && one_group;   // accumulation and weight gradients are one launch
  const bool no_prologue = beside && rows.direct;
  rows.direct = no_prologue;
  // Every tile reads the counts of all, so very long lists go back to tiles that look back (us a step, look back / counted, of
  // 64-view blocks: 576 -> 512 -> 256 bf16, 327 000 images of 16 384 views 221 / 229; 192 -> 128, 290 000 of 20 000 167 / 170, 785 000 of
  // 16 384 262 / 317.  Below: 239 000 of 8000 149 / 137, 158 000 of 4000 views of 576 -> 512 -> 256 152 / 155, 59 000 of 2000 99 / 93, 54 000 of
  // 1200 99 / 100).
  const bool very_long = b->nnz > 128 * kSortTile, counted = long_rows && fit && !very_long;
  // Very long lists beside blocks of 32 views, which leave less of a CU, are on the caller's stream, so that their sorts start ahead
  // of the blocks, which go to the helper's with the weight gradients (us a step, on the helper's / on the caller's: 16 384 views of 20
  // images, 320 -> 256 fp32 209 / 193, 8000 of 40, 192 -> 128 bf16 164 / 151; but blocks of 64, 16 384 of 20, 576 -> 512 -> 256 221 / 230).
  const bool group_here = long_rows && very_long && rows.rows == 32;
  const bool one_stream = out->one_stream != 0 || local_sort || (moderate && is_short);
  const bool carried = one_stream && moderate && !by_rows;
  // Layer by layer, weights that are operands of products on the large tiles lie in those tiles' order (gemm.hip): the forward
  // product's copy, and the transpose but for the rows of the embedding slots where dLoss/dx is made in two products.
  bool w_tiles[GEAR_MAX_LAYERS] = {};
  int wt_tiles_from[GEAR_MAX_LAYERS];
  for (int l = 0; l < L; ++l) wt_tiles_from[l] = INT32_MAX;
  for (int l = 0; l < L - 1 && !by_rows && !carried; ++l) {
    const int in = lay.in_dim[l], width = lay.out_dim[l];
    if (in % 32 || width % 32) continue;
    w_tiles[l] = gemm_nt_takes_tiles(dt, B, width, in, EPI_BIAS_RELU);
    const int from = l == 0 && long_dx ? E2 : 0;
    if (from % 32 == 0 && gemm_nt_takes_tiles(dt, B, in - from, width, l == 0 ? EPI_DX : EPI_MASK_BITS)) wt_tiles_from[l] = from;
  }

  // grouping of the three id lists and the plan of the per-image accumulation
  GroupBatch gb;
  {
    int passes = 1;   // the lists share launches: as many passes for all as the widest ids need
    for (int i = 0; i < kMaxProblems; ++i) {
      const int need = radix_passes(key_bits[i], lay.g[i].total_words, carried ? kSideDigitBits : long_rows && rows.rows == 64 ? kBesideDigitBits : widest_digit(B > b->nnz ? B : b->nnz));
      if (need > passes) passes = need;
    }
    // a pass that is carried costs nothing but its length, and narrow digits make it short: as many as find a launch ahead
    // of the one that takes the segments
    const int rides = L < kMaxRides ? L : kMaxRides;   // the forward products and the logit layer
    if (carried && passes < rides) passes = rides;
    gb.count = kMaxProblems;
    gb.p[0] = make_problem(lay, ws, 0, b->user_id, B, cfg->n_users, counted ? own_passes[0] : passes, key_bits[0]);
    gb.p[1] = make_problem(lay, ws, 1, b->url_id, B, cfg->n_urls, counted ? own_passes[1] : passes, key_bits[1]);
    gb.p[2] = make_problem(lay, ws, 2, b->img_id, b->nnz, cfg->n_images, counted ? own_passes[2] : passes, key_bits[2]);
    gb.tickets = (int32_t *)(ws + lay.tickets);
    gb.seg_state = (uint32_t *)(ws + lay.seg_state);
    if (!out->dbg_img_unique && !out->dbg_img_segoff) gb.p[2].unique = gb.p[2].segoff = nullptr;   // nothing in the step reads them
  }
  AccumPlan plan;
  plan.units = (UnitDesc *)(ws + lay.units);
  plan.row_view = (int32_t *)(ws + lay.row_view);
  plan.row_scale = (float *)(ws + lay.row_scale);
  plan.n_units = (int32_t *)(ws + lay.n_units);
  plan.row_at = local_sort ? gb.p[2].perm : nullptr;
  plan.local = no_prologue ? local_result(rows, gb, b->nnz, out->ready_cap) : LocalResult{};
  LocalOutputs local_out = {};
  if (local_sort) local_out = LocalOutputs{plan.local, out->status, out->n_ready};
  const PlanArgs plan_args = {plan, occ_view, b->img_off, counts, M, out->ready_cap, out->n_ready, out->status};
  // Not carried: what depends only on ids and counters (the check of the ids, the grouping, the accumulation plan) runs on
  // the helper stream while the main stream gathers and runs the forward pass.  The
  // main stream waits for it before the first kernel that changes caller state, so the status word
  // is final by then; until then its kernels write the workspace only, and the gather clamps what it
  // uses as an index.
  // A caller who asks for one stream gets no event either; a step that is short keeps its place in the order.
  const bool ordered = out->one_stream == 0, captured = ordered && capturing(s);
  const bool needs_lane = !one_stream || (ordered && !captured);
  SideLane *side = needs_lane ? side_lane(!one_stream) : nullptr;
  if (needs_lane && !side) return GEAR_ERR_HIP;
  hipStream_t helper = one_stream ? s : side->stream;
  LaneScope lane(side, !one_stream, !by_rows, captured, s);
  // Layer by layer on two streams the helper has all that looks at the store.  Blocks take their place ahead of the launch that
  // first does, and run beside the step of another program until then (us for a step of each of two programs, at once / so, 290 000
  // images of 20 000 views, 192 -> 128 bf16, 344 / 257; 319 000 of 8000 351 / 229; LaneScope::enter).
  if (!long_rows) GEAR_HIP(lane.enter(helper));
  const ViewCheck views = {b->img_off, occ_view, B, b->nnz};
  {
    // Step outputs and counters cleared and the operand copies of the weights made in one launch ahead of everything:
    // the first product then needs no event, and behind the gather's many workgroups the copies would not get onto the
    // device before it ends anyway.
    CastJob jobs[GEAR_MAX_LAYERS];
    const int n_jobs = by_rows ? L - 1 : L;   // the logit layer is one row, which rows.hip takes from the parameters
    for (int l = 0; l < n_jobs; ++l)
      jobs[l] = CastJob{t->mlp_params + lay.w_off[l], ws + lay.wc[l], ws + lay.wct[l], lay.out_dim[l], lay.in_dim[l],
                        w_tiles[l], wt_tiles_from[l]};
    ZeroList zero;
    zero.count = 0;
    if (local_sort)
      local_zero_list(gb, &zero);
    else if (counted)
      counted_zero_list(gb, &zero);
    else
      group_zero_list(gb, &zero);
    FirstCounts first;
    if (counted) first = first_counts(gb, views);
    if (!no_prologue)
      GEAR_RUN(counted ? "group_count" : "begin",
             launch_begin(out->status, failed, out->n_ready, out->loss, zero, dt, jobs, n_jobs, by_rows, counted ? &first : nullptr, s, lane.fork_by()));
  }
  if (!carried && !local_sort) GEAR_HIP(lane.fork(true));
  // Carried: the links of the grouping in order, each taken by the next launch that can.
  SideTask task;
  int link = 0;
  const int links = carried ? group_passes(gb) + 1 : 0;
  auto passenger = [&]() -> const SideTask * {
    if (link >= links) return nullptr;
    task = side_task(gb, plan_args, link++, failed);
    return &task;
  };
  auto links_left = [&]() -> gear_status {   // those that found no launch to ride in
    for (; link < links; ++link)
      GEAR_RUN(link + 1 < links ? "group_ids" : "accum_plan",
               link + 1 < links ? launch_radix_pass(gb, link, failed, s) : launch_segments(gb, &plan_args, failed, s));
    return GEAR_OK;
  };
  // forward
  void *x = ws + lay.x;
  // the weight-gradient products of the hidden layers
  TnProblem wp[GEAR_MAX_LAYERS];
  int n_wp = 0;
  for (int l = L - 2; l >= 0; --l)
    wp[n_wp++] = TnProblem{ws + lay.delta[l], l == 0 ? x : ws + lay.h[l - 1], nullptr, lay.out_dim[l], lay.in_dim[l]};
  float *logits = (float *)(ws + lay.logits), *dz = (float *)(ws + lay.dz);
  float *dx_emb = (float *)(ws + lay.dx_emb);
  void *dx_dfv = ws + lay.dx_dfv;
  if (by_rows) {
    LocalTask local = {};
    if (local_sort) local = local_task(rows, gb, plan_args, views, failed, out->loss);
    hipStream_t caller = s;
    {
      hipStream_t s = group_here ? helper : caller;
      GEAR_RUN("view_blocks", launch_rows(*cfg, lay, rows, *b, *t, dfv_cache, ws, local, s));
    }
  } else {
    const CheckTask check = check_task(gb, b->img_off, occ_view, B, b->nnz, failed, out->status);
    GEAR_RUN("gather_pool", launch_gather_pool(*cfg, *b, *t, dfv_cache, x, s, carried ? &check : nullptr));
  }
  // A bf16 hidden layer below the last one also leaves the sign bitmap of its activations: the backward pass then
  // reads one bit per unit instead of the activation.
  uint8_t *relu_bits[GEAR_MAX_LAYERS] = {};
  if (dt == GEAR_BF16)
    for (int l = 0; l + 2 < L; ++l) relu_bits[l] = (uint8_t *)(ws + lay.relu_bits[l]);
  for (int l = 0; l < L - 1 && !by_rows; ++l) {
    GEAR_RUN(kFwd[l], launch_gemm_nt(dt, l == 0 ? x : ws + lay.h[l - 1], ws + lay.wc[l], B, lay.out_dim[l],
                                     lay.in_dim[l], EPI_BIAS_RELU, t->mlp_params + lay.b_off[l], nullptr,
                                     ws + lay.h[l], 0, nullptr, relu_bits[l], nullptr, s, false, passenger(), w_tiles[l]));
  }
  // The helper stream's launches are issued after the forward pass's: where the host is not ahead of the
  // device (a caller that waits for every step), the gather then starts as soon as the step does, not
  // after the host has issued the grouping's launches.
  if (!carried && !local_sort) {
    hipStream_t caller = s, s = group_here ? caller : helper;  // the stream of this block's launches
    const hipEvent_t end = group_here ? nullptr : long_rows ? lane.mark_by() : lane.mark_checked_by();   // left by the last of them
    if (counted) {
      const int passes = group_passes(gb), plan_behind = gb.p[2].n > 0 ? gb.p[2].passes : 1;   // how many passes the plan comes behind
      for (int pass = 0; pass < passes; ++pass) {
        if (pass > 0 && pass != plan_behind) GEAR_RUN("group_count", launch_count(gb, pass, s));
        GEAR_RUN("group_ids", launch_counted_pass(gb, pass, views, plan_args, failed, s, pass + 1 == passes && pass >= plan_behind ? end : nullptr));
        if (pass + 1 == plan_behind) {
          GEAR_HIP(lane.enter(s));
          GEAR_RUN("accum_plan", launch_segments_count(gb, plan_args, plan_behind, failed, s, pass + 1 == passes ? end : nullptr));
        }
      }
    } else {
      GEAR_RUN("group_ids", launch_check(gb, b->img_off, occ_view, B, b->nnz, failed, out->status, s));
      for (int pass = 0; pass < group_passes(gb); ++pass) GEAR_RUN("group_ids", launch_radix_pass(gb, pass, failed, s));
      if (long_rows) GEAR_HIP(lane.enter(s));
      GEAR_RUN("accum_plan", launch_segments(gb, &plan_args, failed, s, end));
    }
    if (!group_here) GEAR_HIP(long_rows ? lane.mark(true) : lane.mark_checked(true));
  }

  // Until its first kernel that changes caller state (the first SGD on a hidden layer's weights), the
  // caller's stream writes the workspace only and need not know whether the ids were in range or the
  // ready list fits.  Just before that kernel the stream waits for the helper's first part, so that the
  // status word is final.
  if (!by_rows) {
    GEAR_RUN("logit_loss", launch_logit_loss(dt, ws + lay.h[L - 2], ws + lay.wc[L - 1], t->mlp_params + lay.b_off[L - 1],
                                           b->label, B, lay.in_dim[L - 1], logits, dz, ws + lay.delta[L - 2],
                                           (float *)(ws + lay.loss_partial), failed, s, passenger()));
  }

  // backward through the hidden layers down to dLoss/dx (all from the pre-step operand copies)
  // Each product that makes the delta of a hidden layer also leaves that layer's bias gradient (column
  // sums of the delta) as per-row-tile partials; they are added in tile order at the end of the step.
  float *cpart = (float *)(ws + (planned ? rows.colsum : lay.colsum_partial)), *wpart = (float *)(ws + lay.wgrad_partial);
  const EmbeddingWork emb = embedding_work(*cfg, gb.p[0], gb.p[1], dx_emb, t->user_emb, t->url_emb, (float *)(ws + lay.emb_partial),
                                           opt, mom_user, mom_url, plan, counts);
  // Small sums whose results nothing in the step reads: the loss, the logit layer and the biases (column sums of deltas,
  // left as per-row-tile partials by the products that made them).
  ColumnSum columns[kMaxColumnSums];
  int n_columns = 0;
  const LogitSums sums = planned ? rows_sums(rows, (const float *)(ws + lay.loss_partial), lay.in_dim[L - 1])
                                 : logit_sums((const float *)(ws + lay.loss_partial), B, lay.in_dim[L - 1]);
  auto column = [&](const float *partial, int parts, int width, int64_t at) {
    columns[n_columns++] = ColumnSum{partial, t->mlp_params + at, moments_at(mom_mlp, at), parts, width};
  };
  column(sums.w, sums.parts, lay.in_dim[L - 1], lay.w_off[L - 1]);
  column(sums.delta, sums.parts, lay.in_dim[L - 1], lay.b_off[L - 2]);
  column(sums.bias, sums.parts, 1, lay.b_off[L - 1]);
  for (int l = L - 2; l > 0; --l)
    column(cpart + (planned ? rows.colsum_at[l] : lay.colsum_at[l]),
           planned ? rows.blocks : gemm_nt_colsum_parts(dt, B, lay.in_dim[l], lay.out_dim[l], lay.colsum_coarse),
           lay.out_dim[l - 1], lay.b_off[l - 1]);
  const LossSum loss = {sums.loss, out->loss, sums.parts, B};
  bool divided = false;
  for (int l = L - 2; l >= 0 && !by_rows; --l) {
    if (l > 0) {
      const bool by_bits = relu_bits[l - 1] != nullptr;
      GEAR_RUN(kDgrad[l], launch_gemm_nt(dt, ws + lay.delta[l], ws + lay.wct[l], B, lay.in_dim[l], lay.out_dim[l],
                                         by_bits ? EPI_MASK_BITS : EPI_MASK, nullptr,
                                         by_bits ? (const void *)relu_bits[l - 1] : (const void *)(ws + lay.h[l - 1]),
                                         ws + lay.delta[l - 1], 0, as_rows ? nullptr : cpart + lay.colsum_at[l], nullptr, nullptr, s,
                                         lay.colsum_coarse, nullptr, wt_tiles_from[l] == 0));
    } else {
      // dLoss/dx: the embedding slots stay fp32, the DFV slot is kept in the MLP's operand type.
      // When the product is long enough to hide it, it is made in two parts: the embedding slots
      // first, and as soon as they are there the SGD on the touched embedding rows starts on the
      // helper stream, beside the larger product that makes the DFV slot.  Every element is computed
      // the same way in both forms.
      if (long_dx) {
        GEAR_RUN("dgrad_gemm_emb", launch_gemm_nt(dt, ws + lay.delta[0], ws + lay.wct[0], B, E2, lay.out_dim[0], EPI_DX,
                                                  nullptr, dx_dfv, dx_emb, E2, nullptr, nullptr, nullptr, s, false, nullptr, false,
                                                  lane.fork_by()));
        if (gear_status st = links_left()) return st;
        GEAR_HIP(lane.fork(true));
        {
          hipStream_t s = helper;
          GEAR_RUN("small_sums", launch_param_update(nullptr, 0, 1, columns, n_columns, loss, nullptr, LocalOutputs{}, opt, failed, s));
          GEAR_RUN("embedding_update", launch_embedding_update(emb, true, failed, s));
        }
        divided = true;
        GEAR_RUN(kDgrad[0], launch_gemm_nt(dt, ws + lay.delta[0],
                                           ws + lay.wct[0] + (size_t)E2 * lay.out_dim[0] * lay.act_bytes, B, F - E2,
                                           lay.out_dim[0], EPI_DX, nullptr, dx_dfv, dx_emb, 0, nullptr, nullptr, nullptr, s, false, nullptr,
                                           wt_tiles_from[0] == E2, lane.fork_by()));
      } else {
        const bool takes = gemm_nt_carries(dt, B, F, lay.out_dim[0]);
        GEAR_RUN(kDgrad[0], launch_gemm_nt(dt, ws + lay.delta[0], ws + lay.wct[0], B, F, lay.out_dim[0], EPI_DX,
                                           nullptr, dx_dfv, dx_emb, E2, nullptr, nullptr, nullptr, s, false,
                                           takes ? passenger() : nullptr, wt_tiles_from[0] == 0, lane.fork_by()));
        if (gear_status st = links_left()) return st;
      }
    }
  }

  // The per-image gradient bookkeeping only needs dLoss/dx and is bound by memory traffic: it runs on
  // the helper stream beside the weight-gradient products, which are not.  The products are
  // launched first and, where they can, as one launch of at most one round of workgroups, so that
  // they hold their CUs before the bookkeeping's many small workgroups arrive and fill what is
  // left; a product arriving later would wait until all of those have been placed.
  // In blocks of views the two are one launch where the products go on small tiles in one group.
  // Behind blocks of views the grouping may still be at work: the products fill that time, and the bookkeeping follows them
  // on the caller's stream.
  const bool books_here = one_stream || by_rows;
  const bool ends_here = !out->dbg_img_unique && !out->dbg_img_segoff && !out->dbg_img_perm && !out->dbg_n_img_unique;   // with the last update
  if (!by_rows) GEAR_HIP(lane.fork(true));
  auto bookkeeping = [&](hipStream_t s) -> gear_status {
    if (!divided && !books_here) GEAR_RUN("embedding_update", launch_embedding_update(emb, false, failed, s));
    BlockSums riding;
    if (as_rows) riding = block_sums_of(rows, lay, *b, ws);
    GEAR_RUN("accumulate", launch_accumulate(*cfg, gb.p[2], plan, dx_dfv, grad_accum, M, out->ready_ids, out->ready_grads,
                                             divided ? nullptr : &emb, !books_here, as_rows ? &riding : nullptr, failed, s,
                                             books_here ? nullptr : lane.mark_by()));
    return GEAR_OK;
  };
  if (!beside && !long_rows) {
    if (gear_status st = bookkeeping(helper)) return st;
    GEAR_HIP(lane.mark(true));
  }
  // SGD on the hidden layers' weights: split-K wgrad.  With the last of them go the small sums, unless they are done.
  // All layers go out as one launch, in as many ranges of the batch as their partials have room for; a model whose
  // partials do not fit at once (several wide layers and a short batch), or with more large tiles than fill the device,
  // goes in groups of layers.
  for (int first = 0; first < n_wp;) {
    const size_t room = lay.wgrad_partial_bytes / sizeof(float);
    size_t all = 0;
    int n = 0;
    const TnChoice choice = gemm_tn_choice(dt, wp + first, n_wp - first, B);
    while (n < choice.layers && all + (size_t)wp[first + n].M * wp[first + n].N <= room) {
      all += (size_t)wp[first + n].M * wp[first + n].N;
      ++n;
    }
    if (n == 0) return GEAR_ERR_CAPACITY;  // cannot happen: the region holds one range of the widest layer
    bool pairs = !beside;
    int splits = gemm_tn_splits(dt, wp + first, n, B, choice.large, &pairs);
    // Beside the accumulation two thirds as many: the CUs are not theirs alone, and every range is partials to write and to
    // add (us a step, all / two thirds / half: 4096 views 82.2 / 80.4 / 80.4, 5000 64.3 / 63.5 / 65.4).
    if (beside) splits = (2 * splits + 2) / 3;
    if (splits > (int)(room / all)) splits = (int)(room / all);
    float *next = wpart;
    SplitkProblem sp[GEAR_MAX_LAYERS];
    for (int i = 0; i < n; ++i) {
      TnProblem &q = wp[first + i];
      const int l = L - 2 - (first + i);
      q.partial = next;
      next += (size_t)splits * q.M * q.N;
      sp[i] = SplitkProblem{q.partial, t->mlp_params + lay.w_off[l], moments_at(mom_mlp, lay.w_off[l]), (int64_t)q.M * q.N};
    }
    if (beside) {
      GEAR_RUN("accumulate_wgrad", launch_accumulate_wgrad(*cfg, gb.p[2], plan, dx_dfv, grad_accum, M, out->ready_ids, out->ready_grads,
                                                           emb, wp, n, B, splits, failed, s));
    } else {
      hipStream_t caller = s;
      hipStream_t s = group_here ? helper : caller;
      GEAR_RUN("wgrad_gemm", launch_gemm_tn(dt, wp + first, n, B, splits, choice.large, pairs, nullptr, s));
    }
    // The sums of the partials and the SGD change caller state, so the status word has to be final: the
    // stream waits for the helper's first part (long done by now), not for the bookkeeping.  Their
    // workgroups get onto the device as the bookkeeping's leave room and are done before it is, so the
    // step ends with the bookkeeping and the join.
    if (first == 0 && long_rows) {
      if (group_here) GEAR_HIP(lane.mark(false));
      GEAR_HIP(lane.wait(true));
      if (gear_status st = bookkeeping(s)) return st;
    } else if (first == 0) {
      GEAR_HIP(lane.wait_checked());
    }
    first += n;
    const bool sums_too = first == n_wp && !divided;   // else the helper stream has done them
    GEAR_RUN("param_update", launch_param_update(sp, n, splits, columns, sums_too ? n_columns : 0, sums_too ? loss : LossSum{},
                                                 sums_too && books_here ? &emb : nullptr, local_out, opt, failed, s,
                                                 first == n_wp && ends_here ? lane.done_by() : nullptr));
    if (first == n_wp && ends_here) lane.done_left();
  }
  if (!by_rows) GEAR_HIP(lane.wait(true));  // the step ends on the caller's stream
  if (no_prologue && !ends_here)
    GEAR_RUN("grouping_out", launch_unique(plan.local, gb.p[2].unique, gb.p[2].segoff, b->nnz, out->dbg_img_unique, out->dbg_img_segoff,
                                           out->dbg_n_img_unique, s));
  if (!no_prologue && out->dbg_img_unique && b->nnz > 0)
    GEAR_HIP(hipMemcpyAsync(out->dbg_img_unique, gb.p[2].unique, (size_t)b->nnz * 4, hipMemcpyDeviceToDevice, s));
  if (!no_prologue && out->dbg_img_segoff)
    GEAR_HIP(hipMemcpyAsync(out->dbg_img_segoff, gb.p[2].segoff, ((size_t)b->nnz + 1) * 4, hipMemcpyDeviceToDevice, s));
  if (out->dbg_img_perm && b->nnz > 0)
    GEAR_HIP(hipMemcpyAsync(out->dbg_img_perm, gb.p[2].perm, (size_t)b->nnz * 4, hipMemcpyDeviceToDevice, s));
  if (!no_prologue && out->dbg_n_img_unique)
    GEAR_HIP(hipMemcpyAsync(out->dbg_n_img_unique, gb.p[2].n_unique, 4, hipMemcpyDeviceToDevice, s));
  return GEAR_OK;
}

gear_status gear_refresh_dfv(const gear_config *cfg, void *dfv_cache, const int32_t *image_ids, const void *new_dfv,
                             int64_t n, int32_t *status, void *stream) {
  if (!cfg || !config_ok(*cfg) || !dfv_cache || n < 0 || (n > 0 && !new_dfv)) return GEAR_ERR_INVALID;
  if (!aligned16(dfv_cache) || !aligned16(new_dfv)) return GEAR_ERR_INVALID;
  if (!image_ids && n > cfg->n_images) return GEAR_ERR_INVALID;
  GEAR_HIP(launch_refresh(cfg->dfv_dtype, dfv_cache, cfg->n_images, cfg->dfv_dim, image_ids, new_dfv, n, status,
                          (hipStream_t)stream));
  return GEAR_OK;
}

gear_status gear_refresh_dfv_n(const gear_config *cfg, void *dfv_cache, const int32_t *image_ids, const void *new_dfv,
                               const int32_t *n_rows, int64_t max_rows, int32_t *status, void *stream) {
  if (!cfg || !config_ok(*cfg) || !dfv_cache || !image_ids || !n_rows || max_rows < 0 || (max_rows > 0 && !new_dfv))
    return GEAR_ERR_INVALID;
  if (!aligned16(dfv_cache) || !aligned16(new_dfv)) return GEAR_ERR_INVALID;
  GEAR_HIP(launch_refresh(cfg->dfv_dtype, dfv_cache, cfg->n_images, cfg->dfv_dim, image_ids, new_dfv, max_rows, status,
                          (hipStream_t)stream, n_rows));
  return GEAR_OK;
}

gear_status gear_stamp_dfv_n(const gear_config *cfg, int32_t *dfv_stamp, const int32_t *image_ids, const int32_t *n_rows,
                             int64_t max_rows, int32_t now, int32_t *status, void *stream) {
  if (!cfg || !config_ok(*cfg) || !dfv_stamp || !image_ids || !n_rows || max_rows < 0) return GEAR_ERR_INVALID;
  GEAR_HIP(launch_stamp(dfv_stamp, cfg->n_images, image_ids, max_rows, now, status, (hipStream_t)stream, n_rows));
  return GEAR_OK;
}

gear_status gear_group_ids(const gear_config *cfg, const int32_t *keys, int32_t n, int64_t key_range, void *workspace,
                           size_t workspace_bytes, int32_t *unique, int32_t *segoff, int32_t *perm, int32_t *n_unique,
                           void *stream) {
  Layout lay;
  if (!cfg || !make_layout(*cfg, &lay) || !workspace || !unique || !segoff || !perm || !n_unique)
    return GEAR_ERR_INVALID;
  if (n < 0 || n > cfg->max_nnz || (n > 0 && !keys) || key_range < 1 || key_range > ((int64_t)1 << 31))
    return GEAR_ERR_INVALID;
  if ((uintptr_t)workspace & (kAlign - 1)) return GEAR_ERR_INVALID;
  if (workspace_bytes < lay.total) return GEAR_ERR_CAPACITY;
  hipStream_t s = (hipStream_t)stream;
  char *ws = (char *)workspace;
  int32_t *failed = (int32_t *)(ws + lay.failed);  // cleared below: nothing can fail here
  GroupBatch gb;
  gb.count = 1;
  const int bits = bits_for(key_range);
  gb.p[0] = make_problem(lay, ws, 2, keys, n, 0, radix_passes(bits, lay.g[2].total_words, widest_digit(n)), bits);
  gb.tickets = (int32_t *)(ws + lay.tickets);
  gb.seg_state = (uint32_t *)(ws + lay.seg_state);
  ZeroList zero;
  group_zero_list(gb, &zero);
  zero.p[zero.count] = (uint32_t *)failed;
  zero.words[zero.count++] = 1;
  GEAR_HIP(launch_clear(zero, s));
  GEAR_HIP(launch_check(gb, nullptr, nullptr, 0, 0, failed, failed, s));
  for (int pass = 0; pass < group_passes(gb); ++pass) GEAR_HIP(launch_radix_pass(gb, pass, failed, s));
  GEAR_HIP(launch_segments(gb, nullptr, failed, s));
  if (n > 0) {
    GEAR_HIP(hipMemcpyAsync(unique, gb.p[0].unique, (size_t)n * 4, hipMemcpyDeviceToDevice, s));
    GEAR_HIP(hipMemcpyAsync(perm, gb.p[0].perm, (size_t)n * 4, hipMemcpyDeviceToDevice, s));
  }
  GEAR_HIP(hipMemcpyAsync(segoff, gb.p[0].segoff, ((size_t)n + 1) * 4, hipMemcpyDeviceToDevice, s));
  GEAR_HIP(hipMemcpyAsync(n_unique, gb.p[0].n_unique, 4, hipMemcpyDeviceToDevice, s));
  return GEAR_OK;
}

gear_status gear_expired_ids(const gear_config *cfg, const int32_t *image_ids, int32_t n, const int32_t *dfv_stamp,
                             int32_t now, int32_t expiry, void *workspace, size_t workspace_bytes,
                             int32_t *expired_ids, int32_t *n_expired, int32_t *status, void *stream) {
  Layout lay;
  if (!cfg || !make_layout(*cfg, &lay) || !workspace || !dfv_stamp || !expired_ids || !n_expired || !status)
    return GEAR_ERR_INVALID;
  if (n < 0 || n > cfg->max_nnz || (n > 0 && !image_ids) || expiry < 0) return GEAR_ERR_INVALID;
  if ((uintptr_t)workspace & (kAlign - 1)) return GEAR_ERR_INVALID;
  if (workspace_bytes < lay.total) return GEAR_ERR_CAPACITY;
  hipStream_t s = (hipStream_t)stream;
  char *ws = (char *)workspace;
  GEAR_HIP(launch_fill_zero(status, sizeof(int32_t), s));
  GEAR_HIP(launch_expired(image_ids, n, dfv_stamp, cfg->n_images, now, expiry, (uint8_t *)(ws + lay.expiry_marks),
                          (int32_t *)(ws + lay.expiry_tiles), expired_ids, n_expired, status, s));
  return GEAR_OK;
}

gear_status gear_stamp_dfv(const gear_config *cfg, int32_t *dfv_stamp, const int32_t *image_ids, int64_t n,
                           int32_t now, int32_t *status, void *stream) {
  if (!cfg || !config_ok(*cfg) || !dfv_stamp || n < 0) return GEAR_ERR_INVALID;
  if (!image_ids && n > cfg->n_images) return GEAR_ERR_INVALID;
  GEAR_HIP(launch_stamp(dfv_stamp, cfg->n_images, image_ids, n, now, status, (hipStream_t)stream));
  return GEAR_OK;
}

gear_status gear_gemm(int32_t dtype, int32_t form, const void *A, const void *B, int32_t M, int32_t N, int32_t K,
                      int32_t epilogue, const float *bias, const void *aux, void *out, int32_t splits,
                      float *partial, int32_t *status, void *stream) {
  if ((dtype != GEAR_F32 && dtype != GEAR_BF16) || !A || !B || !out || !status || M < 1 || N < 1 || K < 1)
    return GEAR_ERR_INVALID;
  const int vec = dtype == GEAR_BF16 ? 8 : 4;
  if (!aligned16(A) || !aligned16(B) || !aligned16(out)) return GEAR_ERR_INVALID;
  hipStream_t s = (hipStream_t)stream;
  if (form == 0) {
    if (K % vec || N % vec || epilogue < EPI_BIAS_RELU || epilogue > EPI_F32) return GEAR_ERR_INVALID;
    if ((epilogue == EPI_BIAS_RELU && !bias) || (epilogue == EPI_MASK && (!aux || !aligned16(aux))))
      return GEAR_ERR_INVALID;
    GEAR_HIP(launch_gemm_nt(dtype, A, B, M, N, K, epilogue, bias, aux, out, 0, nullptr, nullptr, status, s));
  } else if (form == 1) {
    if (M % vec || N % vec || splits < 1 || splits > 64 || !partial) return GEAR_ERR_INVALID;
    const TnProblem one = {A, B, partial, M, N};
    GEAR_HIP(launch_gemm_tn(dtype, &one, 1, K, splits, gemm_tn_choice(dtype, &one, 1, K).large, true, status, s));
    GEAR_HIP(launch_fill_zero(out, (size_t)M * N * sizeof(float), s));
    const Optim minus = {-1.0f, 0.0f, 0.0f, 0.0f, 1.0f, 0};   // out = 0 - (-1) * sum of the partials
    const Moments none = {nullptr, nullptr};
    const SplitkProblem sum = {partial, (float *)out, none, (int64_t)M * N};
    GEAR_HIP(launch_param_update(&sum, 1, splits, nullptr, 0, LossSum{}, nullptr, LocalOutputs{}, minus, status, s));
  } else {
    return GEAR_ERR_INVALID;
  }
  return GEAR_OK;
}

void gear_debug_fail_launch(int32_t nth) { g_fail_at = nth > 0 ? nth : 0; }

int32_t gear_debug_helper_idle(void) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return -1;
  std::lock_guard<std::mutex> lock(g_side_mutex);
  if (!g_side[dev].ready) return 1;
  const hipError_t e = hipStreamQuery(g_side[dev].stream);
  return e == hipSuccess ? 1 : (e == hipErrorNotReady ? 0 : -1);
}

gear_profile *gear_profile_create(void) {
  gear_profile *p = new (std::nothrow) gear_profile;
  if (!p) return nullptr;
  p->used = 0;
  int made = 0;  // events created so far, start[0], stop[0], start[1], ...
  for (; made < 2 * gear_profile::kMaxSpans; ++made) {
    const int i = made / 2;
    p->name[i] = "";
    if (hipEventCreate(made % 2 ? &p->stop[i] : &p->start[i]) != hipSuccess) break;
  }
  if (made < 2 * gear_profile::kMaxSpans) {
    for (int e = 0; e < made; ++e) (void)hipEventDestroy(e % 2 ? p->stop[e / 2] : p->start[e / 2]);
    delete p;
    return nullptr;
  }
  return p;
}

void gear_profile_destroy(gear_profile *p) {
  if (!p) return;
  for (int i = 0; i < gear_profile::kMaxSpans; ++i) {
    (void)hipEventDestroy(p->start[i]);
    (void)hipEventDestroy(p->stop[i]);
  }
  delete p;
}

int32_t gear_profile_count(const gear_profile *p) { return p ? p->used : 0; }

gear_status gear_profile_span(const gear_profile *p, int32_t i, const char **name, float *ms) {
  if (!p || !name || !ms || i < 0 || i >= p->used) return GEAR_ERR_INVALID;
  *name = p->name[i];
  GEAR_HIP(hipEventElapsedTime(ms, p->start[i], p->stop[i]));
  return GEAR_OK;
}

const char *gear_status_string(gear_status st) {
  switch (st) {
    case GEAR_OK: return "ok";
    case GEAR_ERR_INVALID: return "invalid argument";
    case GEAR_ERR_RANGE: return "id out of range or offsets not a CSR index";
    case GEAR_ERR_CAPACITY: return "workspace or ready list too small";
    case GEAR_ERR_HIP: return "HIP call failed";
  }
  return "unknown status";
}

}  // extern "C"
