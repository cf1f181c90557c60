// A block of views taken through the whole Sparse Part in one launch (Section 3, steps 1-4): gather, forward pass, loss
// and backward pass down to dLoss/dx.  All of it is local to a view except the weights, so a workgroup keeps the
// activations of its 16 to 64 views in LDS from the gather to dLoss/dx and streams every layer's weights past them, once
// forward and once backward; what the batch sums need (x, h, delta, dLoss/dx) is written to the workspace on the way.  Beside
// the blocks of a short step the first workgroups sort the lists of ids (local_group.hpp); a longer one sorts them on the
// other stream.
//
// Layer by layer a short step is a chain of eight to twelve dependent launches of 4 to 16 us, each of which pays its ramp,
// the latency of its first operands and the links of the grouping it carries.  Here the chain is four launches: the prologue,
// this one, accumulation beside weight gradients (accum_wgrad.hip) and the parameter update; small fp32 networks need no prologue
// (kDirectBytes).  us a step, layer by layer / so, 512 views fp32 51 / 25, 4096 views of 320 -> 256 -> 128 fp32 104 / 73, 5000 of 288 ->
// 256 fp32 79 / 59, 1000 of 336 -> 320 -> 72 -> 64 bf16 86 / 41.  What bounds it: a chain of phases.  4096 views in fp32 take 28 us here:
// gather 5, products 6, 4, 3 and 5.5 (the matrix instructions 12 of them), logit layer 1, its columns 1.3, the sums of delta 1; 512 views
// of 96 -> 64 take 9: 3.5, 1.5 and 1, logit 1, columns 1.3.  Run a second time in the same launch a block of the latter is 1 us shorter, so
// neither the fetch of instructions nor that of cold weights is what is left.
//
// The weights come straight from memory (every XCD's L2 holds them) into the registers of the one wavefront that owns
// those columns: they are laid out in operand order ahead of the step (prep.hip), so that a wavefront's load is 1 KB in one
// piece.  Each weight is read once per workgroup: 1.7 MB for 64 views of 576 -> 512 -> 256, at half of the 64 bytes a clock that a CU gets from
// L2, is what bounds the products of the larger networks (touching all of them ahead of the gather made no difference).
//
// Every product adds k in ascending order, in steps of the 16 x 16 matrix instructions, which gives the bits of the
// 32 x 32 ones of the other product kernels: a hidden unit next to zero takes the same branch in either form of a step.
#include "gemm_common.hpp"
#include "local_group.hpp"
#include "rows.hpp"

#include <string.h>

namespace gear {
namespace {

typedef float f32x4_v __attribute__((ext_vector_type(4)));

// A k-step is 64 bytes of every operand row, 16 bytes per lane: lane (q, r) = (lane / 16, lane % 16) holds row r, and of
// the step's k-values 8 q .. 8 q + 7 (bf16) or q, 4 + q, 8 + q, 12 + q (fp32, one for each of four instructions).  LDS rows
// of activations are kept in that order too: fp32 column k sits at 16 (k / 16) + 4 (k % 4) + (k / 4) % 4.
template <typename T> struct Step;
template <> struct Step<bf16_t> {
  static constexpr int K = 32;
  static __device__ __forceinline__ uint32_t byte_of(int k) { return (uint32_t)k * 2u; }
  static __device__ __forceinline__ void mma(f32x4_v &acc, const u32x4_v &w, const u32x4_v &a) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_v, w), __builtin_bit_cast(bf16x8_v, a), acc, 0, 0, 0);
  }
};
template <> struct Step<float> {
  static constexpr int K = 16;
  static __device__ __forceinline__ uint32_t byte_of(int k) { return (uint32_t)((k & ~15) | ((k & 3) << 2) | ((k >> 2) & 3)) * 4u; }
  static __device__ __forceinline__ void mma(f32x4_v &acc, const u32x4_v &w, const u32x4_v &a) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[e]), __uint_as_float(a[e]), acc, 0, 0, 0);
  }
};

// four neighbouring columns (col a multiple of 4) of an activation row in LDS
__device__ __forceinline__ void lds_put4(unsigned char *row, int col, const float (&v)[4], bf16_t) {
  *reinterpret_cast<uint2 *>(row + col * 2) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
}
__device__ __forceinline__ void lds_put4(unsigned char *row, int col, const float (&v)[4], float) {
  float *at = reinterpret_cast<float *>(row + Step<float>::byte_of(col));
#pragma unroll
  for (int j = 0; j < 4; ++j) at[4 * j] = v[j];
}
__device__ __forceinline__ void lds_get4(const unsigned char *row, int col, float (&v)[4], bf16_t) {
  const uint2 t = *reinterpret_cast<const uint2 *>(row + col * 2);
  v[0] = __uint_as_float(t.x << 16), v[1] = __uint_as_float(t.x & 0xffff0000u);
  v[2] = __uint_as_float(t.y << 16), v[3] = __uint_as_float(t.y & 0xffff0000u);
}
__device__ __forceinline__ void lds_get4(const unsigned char *row, int col, float (&v)[4], float) {
  const float *at = reinterpret_cast<const float *>(row + Step<float>::byte_of(col));
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = at[4 * j];
}
template <int CTRL> __device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppRor4 = 0x124, kDppRor8 = 0x128;
// The same in fp32 by whole quads of lanes that have neighbouring columns of one row, the first a multiple of 16: the quad's sixteen
// columns are four 16-byte pieces of LDS, each with one column of every lane.  One access without bank conflicts and a transpose
// in registers, where four accesses of four bytes have eight lanes on every bank.
__device__ __forceinline__ void quad_transpose(float (&v)[4]) {
  const bool odd = threadIdx.x & 1, high = threadIdx.x & 2;
#pragma unroll
  for (int k = 0; k < 4; k += 2) {
    const float t = dpp<kDppXor1>(odd ? v[k] : v[k + 1]);
    v[k] = odd ? t : v[k], v[k + 1] = odd ? v[k + 1] : t;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float t = dpp<kDppXor2>(high ? v[k] : v[k + 2]);
    v[k] = high ? t : v[k], v[k + 2] = high ? v[k + 2] : t;
  }
}
__device__ __forceinline__ void quad_get4(const unsigned char *row, int col, float (&v)[4]) {
  const float4 t = *reinterpret_cast<const float4 *>(row + (size_t)col * 4);
  v[0] = t.x, v[1] = t.y, v[2] = t.z, v[3] = t.w;
  quad_transpose(v);
}

// Sum over the wavefront, in the pairs of lanes that xor by 32, 16, ... 1 makes.  (Behind the first three steps a value depends on the
// lane's last three bits, so a rotation by four is an xor.)  In registers: through LDS the six steps of a logit were 1 us of the 2 to 3
// that the logit layer took.
__device__ __forceinline__ float wave_sum(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  v += dpp<kDppRor8>(v);
  v += dpp<kDppRor4>(v);
  v += dpp<kDppXor2>(v);
  v += dpp<kDppXor1>(v);
  return v;
}

__device__ __forceinline__ void store4(bf16_t *dst, const float (&v)[4]) {
  *reinterpret_cast<uint2 *>(dst) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
}
__device__ __forceinline__ void store4(float *dst, const float (&v)[4]) {
  *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
}

// four values as they are stored
__device__ __forceinline__ void round4(float (&v)[4], bf16_t) {
  const uint32_t a = pack_bf16(v[0], v[1]), b = pack_bf16(v[2], v[3]);
  v[0] = __uint_as_float(a << 16), v[1] = __uint_as_float(a & 0xffff0000u);
  v[2] = __uint_as_float(b << 16), v[3] = __uint_as_float(b & 0xffff0000u);
}
__device__ __forceinline__ void round4(float (&)[4], float) {}

// acc[j][i] += W[16 (tile0 + j) .. + 15][0 .. K) (a + 16 i rows)^T: lane (q, r) ends with columns 16 (tile0 + j) + 4 q .. + 3 of row
// 16 i + r.  `w` is in operand order, `act` the lane's place in the first activation row.  AHEAD k-steps of weights are in
// flight: an L2 latency is one to two k-steps of products.  `meet`: called once, when the first of them are.
template <typename T, int MT, int NT, int AHEAD, typename Meet>
__device__ __forceinline__ void rows_product(f32x4_v (&acc)[NT][MT], const unsigned char *act, int stride, const void *w, int N,
                                             int K, int tile0, int q, int r, Meet meet) {
  constexpr int ES = (int)sizeof(T), SK = Step<T>::K;
  const int steps = K / SK, step_bytes = 64 * N;   // all rows' 64 bytes of a k-step lie together
  // a step's place is a scalar offset, a lane's 32 bits: with 64-bit addresses per lane and tile the registers would not do
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(w), 0, N * K * ES, 0x00020000);
  int lane_at[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int rows = min(16, N - 16 * (tile0 + j));   // the missing rows of a last tile repeat its last one and are not stored
    lane_at[j] = (tile0 + j) * 1024 + (q * rows + min(r, rows - 1)) * 16;
  }
  u32x4_v wf[AHEAD][NT], af[MT];
  auto weights = [&](u32x4_v (&to)[NT], int s) {
    const int at = min(s, steps - 1) * step_bytes;
#pragma unroll
    for (int j = 0; j < NT; ++j) to[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_at[j], at, 0);
  };
  auto views = [&](u32x4_v (&to)[MT], int s) {
#pragma unroll
    for (int i = 0; i < MT; ++i) to[i] = *reinterpret_cast<const u32x4_v *>(act + i * 16 * stride + s * 64);
  };
  auto products = [&](const u32x4_v (&wt)[NT], const u32x4_v (&at)[MT]) {
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int i = 0; i < MT; ++i) Step<T>::mma(acc[j][i], wt[j], at[i]);
  };
  if (steps > 0) {
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) weights(wf[d], d);
  }
  meet();
  int s0 = 0;
  for (; s0 + AHEAD <= steps; s0 += AHEAD) {
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) {
      views(af, s0 + d);
      products(wf[d], af);
      weights(wf[d], s0 + d + AHEAD);
      __builtin_amdgcn_sched_barrier(0);   // registers
    }
  }
#pragma unroll
  for (int d = 0; d < AHEAD - 1; ++d)
    if (s0 + d < steps) {
      views(af, s0 + d);
      products(wf[d], af);
    }
  if (K % SK) {   // the rest of K, zero beyond it (K is a multiple of 8; LDS rows are padded with zeros)
    const char *rest = static_cast<const char *>(w) + (size_t)steps * step_bytes;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int first = 16 * (tile0 + j), rows = min(16, N - first), row = min(r, rows - 1);
      u32x4_v wt = {0u, 0u, 0u, 0u};
      if constexpr (ES == 2) {
        const int pieces = (K % SK) / 8;
        if (q < pieces) wt = *reinterpret_cast<const u32x4_v *>(rest + ((size_t)first * pieces + q * rows + row) * 16);
      } else {
        const uint2 t = *reinterpret_cast<const uint2 *>(rest + ((size_t)first * 4 + q * rows + row) * 8);
        wt.x = t.x, wt.y = t.y;
      }
#pragma unroll
      for (int i = 0; i < MT; ++i)
        Step<T>::mma(acc[j][i], wt, *reinterpret_cast<const u32x4_v *>(act + i * 16 * stride + steps * 64));
    }
  }
}

enum RowsEpi { ROWS_FORWARD, ROWS_BACK, ROWS_DX };

// The same from the fp32 weights themselves, row-major, sixteen views: forward W [N x K], of which a lane has four neighbouring k, and
// the four lanes of a row exchange them; backward W [K x N], four words of four rows.  No launch has to lay them out first.
template <int NT, int AHEAD, bool BACK, typename Meet>
__device__ __forceinline__ void rows_product_direct(f32x4_v (&acc)[NT][1], const unsigned char *act, const void *w, int N, int K, int tile0,
                                                    int q, int r, Meet meet) {
  constexpr int SK = Step<float>::K;
  const int steps = K / SK;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(w), 0, N * K * 4, 0x00020000);
  int lane_at[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int n = min(16 * (tile0 + j) + r, N - 1);   // the missing rows of a last tile repeat its last one and are not stored
    lane_at[j] = BACK ? (q * N + n) * 4 : (n * K + 4 * q) * 4;
  }
  u32x4_v wf[AHEAD][NT];
  auto weights = [&](u32x4_v (&to)[NT], int s) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      if constexpr (BACK) {
#pragma unroll
        for (int e = 0; e < 4; ++e) to[j][e] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, lane_at[j], min(SK * s + 4 * e, K - 4) * N * 4, 0);
      } else {
        to[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_at[j], s * SK * 4, 0);
      }
    }
  };
  auto products = [&](u32x4_v (&wt)[NT], int s) {
    const u32x4_v at = *reinterpret_cast<const u32x4_v *>(act + s * 64);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      if constexpr (!BACK) {   // lane q has k = 4 q + e, and is to have q + 4 e
        auto swap16 = [&](int a, int b) {
          const auto t = __builtin_amdgcn_permlane16_swap(wt[j][a], wt[j][b], false, false);
          wt[j][a] = t[0], wt[j][b] = t[1];
        };
        auto swap32 = [&](int a, int b) {
          const auto t = __builtin_amdgcn_permlane32_swap(wt[j][a], wt[j][b], false, false);
          wt[j][a] = t[0], wt[j][b] = t[1];
        };
        swap16(0, 1), swap16(2, 3), swap32(0, 2), swap32(1, 3);
      }
      Step<float>::mma(acc[j][0], wt[j], at);
    }
  };
#pragma unroll
  for (int d = 0; d < AHEAD; ++d)
    if (d < steps) weights(wf[d], d);
  meet();
  int s0 = 0;
  for (; s0 + AHEAD <= steps; s0 += AHEAD) {
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) {
      products(wf[d], s0 + d);
      weights(wf[d], min(s0 + d + AHEAD, steps - 1));
      __builtin_amdgcn_sched_barrier(0);   // registers
    }
  }
#pragma unroll
  for (int d = 0; d < AHEAD - 1; ++d)
    if (s0 + d < steps) products(wf[d], s0 + d);
  if (K % SK) {   // eight more, zero beyond them (LDS rows are padded with zeros): of a lane's four the first two, or those of two lanes
    u32x4_v last[NT];
    if constexpr (BACK) {
      weights(last, steps);
#pragma unroll
      for (int j = 0; j < NT; ++j) last[j][2] = last[j][3] = 0u;
    } else {
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        last[j] = u32x4_v{0u, 0u, 0u, 0u};
        if (q < 2) last[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_at[j], steps * SK * 4, 0);
      }
    }
    products(last, steps);
  }
}

template <typename T, int MT, bool DIRECT, int NT, int EPI, typename Meet>
__device__ __forceinline__ void rows_tiles_of(const RowsArgs &p, unsigned char *lds, const RowsBuf &in, const RowsBuf &out,
                                              const void *w, int N, int K, const float *bias, T *global, int row0, int tile0,
                                              int lane, Meet meet) {
  constexpr int AHEAD = MT == 1 ? 4 : 2;
  const int q = lane >> 4, r = lane & 15;
  float b[NT][4];
  if constexpr (EPI == ROWS_FORWARD) {   // requested ahead of the products
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int n = 16 * (tile0 + j) + 4 * q;
      const float4 t = n < N ? *reinterpret_cast<const float4 *>(bias + n) : make_float4(0.f, 0.f, 0.f, 0.f);
      b[j][0] = t.x, b[j][1] = t.y, b[j][2] = t.z, b[j][3] = t.w;
    }
  }
  f32x4_v acc[NT][MT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[j][i][e] = 0.0f;
  const unsigned char *act = lds + in.at + r * in.stride + q * 16;
  if constexpr (DIRECT)
    rows_product_direct<NT, AHEAD, EPI != ROWS_FORWARD>(acc, act, w, N, K, tile0, q, r, meet);
  else
    rows_product<T, MT, NT, AHEAD>(acc, act, in.stride, w, N, K, tile0, q, r, meet);
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int n = 16 * (tile0 + j) + 4 * q;
    if (n >= N) continue;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int row = 16 * i + r, view = row0 + row;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = acc[j][i][e];
      if constexpr (EPI == ROWS_DX) {
        const int E2 = 2 * p.d;
        if (view < p.B) {
          if (n < E2)
            store4(p.dx_emb + (size_t)view * E2 + n, v);
          else
            store4(static_cast<T *>(p.dx_dfv) + (size_t)view * p.D + (n - E2), v);
        }
      } else {
        unsigned char *at = lds + out.at + row * out.stride;
        if constexpr (EPI == ROWS_FORWARD) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[e] += b[j][e];
            v[e] = v[e] > 0.0f ? v[e] : 0.0f;
          }
        } else {   // the activation makes room for its delta
          float h[4];
          lds_get4(at, n, h, T{});
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = h[e] > 0.0f ? v[e] : 0.0f;
        }
        lds_put4(at, n, v, T{});
        if constexpr (sizeof(T) == 4 && EPI == ROWS_FORWARD)
          if (view < p.B) store4(global + (size_t)view * N + n, v);
      }
    }
  }
}

// One layer's product by the whole workgroup: the first N / 16 % 8 of eight shares have a column tile more (shares w and w + 4
// are on one SIMD, so those of 36 tiles have nine each).  The workgroups of an XCD start with different shares, so that its
// L2 is not asked for the same lines by all of them at once.  `meet`: what has to come between the launch's earlier phases and the
// first read of `in`, by every wavefront once; its first weights are on their way meanwhile.
template <typename T, int MT, bool DIRECT, int EPI, typename Meet>
__device__ __forceinline__ void rows_layer(const RowsArgs &p, unsigned char *lds, const RowsBuf &in, const RowsBuf &out, const void *w,
                                           int N, int K, const float *bias, T *global, int row0, int wave, int lane, Meet meet) {
  const int tiles = (N + 15) / 16, least = tiles / kRowsWaves, more = tiles % kRowsWaves;
  const int share = (wave + blockIdx.x / kXcds) % kRowsWaves;
  int count = least + (share < more ? 1 : 0), tile = share * least + min(share, more);
  constexpr int MOST = MT == 4 ? (EPI == ROWS_FORWARD ? 4 : 5) : 3;   // column tiles at a time: registers
  bool met = false;
  auto meet_once = [&]() {
    if (!met) meet();
    met = true;
  };
  if (count == 0) meet();
  while (count > 0) {
    const int parts = (count + MOST - 1) / MOST, n = (count + parts - 1) / parts;
    switch (n) {
#define GEAR_TILES(NT)                                                                                          \
  case NT:                                                                                                      \
    if constexpr (NT <= MOST) rows_tiles_of<T, MT, DIRECT, NT, EPI>(p, lds, in, out, w, N, K, bias, global, row0, tile, lane, meet_once); \
    break;
      GEAR_TILES(1)
      GEAR_TILES(2)
      GEAR_TILES(3)
      GEAR_TILES(4)
      GEAR_TILES(5)
#undef GEAR_TILES
    }
    tile += n;
    count -= n;
  }
}

// columns [N, N up to a whole k-step) of a buffer are zero
template <typename T, int R> __device__ __forceinline__ void zero_pad(unsigned char *lds, const RowsBuf &b, int N, int tid) {
  const int pad = (Step<T>::K - N % Step<T>::K) % Step<T>::K;   // a multiple of 8
  for (int i = tid; i < R * (pad / 4); i += kRowsThreads) {
    const float zero[4] = {0.f, 0.f, 0.f, 0.f};
    lds_put4(lds + b.at + (i / (pad / 4)) * b.stride, N + 4 * (i % (pad / 4)), zero, T{});
  }
}

// an activation tile to its place in the workspace, whole rows at a time (fp32 results are stored from the registers)
template <int R> __device__ __forceinline__ void copy_out(const unsigned char *lds, const RowsBuf &b, int N, bf16_t *global, int row0, int B,
                                                          int wave, int lane) {
  for (int row = wave; row < R && row0 + row < B; row += kRowsWaves)
    for (int c = lane; c < N / 8; c += kWave)
      *reinterpret_cast<uint4 *>(global + (size_t)(row0 + row) * N + 8 * c) = *reinterpret_cast<const uint4 *>(lds + b.at + row * b.stride + 16 * c);
}

// ---- gather: x = [user row | URL row | mean of the cached DFVs] (gather.hip), R / 8 views to a wavefront -----------------
template <typename T, int R>
__device__ __forceinline__ void rows_put4(const RowsArgs &p, unsigned char *lds, int row, int row0, int col, const float (&v)[4]) {
  lds_put4(lds + p.x_buf.at + row * p.x_buf.stride, col, v, T{});
  if (row0 + row < p.B) store4(static_cast<T *>(p.x) + (size_t)(row0 + row) * p.F + col, v);
}
__device__ __forceinline__ int rows_clamp(int id, int64_t n) { return id < 0 ? 0 : (int64_t)id >= n ? (int)(n - 1) : id; }

// sum of a view's cached rows over the columns of this lane's piece, for VIEWS views side by side, four rows of each in flight
template <typename T, typename DT, int R, int VIEWS>
__device__ __forceinline__ void gather_views(const RowsArgs &p, unsigned char *lds, int row0, int first, const int (&lo)[VIEWS],
                                             const int (&n)[VIEWS], int lane) {
  constexpr int DN = Vec16<DT>::N;
  const DT *dfv = static_cast<const DT *>(p.dfv);
  int most = 0;
#pragma unroll
  for (int u = 0; u < VIEWS; ++u) most = max(most, n[u]);
  for (int col0 = 0; col0 < p.D; col0 += kWave * DN) {
    const int col = col0 + lane * DN;
    const bool in = col < p.D;
    float acc[VIEWS][DN];
#pragma unroll
    for (int u = 0; u < VIEWS; ++u)
#pragma unroll
      for (int e = 0; e < DN; ++e) acc[u][e] = 0.0f;
    for (int j0 = 0; j0 < most; j0 += kWave) {
      int ids[VIEWS];   // lane j: the view's image j0 + j
#pragma unroll
      for (int u = 0; u < VIEWS; ++u) ids[u] = j0 + lane < n[u] ? rows_clamp(p.img_id[lo[u] + j0 + lane], p.n_images) : 0;
      for (int j = j0; j < min(most, j0 + kWave); j += 4) {
        Vec16<DT> v[VIEWS][4];
#pragma unroll
        for (int u = 0; u < VIEWS; ++u)
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            v[u][k].v = decltype(v[u][k].v){};
            if (j + k < n[u]) {
              const int id = __builtin_amdgcn_readlane(ids[u], j - j0 + k);
              if (in) v[u][k].v = *reinterpret_cast<const decltype(v[u][k].v) *>(dfv + (size_t)id * p.D + col);
            }
          }
#pragma unroll
        for (int u = 0; u < VIEWS; ++u)
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (j + k < n[u])
#pragma unroll
              for (int e = 0; e < DN; ++e) acc[u][e] += v[u][k].get(e);
      }
    }
    if (in)
#pragma unroll
      for (int u = 0; u < VIEWS; ++u) {
        const float inv = n[u] > 0 ? 1.0f / (float)n[u] : 0.0f;
#pragma unroll
        for (int e = 0; e < DN; e += 4) {
          const float m[4] = {acc[u][e] * inv, acc[u][e + 1] * inv, acc[u][e + 2] * inv, acc[u][e + 3] * inv};
          rows_put4<T, R>(p, lds, first + u, row0, 2 * p.d + col + e, m);
        }
      }
  }
}

template <typename T, typename ET, int R>
__device__ __forceinline__ void gather_embeddings(const RowsArgs &p, unsigned char *lds, int row0, int first, int lane) {
  constexpr int EN = Vec16<ET>::N;
  const int pieces = p.d / EN, all = 2 * pieces;   // of a view: user row, URL row
  for (int i = lane; i < all * (R / kRowsWaves); i += kWave) {
    const int row = first + i / all, c = i % all;
    const bool second = c >= pieces;
    const int col = (second ? c - pieces : c) * EN;
    Vec16<ET> v;
    v.v = decltype(v.v){};
    if (row0 + row < p.B) {
      const int64_t id = second ? rows_clamp(p.url_id[row0 + row], p.n_urls) : rows_clamp(p.user_id[row0 + row], p.n_users);
      v.v = *reinterpret_cast<const decltype(v.v) *>(static_cast<const ET *>(second ? p.url_emb : p.user_emb) + id * p.d + col);
    }
#pragma unroll
    for (int e = 0; e < EN; e += 4) {
      const float m[4] = {v.get(e), v.get(e + 1), v.get(e + 2), v.get(e + 3)};
      rows_put4<T, R>(p, lds, row, row0, (second ? p.d : 0) + col + e, m);
    }
  }
}

template <typename T, int R>
__device__ __forceinline__ void rows_gather(const RowsArgs &p, unsigned char *lds, bool local, int row0, int wave, int lane) {
  constexpr int PER = R / kRowsWaves, VIEWS = R == 64 ? 4 : 2;
  const int first = wave * PER;
  // bounds of the wavefront's lists, clamped like every id: the check of the ids may still be running (gather.hip)
  const int at = min(row0 + first + min(lane, PER), p.B);
  const int off = min(max(p.img_off[at], 0), p.nnz);
  if (p.emb_bf16)
    gather_embeddings<T, bf16_t, R>(p, lds, row0, first, lane);
  else
    gather_embeddings<T, float, R>(p, lds, row0, first, lane);
#pragma unroll
  for (int u0 = 0; u0 < PER; u0 += VIEWS) {
    int lo[VIEWS], n[VIEWS];
#pragma unroll
    for (int u = 0; u < VIEWS; ++u) {
      lo[u] = __builtin_amdgcn_readlane(off, u0 + u);
      n[u] = max(__builtin_amdgcn_readlane(off, u0 + u + 1) - lo[u], 0);
      if (row0 + first + u0 + u >= p.B) n[u] = 0;
    }
#pragma unroll
    for (int u = 0; u < VIEWS; ++u)
      for (int j = lane; local && j < n[u]; j += kWave) {
        p.occ_view[lo[u] + j] = row0 + first + u0 + u;
        p.occ_scale[lo[u] + j] = 1.0f / (float)n[u];
      }
    if (p.dfv_bf16)
      gather_views<T, bf16_t, R, VIEWS>(p, lds, row0, first + u0, lo, n, lane);
    else
      gather_views<T, float, R, VIEWS>(p, lds, row0, first + u0, lo, n, lane);
  }
}

// ---- logit layer and loss (mlp_misc.hip has the formulas), on the last hidden activations in LDS ----------------------------
template <typename T> __device__ __forceinline__ float operand(float w) { return to_f32<T>(from_f32<T>(w)); }

template <typename T, int R>
__device__ __forceinline__ void rows_logit(const RowsArgs &p, unsigned char *lds, const RowsBuf &h, const float *s_w, float y, float b0,
                                           float *s_dz, float (*s_red)[2], int row0, int wave, int lane) {
  constexpr int PER = R / kRowsWaves, VEC = Vec16<T>::N;
  // By quads with few rows only: with 32 the grouping beside the blocks waits longer for the transposes (16 384 views fp32 157.2 us a step,
  // by quads 158; of 16 rows 4096 views 73.4 / 72.9, 5000 61.0 / 60.7).
  constexpr bool QUADS = sizeof(T) == 4 && R == 16;
  const int H = p.H, n_vec = H / VEC;
  float dot[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) dot[u] = 0.0f;
  for (int v = lane; v < (QUADS ? (n_vec + 3) & ~3 : n_vec); v += kWave) {   // whole quads
    float w[VEC];
#pragma unroll
    for (int e = 0; e < VEC; e += 4) {
      const float4 t = *reinterpret_cast<const float4 *>(s_w + min(v, n_vec - 1) * VEC + e);
      w[e] = t.x, w[e + 1] = t.y, w[e + 2] = t.z, w[e + 3] = t.w;
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const unsigned char *row = lds + h.at + (wave * PER + u) * h.stride;
#pragma unroll
      for (int e = 0; e < VEC; e += 4) {
        float x[4];
        if constexpr (QUADS)
          quad_get4(row, v * VEC + e, x);
        else
          lds_get4(row, v * VEC + e, x, T{});
        if (v < n_vec)
#pragma unroll
          for (int k = 0; k < 4; ++k) dot[u] += x[k] * w[e + k];
      }
    }
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) dot[u] = wave_sum(dot[u]);
  // lane u evaluates the wavefront's view u
  float z = dot[0];
#pragma unroll
  for (int u = 1; u < PER; ++u) z = lane == u ? dot[u] : z;
  z += b0;
  const int view = row0 + wave * PER + lane;
  const bool mine = lane < PER && view < p.B;
  const float ex = expf(-fabsf(z));
  const float sig = z >= 0.0f ? 1.0f / (1.0f + ex) : ex / (1.0f + ex);
  const float dz = mine ? (sig - y) * (1.0f / (float)p.B) : 0.0f;
  float loss = mine ? fmaxf(z, 0.0f) - z * y + log1pf(ex) : 0.0f, sum = dz;
  if (mine) {
    p.logits[view] = z;
    p.dz[view] = dz;
  }
  if (lane < PER) s_dz[wave * PER + lane] = dz;
  loss = wave_sum(loss), sum = wave_sum(sum);
  if (lane == 0) s_red[wave][0] = loss, s_red[wave][1] = sum;
}

// A thread owns four neighbouring columns and one of `split` parts of the block's rows; the parts are added in order.
// LOGIT: the delta of the last hidden layer from its activation, sums of delta and of dz h.
// Otherwise the delta is there and is summed.  Both leave the delta in the workspace.  Rows beyond the batch are left out: what
// the network makes of no view at all may be infinite, and zero times that is not zero.
template <typename T, int R, bool LOGIT>
__device__ __forceinline__ void rows_columns(const RowsArgs &p, unsigned char *lds, const RowsBuf &b, int N, T *global, float *part_d,
                                             float *part_w, const float *s_w, const float *s_dz, float *scratch, int row0, int tid) {
  const int owners = N / 4, split = rows_split(R, owners);
  const int part = split > 1 ? tid / owners : 0, rows = R / split, begin = part * rows, end = min(begin + rows, p.B - row0);
  for (int c = tid - part * owners; c < owners && part < split; c += kRowsThreads) {
    const int col = 4 * c;
    float gd[4] = {0.f, 0.f, 0.f, 0.f}, gw[4] = {0.f, 0.f, 0.f, 0.f}, w[4];
    if constexpr (LOGIT) {
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = s_w[col + e];
    }
    for (int row = begin; row < end; row += 4) {   // four rows in flight
      unsigned char *at = lds + b.at + row * b.stride;
      float v[4][4], dz[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (row + k < end) {
          lds_get4(at + k * b.stride, col, v[k], T{});
          if constexpr (LOGIT) dz[k] = s_dz[row + k];
        }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (row + k < end) {
          if constexpr (LOGIT) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              gw[e] += dz[k] * v[k][e];
              v[k][e] = v[k][e] > 0.0f ? dz[k] * w[e] : 0.0f;
            }
            round4(v[k], T{});
            lds_put4(at + k * b.stride, col, v[k], T{});
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) gd[e] += v[k][e];
          store4(global + (size_t)(row0 + row + k) * N + col, v[k]);
        }
    }
    store4(scratch + part * N + col, gd);
    if constexpr (LOGIT) store4(scratch + (split + part) * N + col, gw);
  }
  __syncthreads();
  for (int c = tid; c < N; c += kRowsThreads) {
    float d = 0.0f, w = 0.0f;
    for (int k = 0; k < split; ++k) {
      d += scratch[k * N + c];
      if constexpr (LOGIT) w += scratch[(split + k) * N + c];
    }
    part_d[c] = d;
    if constexpr (LOGIT) part_w[c] = w;
  }
}

// The first local.blocks workgroups group the ids.  Two workgroups of up to 32 views share a CU (kHalf below), so they have half
// the registers; those of 64 have the CU to themselves but for the sorts of a long step, which take 96 registers
// beside 191 (group.hip).  In fp32 with 32 views, a form of long steps only, 96 leave room for them too (hotkey 175.5 us a step, with 108 180).
template <typename T, int MT, bool DIRECT>
__global__ void __launch_bounds__(kRowsThreads, MT == 4 ? 2 : MT == 2 && sizeof(T) == 4 ? 5 : 4) k_rows(RowsArgs p, LocalTask local) {
  constexpr int R = 16 * MT;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  if ((int)blockIdx.x < local.blocks) return local_group<DIRECT>(local, blockIdx.x, lds);
  __shared__ float s_dz[R], s_red[kRowsWaves][2];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int block = blockIdx.x - local.blocks, row0 = block * R;
  float *scratch = reinterpret_cast<float *>(lds + p.scratch), *s_w = reinterpret_cast<float *>(lds + p.logit_w);
  // what the logit layer needs is asked for before anything else
  for (int i = tid; i < p.H; i += kRowsThreads) s_w[i] = operand<T>(p.w_last[i]);
  const int my_view = row0 + wave * (R / kRowsWaves) + lane;
  const float b0 = p.b_last[0], y = lane < R / kRowsWaves && my_view < p.B ? p.label[my_view] : 0.0f;

  rows_gather<T, R>(p, lds, local.blocks > 0, row0, wave, lane);
  zero_pad<T, R>(lds, p.x_buf, p.F, tid);
  // A layer's activations are whole in LDS behind the barrier that begins the next phase.
  auto whole = [&](int l) {
    __syncthreads();
    if constexpr (sizeof(T) == 2)
      if (l >= 0) copy_out<R>(lds, p.layer[l].buf, p.layer[l].out, static_cast<bf16_t *>(p.layer[l].h), row0, p.B, wave, lane);
  };
  for (int l = 0; l + 1 < p.L; ++l) {
    const RowsLayer &a = p.layer[l];
    rows_layer<T, MT, DIRECT, ROWS_FORWARD>(p, lds, l == 0 ? p.x_buf : p.layer[l - 1].buf, a.buf, a.w, a.out, a.in, a.bias, static_cast<T *>(a.h), row0,
                                    wave, lane, [&]() { whole(l - 1); });
    zero_pad<T, R>(lds, a.buf, a.out, tid);
  }
  whole(p.L - 2);
  const RowsLayer &last = p.layer[p.L - 2];
  rows_logit<T, R>(p, lds, last.buf, s_w, y, b0, s_dz, s_red, row0, wave, lane);
  __syncthreads();
  if (tid == 0) {
    float loss = 0.0f, dz = 0.0f;
#pragma unroll
    for (int w = 0; w < kRowsWaves; ++w) loss += s_red[w][0], dz += s_red[w][1];
    p.part_loss[block] = loss;
    p.part_b[block] = dz;
  }
  rows_columns<T, R, true>(p, lds, last.buf, p.H, static_cast<T *>(last.delta), last.colsum + (size_t)block * p.H,
                           p.part_w + (size_t)block * p.H, s_w, s_dz, scratch, row0, tid);
  // The deltas are whole behind the barrier in there, and behind the one in the loop, ahead of which the scratch is read.
  const auto nothing = []() {};
  for (int l = p.L - 2; l > 0; --l) {
    const RowsLayer &a = p.layer[l], &below = p.layer[l - 1];
    rows_layer<T, MT, DIRECT, ROWS_BACK>(p, lds, a.buf, below.buf, a.wt, a.in, a.out, nullptr, static_cast<T *>(below.delta), row0, wave, lane, nothing);
    __syncthreads();
    rows_columns<T, R, false>(p, lds, below.buf, a.in, static_cast<T *>(below.delta), below.colsum + (size_t)block * a.in, nullptr,
                              nullptr, nullptr, scratch, row0, tid);
  }
  rows_layer<T, MT, DIRECT, ROWS_DX>(p, lds, p.layer[0].buf, p.layer[0].buf, p.layer[0].wt, p.F, p.layer[0].out, nullptr, nullptr, row0, wave, lane, nothing);
}

template <typename T, int MT, bool DIRECT = false> hipError_t run_rows(const RowsArgs &a, const LocalTask &local, const RowsPlan &plan, hipStream_t s) {
  hipLaunchKernelGGL((k_rows<T, MT, DIRECT>), dim3((unsigned)(local.blocks + plan.blocks)), dim3(kRowsThreads), plan.lds, s, a, local);
  return hipGetLastError();
}

int row_stride(int dtype, int width) {   // an odd number of 16-byte pieces: the sixteen rows of a read lie in different banks
  const int whole = dtype == GEAR_BF16 ? 32 : 16;
  return (width + whole - 1) / whole * 64 + 16;
}

// Where a block of `rows` views keeps its activations: the first hidden layer's, then x, whose place the other hidden layers'
// take.  Returns the bytes of LDS, without what the kernel declares itself.
long long place_buffers(const Layout &lay, int dtype, int rows, RowsArgs *a) {
  auto place = [&](RowsBuf *b, int width, long long *at) {
    b->stride = row_stride(dtype, width);
    b->at = (int)*at;
    *at += (long long)rows * b->stride;
  };
  long long at = 0;
  place(&a->layer[0].buf, lay.out_dim[0], &at);
  long long end = at;
  place(&a->x_buf, lay.F, &end);
  for (int l = 1; l + 1 < lay.L; ++l) place(&a->layer[l].buf, lay.out_dim[l], &at);
  a->scratch = (int)at;   // used when x is not needed any more
  at += 2 * kRowsThreads * 4 * (long long)sizeof(float);
  if (at > end) end = at;
  a->logit_w = (int)end;
  return end + (long long)lay.in_dim[lay.L - 1] * (long long)sizeof(float);
}

}  // namespace

constexpr int kStateSpan = 3 * kMaxParts;   // words of three per part, then a ticket
// Bytes of weights (once forward, once backward) up to which fp32 blocks read them as they are and a step goes without its prologue, a launch
// of 4 us: read row by row they are 64 bytes of a line at a time forward and words backward, so that every block pays for more of
// them.  us a step, with the prologue / without: 96 -> 64 (49 KB) 512 views 30.3 / 26.1, 2000 34.9 / 28.9, 6000 44.4 / 41.0; 96 -> 128
// (98 KB) 512 views 31.7 / 27.1, 6000 47.0 / 43.5; 96 -> 128 -> 64 (164 KB) 512 32.2 / 31.7, 4000 42.4 / 41.7; 320 -> 64 (164 KB) 1000
// 37.3 / 34.1, 4000 57.2 / 53.6.  Beyond: 288 -> 64 -> 64 (180 KB) 1000 33.7 / 34.1; 1056 -> 24 (203 KB) 1000 51.4 / 52.3; 320 -> 256 -> 128
// 4096 74.8 / 78.1; and with more than a block a CU 288 -> 64 (147 KB) 5000 44.6 / 47.3, 288 -> 256 61.0 / 71.0.  bf16 blocks keep the
// prologue, which rounds the weights once for all: every block would read twice the bytes and round them itself (not tried).
constexpr double kDirectBytes = 170e3, kDirectBytesLong = 100e3;   // up to 4096 views, beyond
// And of all occurrences' gradients: where the accumulation is long, what every one of its wavefronts does to find its units
// (local_parts.hpp) keeps it longer.  With the prologue / without, M = 2, however the ids are spread unless it says so: 320 -> 64, 11 500
// occurrences, 12 MB, 3000 views 50.1 / 46.1, 500 44.2 / 42.5; 528 -> 32, 5500, 11 MB, 2000 views 47.2 / 46.7, Zipf 1.1 55.6 / 50.6; 784 -> 24,
// 3900, 12 MB, 500 views 54.1 / 54.5, Zipf 1.1 48.5 / 47.4; a few steps with wider rows lose 1.  Beyond: 320 -> 64, 18 000, 18 MB, 3000
// views 53.9 / 50.6, 500 50.9 / 52.0; 400 -> 48, 28 MB, 4096 views 71.3 / 73.2; 576 -> 32, 37 MB, 2000 views 69.2 / 72.1.
constexpr double kDirectGradients = 12e6;
constexpr int kLocalPart = 1024;   // ids of a part, where they are spread evenly (2048: a step of 4096 views 1.5 us longer)

// A step whose ids are sorted in launches of their own (api.hip), on two streams.  Lines by measurement (us a step; blocks of
// views against layer by layer; three images a view unless it says otherwise):
// - Rows of a block: fp32 32.  bf16 32 to 8192 views, then 64, one workgroup a CU, where 32 read the weights twice as often
//   (576 -> 512 -> 256, eight images a view, of 32 / 64: 9000 125.4 / 122.8, 12 288 135 / 132.5; 384 -> 384 -> 384: 9000 121.8 / 117.9; 640 ->
//   256 -> 128: 8200 126.6 / 123.7), unless 64 do not fit or gather in two loads (below) and 32 do.
// - One round: a CU holds two blocks of 32 views whose activations leave room, else one, and one of 64 (1024 -> 256 bf16, 80 KB
//   and so 8192 views, eight images: 6000 131 / 137, 10 000 178 / 169; 576 -> 512 -> 256: 14 000 134 / 150, 16 384 139 / 160,
//   18 000 180 / 173; 448 -> 384 -> 384: 16 384 132 / 146, 18 000 167 / 156).  A second round of 64-view blocks pays for one narrow
//   hidden layer (192 -> 128: 20 480 119 / 122, with eight images 125 / 135; 256 -> 128 -> 64 -> 32: 157 / 147; 320 -> 256, 76 KB:
//   130 / 129; 768 -> 72 -> 40 -> 24 185 / 156), up to 20 480 (40 000: 146 / 137).
// - bf16: every block streams all weights twice, so wide layers ask for views, as in a short step (832 -> 768 -> 384, 3.7 MB:
//   2000 views 153 / 135, 4500 148 / 143, 6000 148.5 / 150.5, 8192 156 / 162; 1088 -> 1024, 4.5 MB: 4500 157 / 145; 576 -> 512 ->
//   256, 1.7 MB: 500 146 / 147, 1000 116 / 127).
// - A wavefront gathers four views, two at a time, where the gather's launch has one for each: with many images that chain is
//   the step (192 -> 128: 98 images a view 109 / 136, 200 162 / 155, 600 371 / 220; 576 -> 512 -> 256: 80 135 / 131, 98 146 / 147,
//   200 205 / 175).
//   Cached rows of more than a kilobyte are two loads for a lane, one behind the other; eight wavefronts a CU then gather slower than
//   the gather's launch, and three narrow layers and more do not make up for it (768 -> 72 -> 40 -> 24, eight images: 14 000 views
//   164 / 159, 16 384 172 / 165; but 704 -> 256 -> 128 166 / 171 and 178 / 181, 1088 -> 64 168 / 178, 576 -> 512 -> 256 with an fp32
//   cache 166 / 172 and 176 / 188; 640 -> 512 -> 128, which stays, 181 / 175).
// - fp32: products of the layers are bound by the matrix unit either way, so what is gained is their launches, where a full
//   round takes as long for fewer views: small products from 12 288 views on (96 -> 64: 108 / 119, 16 384 114 / 120; 192 -> 128:
//   124 / 123 and 129 / 131, with eight images 133 / 139 and 143 / 151), larger ones only next to the full round (320 -> 256:
//   12 288 162 / 156, 14 000 165 / 163, with eight images 172 / 172 and 177 / 178, 16 384 185 / 188).
bool plan_long(const Layout &lay, int dt, int B, int nnz, double stream, size_t row_bytes, RowsPlan *plan) {
  const bool bf16 = dt == GEAR_BF16;
  if (nnz > 96ll * B) return false;
  if (bf16 ? stream > 1.5e6 + 420.0 * B : stream > 1e6 || B < (stream > 2e5 ? 14336 : 12288)) return false;
  const bool two_loads = lay.L > 3 && row_bytes > kWave * 16;
  RowsArgs a;
  plan->direct = false;
  plan->rows = bf16 && B > 8192 ? 64 : 32;
  if (plan->rows == 64 && B <= 12288 && (two_loads || place_buffers(lay, dt, 64, &a) + 1024 > 160 * 1024)) plan->rows = 32;
  const long long lds = place_buffers(lay, dt, plan->rows, &a);
  if (lds + 1024 > 160 * 1024) return false;
  const int round = 256 * plan->rows * (plan->rows == 32 && lds + 1024 <= 80 * 1024 ? 2 : 1);
  if (plan->rows == 64 && two_loads) return false;
  if (B > round && !(bf16 && plan->rows == 64 && lay.L == 2 && lds <= 64 * 1024 && B <= 20480)) return false;
  plan->lds = (int)lds;
  plan->room = 0;
  // The sorts beside the blocks find a workgroup's LDS free on every CU, or they would wait for a block to end: digits as wide as
  // fit in what the blocks leave (LDS is given out in pieces of 1280 bytes).
  const long long block = (lds + 1024 + 1279) / 1280 * 1280, free = 160 * 1024 - block * (plan->rows == 32 && 2 * block <= 160 * 1024 ? 2 : 1);
  plan->digit_bits = kCountedDigitBits;
  while (plan->digit_bits > 8 && counted_lds_bytes(plan->digit_bits) > free) --plan->digit_bits;
  plan->blocks = (B + plan->rows - 1) / plan->rows;
  if (2 * (size_t)plan->blocks * (lay.in_dim[lay.L - 1] + 1) * sizeof(float) > lay.tickets - lay.loss_partial) return false;
  size_t sums = 0;   // where the layers leave theirs, or behind the digit totals of the sorts
  for (int l = 1; l < lay.L - 1; ++l) {
    plan->colsum_at[l] = sums;
    sums += (size_t)plan->blocks * lay.in_dim[l];
  }
  plan->colsum = sums * sizeof(float) <= lay.emb_partial - lay.colsum_partial ? lay.colsum_partial : lay.pool_rest;
  return plan->colsum == lay.colsum_partial || lay.pool_rest + sums * sizeof(float) <= lay.loss_partial + lay.pool_bytes;
}

// Which short steps go in blocks, and how.  Lines by measurement (us a step; blocks of 16 or 32 views against layer by layer):
// - Rows of a block: fp32 16 (1000 views, 448 -> 512 -> 256: 99, of 32 152); bf16 16 up to 4096 views (4000: 80 / 85), where
//   16 still find a CU for each, then 32, which read the weights half as often (6000: 96 / 89; 12000: 139 / 114).
// - Every block streams all weights twice, at some 70 GB/s, while the launches of a layer share them: wide layers pay only
//   with enough views (bf16, blocks / layers: 1088 -> 1024 -> 512 120 / 104 at 1000 views, 131 / 126 at 3000, 140 / 148 at
//   4000; 1088 -> 1024 96 / 86 at 1000, 112 / 125 at 4000; 832 -> 768 -> 384 89 / 86 at 500, 97 / 100 at 2000).
// - Few views with very many images keep few CUs at the gather (16 views, 192 -> 128 bf16: 300 images each 106 / 116, 600 181 /
//   175; 576 -> 512 -> 256 bf16, 64 views: 150 each 101 / 109, 300 150 / 149, 16 views of 1200 416 / 353; 320 -> 256 fp32, 16
//   views: 300 102 / 103, 600 180 / 153).
// - LDS of at most half a CU: the launch then has two workgroups on a CU, and the sorts keep nobody waiting (8000 views of
//   20 000 ids in one a CU: 134 against 102).
// - A list of at most kLocalMost ids, in as many parts as an item's 32 bits ask for: a longer one whose ids are most of them
//   one image would not fit in its part's LDS (19 000 ids, 96 -> 64 fp32: 30 % of them one image 57 / 74, 60 % 65 / 73, all 76 /
//   71, without a prologue 4 to 5 less; 320 -> 256 fp32: 70 / 86, 75 / 86, 87 / 84; Zipf 1.5 80 / 103; 25 000 ids of Zipf 1.5 in an earlier form 109 / 88).
bool plan_rows(const gear_config &cfg, const Layout &lay, int B, int nnz, bool local, RowsPlan *plan) {
  const int dt = cfg.mlp_dtype, es = (int)dtype_bytes(dt);
  double stream = 0.0;
  for (int l = 0; l < lay.L - 1; ++l) {
    if (lay.out_dim[l] > 4 * kRowsThreads) return false;   // rows_columns
    stream += 2.0 * es * lay.in_dim[l] * lay.out_dim[l];
  }
  if (lay.F > 4 * kRowsThreads) return false;
  if (!local) return plan_long(lay, dt, B, nnz, stream, cfg.dfv_dim * dtype_bytes(cfg.dfv_dtype), plan);
  if (stream > (lay.L - 1) * (1.5e6 + 500.0 * B)) return false;
  if (nnz > 256ll * B) return false;
  // the lists of ids
  const int64_t range[kMaxProblems] = {cfg.n_users, cfg.n_urls, cfg.n_images};
  int most = 0;
  for (int i = 0; i < kMaxProblems; ++i) {
    const bool last = i == kMaxProblems - 1;
    const int n = last ? nnz : B, bits = bits_for(range[i]);
    if (n > kLocalMost) return false;
    plan->value_bits[i] = bits_for(n);
    int &log2 = plan->parts_log2[i];
    log2 = bits + plan->value_bits[i] - 32;
    if (log2 < 0) log2 = 0;
    while (log2 < bits && n > kLocalPart << log2) ++log2;
    if ((1 << log2) > (last ? kMaxParts : 128)) return false;   // those of the last list are read by a lane each
    if (n > most) most = n;
  }
  const int counts = kLocalWaves * kLocalRadix * 2;
  plan->rows = dt == GEAR_BF16 && B > 4096 ? 32 : 16;
  plan->direct = dt == GEAR_F32 && stream <= (B <= 4096 ? kDirectBytes : kDirectBytesLong) && 4.0 * nnz * cfg.dfv_dim <= kDirectGradients;
  RowsArgs a;
  long long lds = place_buffers(lay, dt, plan->rows, &a);
  // room for two sets of the longest list's ids, as far as that leaves room for a second workgroup on the CU
  constexpr long long kHalf = 80 * 1024 - 1024;
  static_assert((kHalf - kLocalWaves * kLocalRadix * 2) / 8 * 2 >= kLocalMost, "a part of any list fits");
  long long sorts = counts + 8 * (long long)most;
  if (sorts > kHalf) sorts = kHalf;
  if (lds < sorts) lds = sorts;
  if (lds > kHalf) return false;
  plan->lds = (int)lds;
  plan->room = (int)((lds - counts) / 8 * 2);
  plan->blocks = (B + plan->rows - 1) / plan->rows;
  // the sums of the logit layer, then those of the deltas below
  const size_t at = 2 * (size_t)plan->blocks * (lay.in_dim[lay.L - 1] + 1);
  plan->colsum = lay.loss_partial + at * sizeof(float);
  size_t sums = 0;
  for (int l = 1; l < lay.L - 1; ++l) {
    plan->colsum_at[l] = sums;
    sums += (size_t)plan->blocks * lay.in_dim[l];
  }
  return (at + sums) * sizeof(float) <= lay.pool_bytes;
}

LogitSums rows_sums(const RowsPlan &plan, const float *partials, int H) {
  const float *d = partials + (size_t)plan.blocks * H, *b = d + (size_t)plan.blocks * H;
  return LogitSums{partials, d, b, b + plan.blocks, plan.blocks};
}

BlockSums block_sums_of(const RowsPlan &plan, const Layout &lay, const gear_batch &b, char *ws) {
  const LogitSums sums = rows_sums(plan, (const float *)(ws + lay.loss_partial), lay.in_dim[lay.L - 1]);
  BlockSums w;
  memset(&w, 0, sizeof(w));
  w.B = b.B;
  w.rows = plan.rows;
  w.blocks = plan.blocks;
  w.layers = lay.L - 1;
  w.dz = (const float *)(ws + lay.dz), w.logits = (const float *)(ws + lay.logits), w.label = b.label;
  w.h = ws + lay.h[lay.L - 2];
  w.part_w = const_cast<float *>(sums.w), w.part_b = const_cast<float *>(sums.bias), w.part_loss = const_cast<float *>(sums.loss);
  for (int l = lay.L - 2; l >= 0; --l)
    w.layer[lay.L - 2 - l] = BlockSums::Columns{ws + lay.delta[l], l == lay.L - 2 ? const_cast<float *>(sums.delta)
                                                                                 : (float *)(ws + plan.colsum) + plan.colsum_at[l + 1],
                                                lay.out_dim[l]};
  return w;
}

// The parts' counts and the codes lie where the sorts of longer steps publish and count: 768 bytes and more.
LocalResult local_result(const RowsPlan &plan, const GroupBatch &gb, int nnz, int ready_cap) {
  LocalResult r;
  r.parts = (PartCounts *)gb.seg_state;
  r.codes = (uint8_t *)gb.p[0].state;
  r.n_parts = 1 << plan.parts_log2[kMaxProblems - 1];
  r.n_codes = 0;
  for (int i = 0; i < kMaxProblems; ++i) r.n_codes += 1 << plan.parts_log2[i];
  r.ready_cap = ready_cap < nnz ? ready_cap : -1;   // an emission has an occurrence of its own
  return r;
}

LocalTask local_task(const RowsPlan &plan, const GroupBatch &gb, const PlanArgs &args, const ViewCheck &views, int32_t *failed, float *loss) {
  LocalTask t;
  t.blocks = 0;
  t.room = plan.room;
  for (int i = 0; i < kMaxProblems; ++i) {
    const GroupProblem &p = gb.p[i];
    t.list[i] = LocalList{p.keys_in, p.range, p.n, bits_for(p.range), plan.parts_log2[i], plan.value_bits[i], p.sorted_keys,
                          p.perm, (uint32_t *)p.keys[(p.passes + 1) & 1]};
    t.blocks += 1 << plan.parts_log2[i];
  }
  const GroupProblem &img = gb.p[kMaxProblems - 1];
  t.plan = args;
  t.views = views;
  t.unique = img.unique, t.segoff = img.segoff, t.n_unique = img.n_unique;
  t.state = gb.seg_state;
  t.ticket = (int32_t *)gb.seg_state + kStateSpan;
  t.failed = failed;
  t.loss = loss;
  return t;
}

void local_zero_list(const GroupBatch &gb, ZeroList *z) {
  z->count = 1;
  z->p[0] = gb.seg_state;
  z->words[0] = kStateSpan + 1;
}

hipError_t launch_rows(const gear_config &cfg, const Layout &lay, const RowsPlan &plan, const gear_batch &b, const gear_tables &t,
                       const void *dfv_cache, char *ws, const LocalTask &local, hipStream_t s) {
  if (b.B <= 0) return hipSuccess;
  const int L = lay.L;
  RowsArgs a;
  memset(&a, 0, sizeof(a));
  (void)place_buffers(lay, cfg.mlp_dtype, plan.rows, &a);
  a.B = b.B;
  a.nnz = b.nnz;
  a.d = cfg.emb_dim;
  a.D = cfg.dfv_dim;
  a.F = lay.F;
  a.L = L;
  a.H = lay.in_dim[L - 1];
  a.emb_bf16 = cfg.emb_dtype == GEAR_BF16;
  a.dfv_bf16 = cfg.dfv_dtype == GEAR_BF16;
  a.n_users = cfg.n_users, a.n_urls = cfg.n_urls, a.n_images = cfg.n_images;
  a.user_id = b.user_id, a.url_id = b.url_id, a.img_off = b.img_off, a.img_id = b.img_id;
  a.label = b.label;
  a.occ_view = local.plan.plan.row_view, a.occ_scale = local.plan.plan.row_scale;
  a.user_emb = t.user_emb, a.url_emb = t.url_emb, a.dfv = dfv_cache;
  a.w_last = t.mlp_params + lay.w_off[L - 1], a.b_last = t.mlp_params + lay.b_off[L - 1];
  a.x = ws + lay.x;
  a.logits = (float *)(ws + lay.logits), a.dz = (float *)(ws + lay.dz);
  a.dx_emb = (float *)(ws + lay.dx_emb), a.dx_dfv = ws + lay.dx_dfv;
  const LogitSums sums = rows_sums(plan, (const float *)(ws + lay.loss_partial), a.H);
  a.part_w = (float *)(ws + lay.loss_partial);
  a.part_b = const_cast<float *>(sums.bias), a.part_loss = const_cast<float *>(sums.loss);
  for (int l = 0; l + 1 < L; ++l) {
    RowsLayer &r = a.layer[l];
    r.w = ws + lay.wc[l], r.wt = ws + lay.wct[l];
    if (plan.direct) r.w = r.wt = t.mlp_params + lay.w_off[l];
    r.bias = t.mlp_params + lay.b_off[l];
    r.h = ws + lay.h[l], r.delta = ws + lay.delta[l];
    r.in = lay.in_dim[l], r.out = lay.out_dim[l];
    r.colsum = l == L - 2 ? const_cast<float *>(sums.delta) : (float *)(ws + plan.colsum) + plan.colsum_at[l + 1];
  }
  const int rows = plan.rows;
  if (cfg.mlp_dtype == GEAR_BF16) {
    if (rows == 64) return run_rows<bf16_t, 4>(a, local, plan, s);
    if (rows == 32) return run_rows<bf16_t, 2>(a, local, plan, s);
    if (rows == 16) return run_rows<bf16_t, 1>(a, local, plan, s);
  } else {
    if (rows == 32) return run_rows<float, 2>(a, local, plan, s);
    if (rows == 16) return plan.direct ? run_rows<float, 1, true>(a, local, plan, s) : run_rows<float, 1>(a, local, plan, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace gear
