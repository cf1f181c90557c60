// Pieces shared by the matrix-product kernels (gfx950 only): MFMA and LDS access forms, waits, and the
// epilogue that leaves bf16 results through a per-wave LDS patch.
#pragma once

#include "gear_internal.hpp"

namespace gear {
namespace {

typedef __bf16 bf16x8_v __attribute__((ext_vector_type(8)));
typedef float f32x16_v __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void *lds_ptr_t;

constexpr int kXcds = 8;
constexpr int WN = 64, TN = WN / 32;   // columns of a wave tile that leaves through a patch, and its MFMA tiles

union Pack16 {
  uint4 u;
  float4 f;
  bf16x8_v b;
  uint32_t w[4];
  float s[4];
};

// workgroup id -> tile id such that the workgroups of one XCD (ids congruent modulo 8) cover a
// contiguous range of tiles
__device__ __forceinline__ int xcd_remap(int bid, int n_blocks) {
  const int per = n_blocks / kXcds, rem = n_blocks % kXcds;
  const int xcd = bid % kXcds, local = bid / kXcds;
  // the first `rem` XCDs own per + 1 tiles
  const int start = xcd * per + (xcd < rem ? xcd : rem);
  return start + local;
}

template <int N> __device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}
__device__ __forceinline__ void block_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// MFMA operands are fetched with explicit ds_read_b128 so that the only waits on the LDS path are
// the ones written here (the compiler would otherwise make every LDS read wait for all DMA in flight).
#define LDS_READ16(dst, addr, OFF) asm volatile("ds_read_b128 %0, %1 offset:" #OFF : "=v"(dst) : "v"(addr) : "memory")
#define MFMA_BF16(acc_, a_, b_) \
  acc_ = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_v, a_), __builtin_bit_cast(bf16x8_v, b_), acc_, 0, 0, 0)
// The NT kernel takes the product as (B rows) x (A rows)^T: a lane then holds, for ONE row
// m = lane % 32 of the result, the columns n = 8 (e / 4) + 4 (lane / 32) + e % 4 -- four consecutive
// columns per group of four accumulator elements, which is what its epilogue packs and stores.
#define MFMA_BF16_T(acc_, a_, b_) MFMA_BF16(acc_, b_, a_)

// Results of the DMA kernel.  A lane holds row m = lane % 32 of each 32 x 32 tile and, per group of
// four accumulator elements, four consecutive columns.  fp32 results are stored from there as
// 16-byte pieces.  bf16 results are converted in pairs (v_cvt_pk_bf16_f32), written as 8-byte pieces
// into a per-wave LDS patch of 32 rows x 64 columns and read back row-wise so that every lane stores
// 16 contiguous bytes and a row of the patch leaves as one 128-byte line; the ReLU mask of a dgrad
// (EPI_MASK) is read with the same 16-byte pattern before the patch is written.  EPI_DX splits the
// columns: below `split` fp32 into `out` [M x split], the rest bf16 into `aux` [M x (N - split)].
constexpr int PATCH_LD = WN + 8;  // bf16 elements per patch row (144 bytes: the 8-byte writes of a wave spread over all banks)

template <int EPI, int TMW>
__device__ __forceinline__ void epilogue_patch(const f32x16_v (&acc)[TMW][TN], bf16_t *patch, int m0, int n0, int wm,
                                               int wn, int lane, int M, int N, const float *__restrict__ bias,
                                               const bf16_t *__restrict__ aux, void *__restrict__ out, int split,
                                               uint8_t *__restrict__ relu_bits, float (&colacc)[8],
                                               const float *tile_bias, const uint32_t (&hbits)[TMW][4]) {
  const int c = lane & 31, g = lane >> 5;
  const int wave_m0 = m0 + wm * (32 * TMW), wave_n0 = n0 + wn * WN;
  // where this wave's columns go
  bool direct_f32 = EPI == EPI_F32, mixed = false;
  int ld_f32 = N, ld_bf = N, col_shift = 0;
  bf16_t *out_bf = static_cast<bf16_t *>(out);
  if constexpr (EPI == EPI_DX) {
    ld_f32 = split;
    ld_bf = N - split;
    col_shift = split;
    out_bf = const_cast<bf16_t *>(aux);
    direct_f32 = wave_n0 + WN <= split;
    mixed = !direct_f32 && wave_n0 < split;
  }
  if (mixed) {  // the split falls inside this wave's columns: element by element
#pragma unroll
    for (int i = 0; i < TMW; ++i) {
      const int m = wave_m0 + i * 32 + c;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int n = wave_n0 + j * 32 + 8 * (e / 4) + 4 * g + (e % 4);
          if (m < M && n < N) {
            if (n < split)
              static_cast<float *>(out)[(size_t)m * ld_f32 + n] = acc[i][j][e];
            else
              out_bf[(size_t)m * ld_bf + (n - col_shift)] = f32_to_bf16(acc[i][j][e]);
          }
        }
    }
    return;
  }
  if (direct_f32) {
    // column counts are multiples of 8, so a group of four columns is inside the matrix or outside
#pragma unroll
    for (int i = 0; i < TMW; ++i) {
      const int m = wave_m0 + i * 32 + c;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int n = wave_n0 + j * 32 + 8 * q + 4 * g;
          if (m < M && n < N)
            *reinterpret_cast<float4 *>(static_cast<float *>(out) + (size_t)m * ld_f32 + n) =
                make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
        }
    }
    return;
  }
  if constexpr (EPI != EPI_F32) {
    float bn[TN][16];
    if constexpr (EPI == EPI_BIAS_RELU) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          // the tile's biases were staged in LDS before the main loop (zero beyond N)
          bn[j][e] = tile_bias[wn * WN + j * 32 + 8 * (e / 4) + 4 * g + (e % 4)];
        }
    }
    // lane's 16-byte pieces: rows it*8 + lane/8 of each 32-row band, columns (lane%8)*8 .. +7
    const int prow = lane >> 3, cv = (lane & 7) * 8;
    const int n_vec = wave_n0 + cv;
    Pack16 h[EPI == EPI_MASK ? TMW : 1][4];
    if constexpr (EPI == EPI_MASK) {
#pragma unroll
      for (int i = 0; i < TMW; ++i)
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int m = wave_m0 + i * 32 + it * 8 + prow;
          if (m < M && n_vec < N)
            h[i][it].u = *reinterpret_cast<const uint4 *>(aux + (size_t)m * N + n_vec);
          else
            h[i][it].u = make_uint4(0u, 0u, 0u, 0u);
        }
    }
#pragma unroll
    for (int i = 0; i < TMW; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            v[r] = acc[i][j][4 * q + r];
            if constexpr (EPI == EPI_BIAS_RELU) {
              v[r] += bn[j][4 * q + r];
              v[r] = v[r] > 0.0f ? v[r] : 0.0f;
            }
          }
          *reinterpret_cast<uint2 *>(patch + c * PATCH_LD + j * 32 + 8 * q + 4 * g) =
              make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
        }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int row = it * 8 + prow;
        const int m = wave_m0 + i * 32 + row;
        Pack16 v;
        v.u = *reinterpret_cast<const uint4 *>(patch + row * PATCH_LD + cv);
        if (m < M && n_vec < N) {
          if constexpr (EPI == EPI_BIAS_RELU) {
            if (relu_bits) {
              // results are >= 0: a value is positive exactly when its bf16 pattern is not zero
              uint32_t byte = 0u;
#pragma unroll
              for (int w = 0; w < 4; ++w) {
                if (v.w[w] & 0x0000ffffu) byte |= 1u << (2 * w);
                if (v.w[w] & 0xffff0000u) byte |= 2u << (2 * w);
              }
              relu_bits[(size_t)m * (N >> 3) + (n_vec >> 3)] = (uint8_t)byte;
            }
          }
          if constexpr (EPI == EPI_MASK || EPI == EPI_MASK_BITS) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              uint32_t keep = 0u;
              if constexpr (EPI == EPI_MASK) {
                // keep a half-word where the forward activation was positive (bf16 > 0: sign clear, not zero)
                const uint32_t lo = h[i][it].w[w] & 0xffffu, hi = h[i][it].w[w] >> 16;
                if (lo != 0u && lo < 0x8000u) keep |= 0x0000ffffu;
                if (hi != 0u && hi < 0x8000u) keep |= 0xffff0000u;
              } else {
                if (hbits[i][it] & (1u << (2 * w))) keep |= 0x0000ffffu;
                if (hbits[i][it] & (2u << (2 * w))) keep |= 0xffff0000u;
              }
              v.w[w] &= keep;
              // column sums of what is stored (the bias gradient of the layer below)
              colacc[2 * w] += __uint_as_float(v.w[w] << 16);
              colacc[2 * w + 1] += __uint_as_float(v.w[w] & 0xffff0000u);
            }
          }
          // streamed out: nobody on this XCD reads these lines again before they would be evicted,
          // and operand lines that other tiles are about to share stay in its L2 instead
          __builtin_nontemporal_store(u32x4_v{v.u.x, v.u.y, v.u.z, v.u.w},
                                      reinterpret_cast<u32x4_v *>(out_bf + (size_t)m * ld_bf + (n_vec - col_shift)));
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}

}  // namespace
}  // namespace gear
