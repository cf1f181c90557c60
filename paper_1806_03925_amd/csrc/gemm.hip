// Dense contractions of the Sparse-Part MLP on the matrix cores (Section 3, step 4: the Fastgear
// Worker runs the Sparse Part forward to the loss and back-propagates through it).
//
//   forward   a_l      = h_{l-1} W_l^T + b_l           NT, epilogue bias + ReLU
//   dgrad     d_{l-1}  = (d_l W_l) * [a_{l-1} > 0]     NT on the transposed weight copy
//   wgrad     dW_l     = d_l^T h_{l-1}                  TN, split over the batch, fixed-order sum
//
// bf16, K a multiple of 32, about a tile for every CU (nt_dma, gemm_tn_choice): one workgroup = 8 wavefronts (2 x 4) on a 256 x 256
// block tile, a wavefront owns 128 x 64 as 4 x 2 MFMA 32x32x16 tiles.  Operand tiles of k-depth 32
// are copied global -> LDS by DMA (global_load_lds_dwordx4) into four stages.  NT form: two k-tiles
// are copied together while the two before them are multiplied (the halves of a 128-byte line then
// meet in the vector cache), one wait and one s_barrier per pair; LDS rows are [row][32 k] with the
// four 16-byte k-pieces XOR-swizzled by the row so that ds_read_b128 operand fetches do not conflict.  The weights of a step
// come in operand order instead, straight into registers (nt_main_loop_packed).
// TN form (wgrad): one k-tile per barrier, two in flight; LDS keeps the global [k][row] order and
// ds_read_b64_tr_b16 assembles the operand.
// bf16 results leave through a per-wave LDS patch so that every lane stores 16 contiguous bytes.
// Consecutive workgroup ids are spread over the eight XCDs by the hardware; the tile index is
// remapped so that workgroups on one XCD walk neighbouring tiles and share operands in its L2.
//
// Everything else (fp32 operands with v_mfma_f32_32x32x2_f32, products of few rows, K not a multiple of 32)
// goes through the kernels of gemm_tile.hip.
#include "gemm_common.hpp"

namespace gear {
namespace {

constexpr int WM = 128, TM = WM / 32;      // rows of a wave tile and its MFMA tiles

// ---- NT form, bf16, K % 32 == 0: global -> LDS by DMA, four stages, 256 x 256 tile, 8 waves ---------
constexpr int DK = 32;                      // k-depth of a stage
constexpr int DM = 256, DN = 256, DTHREADS = 512;
constexpr int A_ELEMS = DM * DK;
// Two shapes of the workgroup's tile.  Wide: 256 result columns, four stages, one pair of k-tiles in flight
// beside the pair that is being multiplied.  Narrow, for results of at most 128 columns (dLoss/dx of the
// embedding slots): a product of so few columns has little arithmetic per k-tile and waits for its copies,
// so the B tile is 128 rows, a stage is 24 KB, and six stages keep two pairs in flight.
// The eight wavefronts cover the tile as 2 x 4 wave tiles of 128 x 64 (wide) or as 4 x 2 of 64 x 64 (narrow),
// so that all of them have columns in either shape; TMW = 32-row MFMA tiles per wave tile.
struct NtWide {
  static constexpr int BN = 256, STAGES = 4, AHEAD = 1, TMW = 4, WAVES_N = 4;
};
struct NtNarrow {
  static constexpr int BN = 128, STAGES = 6, AHEAD = 2, TMW = 2, WAVES_N = 2;
};
template <typename C, bool PB = false> constexpr int stage_elems() { return A_ELEMS + (PB ? 0 : C::BN * DK); }
// global_load_lds instructions a wave issues per pair of k-tiles: 16 rows of A twice, 16 rows of B per 128, two k-tiles
template <typename C> constexpr int dma_per_pair() { return 2 * (2 + C::BN / 128); }

__device__ __forceinline__ int swz(int row) { return (row >> 2) & 3; }


struct DmaPlan {
  size_t a_off[2], b_off[2];  // element offsets of this lane's 16-byte pieces at k0 = 0
};

// Two consecutive k-tiles at once: a 128-byte line of an operand row holds the row's share of both,
// and its two 64-byte halves are requested by back-to-back instructions of one wave, which meet in
// the vector cache -- one L2 access per line instead of two.
template <typename C>
__device__ __forceinline__ void dma_pair(const bf16_t *__restrict__ A, const bf16_t *__restrict__ B, const DmaPlan &p,
                                         int k0, int k1, bf16_t *s0, bf16_t *s1, int wave) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    __builtin_amdgcn_global_load_lds((const void *)(A + p.a_off[i] + k0), (lds_ptr_t)(s0 + (i * 8 + wave) * 512), 16, 0, 0);
    __builtin_amdgcn_global_load_lds((const void *)(A + p.a_off[i] + k1), (lds_ptr_t)(s1 + (i * 8 + wave) * 512), 16, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < C::BN / 128; ++i) {
    __builtin_amdgcn_global_load_lds((const void *)(B + p.b_off[i] + k0), (lds_ptr_t)(s0 + A_ELEMS + (i * 8 + wave) * 512), 16, 0, 0);
    __builtin_amdgcn_global_load_lds((const void *)(B + p.b_off[i] + k1), (lds_ptr_t)(s1 + A_ELEMS + (i * 8 + wave) * 512), 16, 0, 0);
  }
}

__device__ __forceinline__ void mma_stage(f32x16_v (&acc)[2][TN], uint32_t a_addr0, uint32_t a_addr1, uint32_t b_addr0,
                                          uint32_t b_addr1) {
  u32x4_v p0, p1, q0, q1;   // k-step 0: A rows of the two m-tiles, B rows of the two n-tiles
  u32x4_v r0, r1, s0, s1;   // k-step 1
  LDS_READ16(p0, a_addr0, 0);
  LDS_READ16(p1, a_addr0, 2048);
  LDS_READ16(q0, b_addr0, 0);
  LDS_READ16(q1, b_addr0, 2048);
  LDS_READ16(r0, a_addr1, 0);
  LDS_READ16(r1, a_addr1, 2048);
  LDS_READ16(s0, b_addr1, 0);
  LDS_READ16(s1, b_addr1, 2048);
  asm volatile("s_waitcnt lgkmcnt(4)" : "+v"(p0), "+v"(p1), "+v"(q0), "+v"(q1)::"memory");
  MFMA_BF16_T(acc[0][0], p0, q0);
  MFMA_BF16_T(acc[0][1], p0, q1);
  MFMA_BF16_T(acc[1][0], p1, q0);
  MFMA_BF16_T(acc[1][1], p1, q1);
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(r0), "+v"(r1), "+v"(s0), "+v"(s1)::"memory");
  MFMA_BF16_T(acc[0][0], r0, s0);
  MFMA_BF16_T(acc[0][1], r0, s1);
  MFMA_BF16_T(acc[1][0], r1, s0);
  MFMA_BF16_T(acc[1][1], r1, s1);
}

__device__ __forceinline__ void mma_stage(f32x16_v (&acc)[TM][TN], uint32_t a_addr0, uint32_t a_addr1, uint32_t b_addr0,
                                          uint32_t b_addr1) {
  u32x4_v p0, p1, p2, p3, q0, q1;   // k-step 0: A rows of the four m-tiles, B rows of the two n-tiles
  u32x4_v r0, r1, r2, r3, s0, s1;   // k-step 1
  LDS_READ16(p0, a_addr0, 0);
  LDS_READ16(p1, a_addr0, 2048);
  LDS_READ16(p2, a_addr0, 4096);
  LDS_READ16(p3, a_addr0, 6144);
  LDS_READ16(q0, b_addr0, 0);
  LDS_READ16(q1, b_addr0, 2048);
  LDS_READ16(r0, a_addr1, 0);
  LDS_READ16(r1, a_addr1, 2048);
  LDS_READ16(r2, a_addr1, 4096);
  LDS_READ16(r3, a_addr1, 6144);
  LDS_READ16(s0, b_addr1, 0);
  LDS_READ16(s1, b_addr1, 2048);
  asm volatile("s_waitcnt lgkmcnt(6)" : "+v"(p0), "+v"(p1), "+v"(p2), "+v"(p3), "+v"(q0), "+v"(q1)::"memory");
  MFMA_BF16_T(acc[0][0], p0, q0);
  MFMA_BF16_T(acc[0][1], p0, q1);
  MFMA_BF16_T(acc[1][0], p1, q0);
  MFMA_BF16_T(acc[1][1], p1, q1);
  MFMA_BF16_T(acc[2][0], p2, q0);
  MFMA_BF16_T(acc[2][1], p2, q1);
  MFMA_BF16_T(acc[3][0], p3, q0);
  MFMA_BF16_T(acc[3][1], p3, q1);
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(r0), "+v"(r1), "+v"(r2), "+v"(r3), "+v"(s0), "+v"(s1)::"memory");
  MFMA_BF16_T(acc[0][0], r0, s0);
  MFMA_BF16_T(acc[0][1], r0, s1);
  MFMA_BF16_T(acc[1][0], r1, s0);
  MFMA_BF16_T(acc[1][1], r1, s1);
  MFMA_BF16_T(acc[2][0], r2, s0);
  MFMA_BF16_T(acc[2][1], r2, s1);
  MFMA_BF16_T(acc[3][0], r3, s0);
  MFMA_BF16_T(acc[3][1], r3, s1);
}

// The same with the B operand in registers: b[k-step][n-tile].
__device__ __forceinline__ void mma_stage_packed(f32x16_v (&acc)[TM][TN], uint32_t a_addr0, uint32_t a_addr1, const u32x4_v (&b)[2][TN]) {
  u32x4_v p0, p1, p2, p3, r0, r1, r2, r3;
  LDS_READ16(p0, a_addr0, 0);
  LDS_READ16(p1, a_addr0, 2048);
  LDS_READ16(p2, a_addr0, 4096);
  LDS_READ16(p3, a_addr0, 6144);
  LDS_READ16(r0, a_addr1, 0);
  LDS_READ16(r1, a_addr1, 2048);
  LDS_READ16(r2, a_addr1, 4096);
  LDS_READ16(r3, a_addr1, 6144);
  asm volatile("s_waitcnt lgkmcnt(4)" : "+v"(p0), "+v"(p1), "+v"(p2), "+v"(p3)::"memory");
  MFMA_BF16_T(acc[0][0], p0, b[0][0]);
  MFMA_BF16_T(acc[0][1], p0, b[0][1]);
  MFMA_BF16_T(acc[1][0], p1, b[0][0]);
  MFMA_BF16_T(acc[1][1], p1, b[0][1]);
  MFMA_BF16_T(acc[2][0], p2, b[0][0]);
  MFMA_BF16_T(acc[2][1], p2, b[0][1]);
  MFMA_BF16_T(acc[3][0], p3, b[0][0]);
  MFMA_BF16_T(acc[3][1], p3, b[0][1]);
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(r0), "+v"(r1), "+v"(r2), "+v"(r3)::"memory");
  MFMA_BF16_T(acc[0][0], r0, b[1][0]);
  MFMA_BF16_T(acc[0][1], r0, b[1][1]);
  MFMA_BF16_T(acc[1][0], r1, b[1][0]);
  MFMA_BF16_T(acc[1][1], r1, b[1][1]);
  MFMA_BF16_T(acc[2][0], r2, b[1][0]);
  MFMA_BF16_T(acc[2][1], r2, b[1][1]);
  MFMA_BF16_T(acc[3][0], r3, b[1][0]);
  MFMA_BF16_T(acc[3][1], r3, b[1][1]);
}

constexpr int STAGES = 4;                       // of the TN kernel below

// Tiles t and t + 1 (t even) are copied together into stages t % S and (t + 1) % S while the pairs
// before them are multiplied: one wait and one barrier per pair.  C::AHEAD pairs are in flight beyond the
// one being multiplied; vector memory operations finish in issue order, so waiting until only the later
// pairs' instructions are outstanding means the current pair has landed.  When nk is odd the last pair's
// second half copies the last tile again, into a stage nobody reads.
template <bool MMA, typename C>
__device__ __forceinline__ void nt_main_loop(f32x16_v (&acc)[C::TMW][TN], const bf16_t *__restrict__ A,
                                             const bf16_t *__restrict__ B, const DmaPlan &plan, bf16_t *lds, int nk,
                                             int wave, const uint32_t (&a_rel)[2], const uint32_t (&b_rel)[2]) {
  constexpr int SE = stage_elems<C>();
  static_assert(C::AHEAD == 1 || C::AHEAD == 2, "pairs in flight");
  static_assert(C::STAGES == 2 * (C::AHEAD + 1), "a pair being multiplied and AHEAD pairs being copied");
  auto issue = [&](int t) {
    const int t1 = min(t + 1, nk - 1);
    dma_pair<C>(A, B, plan, t * DK, t1 * DK, lds + (t % C::STAGES) * SE, lds + ((t + 1) % C::STAGES) * SE, wave);
  };
  issue(0);
  if (C::AHEAD == 2 && 2 < nk) issue(2);
  for (int t = 0; t < nk; ++t) {
    if ((t & 1) == 0) {
      // this wave's share of tiles t and t + 1 has landed
      if (C::AHEAD == 2 && t + 2 < nk)
        wait_vm<dma_per_pair<C>()>();
      else
        wait_vm<0>();
      block_barrier();  // ... everybody's has, and everybody is done reading tiles t - 2 and t - 1
      if (t + 2 * C::AHEAD < nk) issue(t + 2 * C::AHEAD);
    }
    const uint32_t so = (uint32_t)(t % C::STAGES) * (2u * SE);
    if constexpr (MMA) mma_stage(acc, a_rel[0] + so, a_rel[1] + so, b_rel[0] + so, b_rel[1] + so);
  }
}

// B (the weights of a step) in operand order (prep.hip: 1 KB for every 32 rows and 16 k, a lane's sixteen bytes together): a
// wavefront's operand is one contiguous load into registers and never passes through LDS; the k-tile after next is requested
// when a k-tile's products are done.  What bounds the form with both operands in LDS is LDS itself: 128 KB pass through it per
// k-tile, 1024 cycles of its 128 bytes, which is what the k-tile's products take; here it is 80 KB.  Four DMA copies of A and
// eight loads of B per pair, always issued in that order (past the end the last tile's again): with eight operations outstanding
// the pair's share of A has landed.  Buffer accesses throughout, which the compiler counts one by one: beside global_load_lds it
// waits for all of them.  us, through LDS / so: 65 536 x 1024 x 1152 bias + ReLU 173 / 150 (1.03 PFLOP/s), x 1024 x 1024 dLoss/dx
// 140 / 127, x 1024 x 256 masked 68 / 64.5, x 256 x 1024 42 / 42.5; a step of that network 963 / 939.  Eight stages of A instead
// of four, two pairs ahead: 156 / 131 / 66.
template <bool MMA>
__device__ __forceinline__ void nt_main_loop_packed(f32x16_v (&acc)[TM][TN], const bf16_t *__restrict__ A, const bf16_t *__restrict__ B,
                                                    const DmaPlan &plan, bf16_t *lds, int nk, int wave, const uint32_t (&a_rel)[2],
                                                    int m0, int b_row, int M, int N, int K, int lane) {
  constexpr int SE = stage_elems<NtWide, true>();
  const auto a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(A) + (size_t)m0 * K, 0, min(DM, M - m0) * K * 2, 0x00020000);
  int a_at[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) a_at[i] = (int)(plan.a_off[i] - (size_t)m0 * K) * 2;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(B), 0, N * K * 2, 0x00020000);   // rows beyond N read as zero
  int b_at[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) b_at[j] = (b_row / 32 + j) * (K / 16) * 1024 + lane * 16;
  u32x4_v b[2][2][TN];
  auto load = [&](u32x4_v (&to)[2][TN], int t) {
    const int at = min(t, nk - 1) * 2048;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        if constexpr (MMA) to[ks][j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, b_at[j], at + ks * 1024, 0);
    asm volatile("" ::: "memory");
  };
  auto copy = [&](int t) {
    const int k0 = min(t, nk - 1) * DK * 2, k1 = min(t + 1, nk - 1) * DK * 2;
    bf16_t *s0 = lds + (t & 3) * SE, *s1 = lds + ((t + 1) & 3) * SE;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_ptr_t)(s0 + (i * 8 + wave) * 512), 16, a_at[i], k0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_ptr_t)(s1 + (i * 8 + wave) * 512), 16, a_at[i], k1, 0, 0);
    }
    asm volatile("" ::: "memory");
  };
  copy(0);
  load(b[0], 0);
  load(b[1], 1);
  for (int t = 0; t < nk; t += 2) {
    if constexpr (MMA)
      wait_vm<8>();
    else
      wait_vm<0>();
    block_barrier();
    copy(t + 2);
    const uint32_t so = (uint32_t)(t & 3) * (2u * SE);
    if constexpr (MMA) mma_stage_packed(acc, a_rel[0] + so, a_rel[1] + so, b[0]);
    load(b[0], t + 2);
    if (t + 1 < nk) {
      if constexpr (MMA) mma_stage_packed(acc, a_rel[0] + so + 2u * SE, a_rel[1] + so + 2u * SE, b[1]);
    }
    load(b[1], t + 3);
  }
}

template <int EPI, typename C = NtWide, bool PB = false>
__global__ void __launch_bounds__(DTHREADS)
k_gemm_nt_dma(const bf16_t *__restrict__ A, const bf16_t *__restrict__ B, int M, int N, int K,
              const float *__restrict__ bias, const bf16_t *__restrict__ aux, void *__restrict__ out, int split,
              float *__restrict__ colpart, uint8_t *__restrict__ relu_bits, const int32_t *__restrict__ status) {
  if (status && *status != 0) return;
  static_assert(!PB || std::is_same_v<C, NtWide>, "the narrow shape reads B through LDS");
  __shared__ __attribute__((aligned(1024))) bf16_t lds[C::STAGES * stage_elems<C, PB>()];   // [stage][A tile | B tile]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int TMW = C::TMW, WMW = 32 * C::TMW;   // this shape's wave tile: WMW rows x WN columns
  const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
  const int n_tiles = (N + C::BN - 1) / C::BN;
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int m0 = (tile / n_tiles) * DM, n0 = (tile % n_tiles) * C::BN;

  DmaPlan plan;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = (i * 8 + wave) * 16 + (lane >> 2);
    const int kv = (lane & 3) ^ swz(row);
    plan.a_off[i] = (size_t)min(m0 + row, M - 1) * K + kv * 8;
    plan.b_off[i] = (size_t)min(n0 + row, N - 1) * K + kv * 8;
  }
  // byte offsets, inside a stage, of this lane's MFMA operands for the two k-steps
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
  uint32_t a_rel[2], b_rel[2];
  {
    const int r = lane & 31, g = lane >> 5;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int off = r * DK + (((2 * kk + g) ^ swz(r)) * 8);
      a_rel[kk] = lds_base + 2u * (uint32_t)(wm * WMW * DK + off);
      b_rel[kk] = lds_base + 2u * (uint32_t)(A_ELEMS + wn * WN * DK + off);
    }
  }

  // What the epilogue needs from global memory is requested here, so that it arrives while the
  // products run: the tile's biases go to LDS (the barriers of the main loop make them visible), the
  // sign bits of the lane's sixteen 16-byte pieces (eight bits each) stay in registers.
  __shared__ float s_bias[EPI == EPI_BIAS_RELU ? C::BN : 1];
  if constexpr (EPI == EPI_BIAS_RELU) {
    if (tid < C::BN) s_bias[tid] = n0 + tid < N ? bias[n0 + tid] : 0.0f;
  }
  uint32_t hbits[TMW][4];
#pragma unroll
  for (int i = 0; i < TMW; ++i)
#pragma unroll
    for (int it = 0; it < 4; ++it) hbits[i][it] = 0u;
  if constexpr (EPI == EPI_MASK_BITS) {
    const uint8_t *bits = reinterpret_cast<const uint8_t *>(aux);
    const int n_vec = n0 + wn * WN + (lane & 7) * 8;
#pragma unroll
    for (int i = 0; i < TMW; ++i)
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int m = m0 + wm * WMW + i * 32 + it * 8 + (lane >> 3);
        if (m < M && n_vec < N) hbits[i][it] = bits[(size_t)m * (N >> 3) + (n_vec >> 3)];
      }
  }

  f32x16_v acc[TMW][TN];
#pragma unroll
  for (int i = 0; i < TMW; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  // in a tile whose right part lies beyond N, the waves without columns copy tiles and meet the
  // barriers but skip the operand reads and the products
  const bool has_columns = n0 + wn * WN < N;
  if constexpr (PB) {
    if (has_columns)
      nt_main_loop_packed<true>(acc, A, B, plan, lds, K / DK, wave, a_rel, m0, n0 + wn * WN, M, N, K, lane);
    else
      nt_main_loop_packed<false>(acc, A, B, plan, lds, K / DK, wave, a_rel, m0, n0 + wn * WN, M, N, K, lane);
  } else if (has_columns)
    nt_main_loop<true, C>(acc, A, B, plan, lds, K / DK, wave, a_rel, b_rel);
  else
    nt_main_loop<false, C>(acc, A, B, plan, lds, K / DK, wave, a_rel, b_rel);
  wait_vm<0>();
  block_barrier();  // every wave is done with the operand tiles: the first stages become the output patches
  static_assert((8 * 32 * PATCH_LD) * 2 + 8 * 64 * 4 <= C::STAGES * stage_elems<C, PB>() * 2, "patches and column sums fit");
  bf16_t *patch = lds + wave * 32 * PATCH_LD;
  float colacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (has_columns)
    epilogue_patch<EPI, TMW>(acc, patch, m0, n0, wm, wn, lane, M, N, bias, aux, out, split, relu_bits, colacc, s_bias, hbits);
  if constexpr (EPI == EPI_MASK || EPI == EPI_MASK_BITS) {
    static_assert(C::WAVES_N == 4, "the column sums below add the two wave rows of the wide shape");
    if (colpart) {
      // colpart[m-tile][n] = sum over the tile's rows of the stored values: lanes that share lane % 8
      // hold the same eight columns, then the two waves that share the columns are added
      float *s_col = reinterpret_cast<float *>(lds + 8 * 32 * PATCH_LD);  // behind the eight output patches
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float v = colacc[e];
        v += __shfl_xor(v, 8, kWave);
        v += __shfl_xor(v, 16, kWave);
        v += __shfl_xor(v, 32, kWave);
        if (lane < 8) s_col[wave * 64 + lane * 8 + e] = v;
      }
      __syncthreads();
      if (wm == 0 && lane < 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int n = n0 + wn * WN + lane * 8 + e;
          if (n < N) colpart[(size_t)(m0 / DM) * N + n] = s_col[wave * 64 + lane * 8 + e] + s_col[(wave + 4) * 64 + lane * 8 + e];
        }
      }
    }
  }
}

// ---- TN form (wgrad), bf16, by DMA and LDS transpose reads ---------------------------------------
// Global tiles are [k][row] with `row` contiguous, which is also how they are kept in LDS: a DMA
// instruction copies two k-rows of 256 values (1 KB).  The MFMA operand (8 k-values of one row per
// lane) is assembled by ds_read_b64_tr_b16: sixteen lanes hand in the addresses of a 4(k) x 16(row)
// block as four-value pieces and each lane gets back one row's four k-values.  Both operands use
// the same pattern, so they agree on which k sits in which slot.
constexpr int TCHUNK = 1024 + 32;                 // bytes: two k-rows of 512 B, then a pad
constexpr int TSTAGE = 2 * 16 * TCHUNK;           // A chunks then B chunks
#define LDS_READ_TR(dst, addr, OFF) \
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "i"(OFF) : "memory")

struct TnPlan {
  size_t a_off[2], b_off[2];
};

__device__ __forceinline__ void dma_tile_tn(const bf16_t *__restrict__ A, const bf16_t *__restrict__ B,
                                            const TnPlan &p, int k0, int M, int N, unsigned char *stage, int wave) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
    __builtin_amdgcn_global_load_lds((const void *)(A + p.a_off[i] + (size_t)k0 * M),
                                     (lds_ptr_t)(stage + (i * 8 + wave) * TCHUNK), 16, 0, 0);
#pragma unroll
  for (int i = 0; i < 2; ++i)
    __builtin_amdgcn_global_load_lds((const void *)(B + p.b_off[i] + (size_t)k0 * N),
                                     (lds_ptr_t)(stage + (16 + i * 8 + wave) * TCHUNK), 16, 0, 0);
}

// operand of MFMA tile at immediate OFF (bytes) for k-step KK: two transpose reads, k-rows +0..3 and +4..7
#define TN_OPERAND(dst, base, OFF, KK)                                   \
  {                                                                      \
    u32x2_v lo_, hi_;                                                    \
    LDS_READ_TR(lo_, base, (KK) * 8 * TCHUNK + (OFF));                   \
    LDS_READ_TR(hi_, base, (KK) * 8 * TCHUNK + 2 * TCHUNK + (OFF));      \
    dst = u32x4_v{lo_.x, lo_.y, hi_.x, hi_.y};                           \
  }

__device__ __forceinline__ void mma_stage_tn(f32x16_v (&acc)[TM][TN], uint32_t a_even, uint32_t a_odd, uint32_t b_even,
                                             uint32_t b_odd) {
#define TN_KSTEP(KK)                                       \
  {                                                        \
    u32x4_v p0, p1, p2, p3, q0, q1;                        \
    TN_OPERAND(p0, a_even, 0, KK)                          \
    TN_OPERAND(p1, a_odd, 64, KK)                          \
    TN_OPERAND(p2, a_even, 128, KK)                        \
    TN_OPERAND(p3, a_odd, 192, KK)                         \
    TN_OPERAND(q0, b_even, 0, KK)                          \
    TN_OPERAND(q1, b_odd, 64, KK)                          \
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(p0), "+v"(p1), "+v"(p2), "+v"(p3), "+v"(q0), "+v"(q1)::"memory"); \
    MFMA_BF16(acc[0][0], p0, q0);                          \
    MFMA_BF16(acc[0][1], p0, q1);                          \
    MFMA_BF16(acc[1][0], p1, q0);                          \
    MFMA_BF16(acc[1][1], p1, q1);                          \
    MFMA_BF16(acc[2][0], p2, q0);                          \
    MFMA_BF16(acc[2][1], p2, q1);                          \
    MFMA_BF16(acc[3][0], p3, q0);                          \
    MFMA_BF16(acc[3][1], p3, q1);                          \
  }
  TN_KSTEP(0)
  TN_KSTEP(1)
#undef TN_KSTEP
}

template <bool MMA>
__device__ __forceinline__ void tn_main_loop(f32x16_v (&acc)[TM][TN], const bf16_t *__restrict__ A,
                                             const bf16_t *__restrict__ B, const TnPlan &plan, int k_begin, int nk, int M,
                                             int N, unsigned char *lds, int wave, uint32_t a_even, uint32_t a_odd,
                                             uint32_t b_even, uint32_t b_odd) {
#pragma unroll
  for (int p = 0; p < STAGES - 1; ++p)
    if (p < nk) dma_tile_tn(A, B, plan, k_begin + p * DK, M, N, lds + p * TSTAGE, wave);

  int stage = 0;
  for (int t = 0; t < nk; ++t) {
    if (t + 2 < nk)
      wait_vm<8>();
    else if (t + 1 < nk)
      wait_vm<4>();
    else
      wait_vm<0>();
    block_barrier();
    if (t + 3 < nk) dma_tile_tn(A, B, plan, k_begin + (t + 3) * DK, M, N, lds + ((stage + 3) & 3) * TSTAGE, wave);
    const uint32_t so = (uint32_t)stage * TSTAGE;
    if constexpr (MMA) mma_stage_tn(acc, a_even + so, a_odd + so, b_even + so, b_odd + so);
    stage = (stage + 1) & 3;
  }
}

// One workgroup's share: tile `tile` of the [M x N] result over the k-range `split`, left in
// partial[split][M x N].
__device__ __forceinline__ void tn_dma_work(const bf16_t *__restrict__ A, const bf16_t *__restrict__ B, int M, int N,
                                            int K, int k_chunk, float *__restrict__ partial, int split, int tile,
                                            unsigned char *lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  const int n_tiles = (N + DN - 1) / DN;
  const int m0 = (tile / n_tiles) * DM, n0 = (tile % n_tiles) * DN;
  const int k_begin = split * k_chunk;
  const int k_end = min(K, k_begin + k_chunk);

  // DMA: chunk c = k-rows 2c, 2c+1; lane p holds LDS slot p%32 of k-row p/32, which receives the
  // 8-value piece (p%32) ^ (4 * (p/32)) so that odd k-rows sit 64 bytes away from even ones
  TnPlan plan;
  {
    const int krow = lane >> 5, piece = (lane & 31) ^ (4 * krow);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = 2 * (i * 8 + wave) + krow;
      const int ma = min(m0 + piece * 8, M - 8), nb = min(n0 + piece * 8, N - 8);  // stay inside the row
      plan.a_off[i] = (size_t)k * M + ma;
      plan.b_off[i] = (size_t)k * N + nb;
    }
  }
  // transpose reads: lane l -> j = l%16, half = (l/16)%2 (rows +16), g = l/32 (k-rows +8);
  // it addresses k-row 8 g + j/4 (+4 for the second read), rows 16 half + 4 (j%4) .. +3
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
  uint32_t a_even, a_odd, b_even, b_odd;
  {
    const int j = lane & 15, half = (lane >> 4) & 1, g = lane >> 5;
    const int k = 8 * g + (j >> 2);
    const int odd = k & 1;
    const uint32_t row_off = (uint32_t)(k >> 1) * TCHUNK + (uint32_t)odd * 512u;
    const uint32_t ca = 2u * (uint32_t)(wm * WM + 16 * half + 4 * (j & 3));
    const uint32_t cb = 2u * (uint32_t)(wn * WN + 16 * half + 4 * (j & 3));
    // odd k-rows are stored with the 64-byte halves of every 128 bytes swapped
    a_even = lds_base + row_off + ca + (odd ? 64u : 0u);
    a_odd = lds_base + row_off + ca - (odd ? 64u : 0u);
    b_even = lds_base + 16u * TCHUNK + row_off + cb + (odd ? 64u : 0u);
    b_odd = lds_base + 16u * TCHUNK + row_off + cb - (odd ? 64u : 0u);
  }

  f32x16_v acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  const int nk = (k_end - k_begin + DK - 1) / DK;   // k_end - k_begin is a multiple of DK (checked by the host)
  // in a tile whose right part lies beyond N, the waves without columns copy tiles and meet the
  // barriers but skip the operand reads and the products
  if (n0 + wn * WN < N)
    tn_main_loop<true>(acc, A, B, plan, k_begin, nk, M, N, lds, wave, a_even, a_odd, b_even, b_odd);
  else
    tn_main_loop<false>(acc, A, B, plan, k_begin, nk, M, N, lds, wave, a_even, a_odd, b_even, b_odd);
  // fp32 partial of this k range
  float *dst = partial + (size_t)split * M * N;
  const int c = lane & 31, g = lane >> 5;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn * WN + j * 32 + c;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = m0 + wm * WM + i * 32 + 8 * (e / 4) + 4 * g + (e % 4);
        if (m < M && n < N) dst[(size_t)m * N + n] = acc[i][j][e];
      }
    }
}

// Several contractions over the same K rows in one launch: the grid is k-ranges x (all tiles of all
// problems), so every workgroup does the same amount of work whichever result it belongs to.
struct TnBatchArgs {
  int count, tiles;
  TnProblem p[GEAR_MAX_LAYERS];
  int first_tile[GEAR_MAX_LAYERS];
};

__global__ void __launch_bounds__(DTHREADS)
k_gemm_tn_dma_batch(TnBatchArgs args, int K, int k_chunk, const int32_t *__restrict__ status) {
  if (status && *status != 0) return;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[STAGES * TSTAGE];
  const int work = xcd_remap(blockIdx.x, gridDim.x);
  const int split = work / args.tiles, tile = work % args.tiles;
  int which = 0;
  for (int i = 1; i < args.count; ++i)
    if (tile >= args.first_tile[i]) which = i;
  const TnProblem &q = args.p[which];
  tn_dma_work((const bf16_t *)q.A, (const bf16_t *)q.B, q.M, q.N, K, k_chunk, q.partial, split,
              tile - args.first_tile[which], lds);
}

// Which of the two bf16 NT kernels a product takes.  The 256 x 256 tiles of the kernel above move the fewest bytes
// per product, but a CU holds one: below one tile per CU the smaller tiles of gemm_tile.hip mostly win.
bool nt_fills(int dtype, int M, int N, int K, bool narrow) {
  if (dtype != GEAR_BF16 || K % DK != 0) return false;
  return (long long)((M + DM - 1) / DM) * (narrow ? 1 : (N + DN - 1) / DN) >= 256;
}
// Not so a long product that leaves few CUs out: from about 216 whole tiles on with K >= 512, from 174 on with K >= 1024,
// a CU's one large tile ends before the two rounds of small ones it would have instead.  (bias + ReLU, us, 256 x 256 /
// smaller: 20000 x 768 x 1152 37.0 / 47.6, 28672 x 512 x 512 20.2 / 22.4, 24000 x 512 x 1024 31.1 / 33.7, 20000 x 576 x
// 1024 30.1 / 33.9; on the other side 24000 x 512 x 512 masked 23.3 / 20.7, 20000 x 512 x 1152 33.6 / 31.5, 16384 x 576 x
// 1152 32.1 / 30.6.  The narrow form has N <= 128 and never as many.)
bool nt_dma(int dtype, int M, int N, int K, bool narrow) {
  if (nt_fills(dtype, M, N, K, narrow)) return true;
  const long long whole = (long long)M * N / (DM * DN);
  return dtype == GEAR_BF16 && K % DK == 0 && !narrow && ((whole >= 215 && K >= 512) || (whole >= 174 && K >= 1024));
}

int tn_dma_tiles(const TnProblem &p) { return ((p.M + DM - 1) / DM) * ((p.N + DN - 1) / DN); }

// Ranges of the 256 x 256 kernel: one round of the 256 CUs, every range at least 512 rows.
int tn_dma_splits(int tiles, int K) {
  int s = 256 / tiles;
  if (s > K / 512) s = K / 512;
  if (s > 64) s = 64;
  return s < 1 ? 1 : s;
}

}  // namespace

// Number of row-tile partials a masked product leaves in `colpart` ([parts x N] column sums of its result).
int gemm_nt_colsum_parts(int dtype, int M, int N, int K, bool coarse) {
  return nt_dma(dtype, M, N, K, false) ? (M + DM - 1) / DM : nt_tile_colsum_parts(dtype, M, N, coarse);
}

bool gemm_nt_takes_tiles(int dtype, int M, int N, int K, int epi) {
  const bool narrow = N <= NtNarrow::BN && (epi == EPI_DX || epi == EPI_F32);
  return !narrow && N % 32 == 0 && (long long)N * K < (1ll << 30) && K < (1 << 21) && nt_dma(dtype, M, N, K, false);
}

bool gemm_nt_carries(int dtype, int M, int N, int K) { return !nt_fills(dtype, M, N, K, false); }

hipError_t launch_gemm_nt(int dtype, const void *A, const void *B, int M, int N, int K, int epi, const float *bias,
                          const void *aux, void *out, int split, float *colpart, uint8_t *relu_bits,
                          const int32_t *status, hipStream_t s, bool coarse, const SideTask *side, bool tiles, hipEvent_t stop) {
  if (M <= 0 || N <= 0) return leave(stop, s);
  if (tiles && (side || !gemm_nt_takes_tiles(dtype, M, N, K, epi))) return hipErrorInvalidValue;
  if (epi == EPI_MASK_BITS && dtype != GEAR_BF16) return hipErrorInvalidValue;
  const bool narrow = N <= NtNarrow::BN && (epi == EPI_DX || epi == EPI_F32);
  if (side ? !nt_fills(dtype, M, N, K, narrow) : !nt_dma(dtype, M, N, K, narrow))
    return launch_gemm_nt_tile(dtype, A, B, M, N, K, epi, bias, aux, out, split, colpart, relu_bits, status, s, coarse, side, stop);
  if (side) return hipErrorInvalidValue;
  const dim3 grid(((M + DM - 1) / DM) * (narrow ? 1 : (N + DN - 1) / DN));
#define GEAR_DMA(E, ...)                                                                                              \
  launch_leaving(stop, k_gemm_nt_dma<E, __VA_ARGS__>, grid, DTHREADS, 0, s, (const bf16_t *)A, (const bf16_t *)B, M, N, K, bias, \
                 (const bf16_t *)aux, out, split, colpart, relu_bits, status)
  if (tiles) {
    if (epi == EPI_BIAS_RELU)
      GEAR_DMA(EPI_BIAS_RELU, NtWide, true);
    else if (epi == EPI_MASK_BITS)
      GEAR_DMA(EPI_MASK_BITS, NtWide, true);
    else if (epi == EPI_DX)
      GEAR_DMA(EPI_DX, NtWide, true);
    else
      return hipErrorInvalidValue;
  } else if (epi == EPI_BIAS_RELU)
    GEAR_DMA(EPI_BIAS_RELU, NtWide);
  else if (epi == EPI_MASK)
    GEAR_DMA(EPI_MASK, NtWide);
  else if (epi == EPI_MASK_BITS)
    GEAR_DMA(EPI_MASK_BITS, NtWide);
  else if (epi == EPI_DX && narrow)
    GEAR_DMA(EPI_DX, NtNarrow);
  else if (epi == EPI_DX)
    GEAR_DMA(EPI_DX, NtWide);
  else if (narrow)
    GEAR_DMA(EPI_F32, NtNarrow);
  else
    GEAR_DMA(EPI_F32, NtWide);
#undef GEAR_DMA
  return hipGetLastError();
}

// Which weight-gradient kernel the layers take, and how many of them (from the first on) go in one launch.  What either
// kernel needs follows from the rows of the batch that a CU walks one range after another: 28 ns each on 256 x 256 tiles, a
// workgroup to a CU, 18.5 ns on 128 x 128 (gemm_tile.hip), two to a CU; and ahead of them what starting and ending costs,
// more on the large tiles, which leave more partials.  That shrinks with the length of the batch because the large tiles
// also move half the bytes, beside an accumulation that is bound by them.  Layers go to the large tiles in groups of up to
// 128, so that the ranges fill the CUs.
// Products and sums alone, us, 256 x 256 / 128 x 128: layers 1024-256 (F = 1152) over 12288 rows 62 / 57, 32736 120 / 133;
// 2048-1024 over 4096 66 / 79, 16384 165 / 249, 32736 320 / 479; 512-256 (F = 576) over 32736 54 / 50.  Whole steps, eight
// images a view: 1024-256 over 12288 views 254 / 254, 24576 424 / 449; 1024 over 16384 253 / 253, 24576 357 / 373, 32736
// 416 / 442; 512-512-512 over 20000 289 / 283, 32736 355 / 353; 512-256 over 32736 265 / 263.  From 32768 rows on up to 128
// tiles are the larger kernel's (512-256 over 65536 views 441 / 445, 1024-256 857 / 953, 320-72 531 / 546; a layer of 256
// columns 227 / 222).  (All with single workgroups on 128 x 128; pairs of them, gemm_tile.hip, save 2 to 6 of a step.)
TnChoice gemm_tn_choice(int dtype, const TnProblem *p, int count, int K) {
  if (dtype == GEAR_BF16 && K % DK == 0) {
    long long cost = min(2200, 20000000 / K);   // in half rows of the smaller kernel, 9 ns; a launch more is 1100
    int first = 0, all = 0;
    for (int i = 0; i < count;) {
      int tiles = tn_dma_tiles(p[i]), n = 1;
      for (; i + n < count && tiles + tn_dma_tiles(p[i + n]) <= 128; ++n) tiles += tn_dma_tiles(p[i + n]);
      const int splits = tn_dma_splits(tiles, K);
      cost += 3 * (((long long)tiles * splits + 255) / 256 * ((K + splits - 1) / splits)) + (i > 0 ? 1100 : 0);
      if (i == 0) first = n;
      all += tiles;
      i += n;
    }
    if ((K >= 32768 && all <= 128) || cost <= 2 * tn_tile_rows(dtype, p, count, K)) return TnChoice{first, true};
  }
  return TnChoice{count, false};
}

int gemm_tn_splits(int dtype, const TnProblem *p, int count, int K, bool large, bool *pairs) {
  if (!large) return tn_tile_splits(dtype, p, count, K, pairs);
  *pairs = false;
  int tiles = 0;
  for (int i = 0; i < count; ++i) tiles += tn_dma_tiles(p[i]);
  return tn_dma_splits(tiles, K);
}

hipError_t launch_gemm_tn(int dtype, const TnProblem *p, int count, int K, int splits, bool large, bool pairs, const int32_t *status,
                          hipStream_t s, const int32_t *k_dev) {
  if (count < 1 || count > GEAR_MAX_LAYERS || splits < 1) return hipErrorInvalidValue;
  for (int i = 0; i < count; ++i)
    if (p[i].M < 4 || p[i].N < 4 || !p[i].A || !p[i].B || !p[i].partial) return hipErrorInvalidValue;
  if (!large) return launch_gemm_tn_tile(dtype, p, count, K, splits, pairs, status, s, k_dev);
  if (k_dev || dtype != GEAR_BF16 || K % DK != 0) return hipErrorInvalidValue;
  TnBatchArgs args;
  args.count = count;
  args.tiles = 0;
  for (int i = 0; i < GEAR_MAX_LAYERS; ++i) {
    args.p[i] = i < count ? p[i] : TnProblem{nullptr, nullptr, nullptr, 0, 0};
    args.first_tile[i] = args.tiles;
    if (i < count) args.tiles += tn_dma_tiles(p[i]);
  }
  const int kc = ((((K + splits - 1) / splits) + DK - 1) / DK) * DK;
  hipLaunchKernelGGL(k_gemm_tn_dma_batch, dim3(args.tiles * splits), dim3(DTHREADS), 0, s, args, K, kc, status);
  return hipGetLastError();
}

}  // namespace gear
