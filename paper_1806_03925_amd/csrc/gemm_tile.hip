// Matrix products on tiles of moderate size, both operand types, any inner length (Section 3, step 4: the
// Sparse Part forward and backward).  The large bf16 products have kernels of their own (gemm.hip); what runs
// here is bound by latency and by how many CUs have a tile at all, not by any peak: a layer of 256 columns over
// 4096 rows is sixteen tiles of 256 x 256, but 256 tiles of 64 x 64.
//
// Operand tiles are copied global -> LDS by DMA into a ring of stages, several stages ahead, so that one memory
// latency is paid per product and not one per k-tile.  (A register-staged form with one k-tile ahead took 15 us
// for 4096 x 256 x 320 in fp32, this one 10; the weight gradients of 4096 x (320 -> 256 -> 128) took 63 us in four
// launches, now 19 in two.)  What lies beyond an operand's inner length is copied from a line of
// zeros, so no inner length needs padding, and rows beyond the matrix repeat its last row and are not stored.
#include "group_device.hpp"
#include "tn_tile.hpp"

#include <type_traits>

namespace gear {
namespace {

// ---- NT: C = A B^T, a stage is 128 bytes of k per operand row (64 bf16 or 32 fp32) --------------------------
template <typename T_, int WTM_, int WTN_, int WAVES_M_, int WAVES_N_, int STAGES_> struct NtTile {
  using T = T_;
  static constexpr int WTM = WTM_, WTN = WTN_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, STAGES = STAGES_;
  static constexpr int WAVES = WAVES_M * WAVES_N, THREADS = WAVES * kWave;
  static constexpr int BM = 32 * WTM * WAVES_M, BN = 32 * WTN * WAVES_N;
  static constexpr int VEC = 16 / (int)sizeof(T), KS = 8 * VEC;
  static constexpr int STAGE_BYTES = (BM + BN) * 128;
  static constexpr int DMA_A = BM / 8 / WAVES, DMA_B = BN / 8 / WAVES;   // instructions of a wave per stage
  static constexpr int PER_STAGE = DMA_A + DMA_B;
  static_assert(DMA_A * 8 * WAVES == BM && DMA_B * 8 * WAVES == BN, "a DMA instruction copies eight rows");
  static_assert((STAGES - 1) * PER_STAGE < 64, "outstanding copies are counted in six bits");
};

// Operands of one k-step (a quarter of a stage) in registers.  LDS rows are 128 bytes with their eight 16-byte pieces
// XOR-ed by the row's number modulo 8, so that the 32 rows a read touches spread over all banks; a k-step is two
// neighbouring pieces of a row, one for either half-wave.  One bf16 product takes all sixteen values as they are; an
// fp32 product takes two neighbouring k-values, one from either half-wave, so the halves trade values first.
template <typename C> struct Frag {
  u32x4_v a[C::WTM], b[C::WTN];
  __device__ __forceinline__ void fetch(uint32_t a_addr, uint32_t b_addr) {
    static_assert(C::WTM <= 2 && C::WTN <= 2, "tiles of a wave");
    lds_read16<0>(a[0], a_addr);
    if constexpr (C::WTM > 1) lds_read16<4096>(a[1], a_addr);
    lds_read16<0>(b[0], b_addr);
    if constexpr (C::WTN > 1) lds_read16<4096>(b[1], b_addr);
  }
  template <int LATER> __device__ __forceinline__ void wait() {   // at most LATER reads issued after these are outstanding
    wait_lgkm<LATER>();
#pragma unroll
    for (int i = 0; i < C::WTM; ++i) landed(a[i]);
#pragma unroll
    for (int j = 0; j < C::WTN; ++j) landed(b[j]);
  }
  // fp32: the half-waves hold k 0..3 and 4..7 of the step; afterwards registers 0, 2, 1, 3 hold (0, 1), (2, 3), (4, 5),
  // (6, 7).  Two v_permlane32_swap per operand and step; products then add k in ascending pairs, in every tile shape,
  // so that a hidden unit next to zero takes the same branch whichever shape its layer's product has.
  static __device__ __forceinline__ void trade(u32x4_v &v) {
    const auto lo = __builtin_amdgcn_permlane32_swap(v[0], v[1], false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(v[2], v[3], false, false);
    v[0] = lo[0], v[1] = lo[1], v[2] = hi[0], v[3] = hi[1];
  }
  // bf16 is taken transposed (a lane holds four consecutive columns of a row, see epilogue_patch); fp32 is not (a lane
  // holds one column, half a wave stores 128 contiguous bytes).
  // The scheduler may not move products across: it would otherwise put the next wait between them.
  __device__ __forceinline__ void mma(f32x16_v (&acc)[C::WTM][C::WTN]) {
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (sizeof(typename C::T) == 2) {
#pragma unroll
      for (int i = 0; i < C::WTM; ++i)
#pragma unroll
        for (int j = 0; j < C::WTN; ++j) MFMA_BF16_T(acc[i][j], a[i], b[j]);
    } else {
#pragma unroll
      for (int i = 0; i < C::WTM; ++i) trade(a[i]);
#pragma unroll
      for (int j = 0; j < C::WTN; ++j) trade(b[j]);
      constexpr int kAscending[4] = {0, 2, 1, 3};
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < C::WTM; ++i)
#pragma unroll
          for (int j = 0; j < C::WTN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[i][kAscending[e]]),
                                                             __uint_as_float(b[j][kAscending[e]]), acc[i][j], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
};

// The main loop, one form per number of stages.
//
// Two stages (bf16): the next stage is copied while this one is multiplied; 64 KB, so two workgroups share a CU and
// one multiplies while the other waits.
//
// More (fp32): an fp32 product keeps the SIMD's vector unit busy as well (measured: every vector instruction between
// two of them adds its own four cycles, 153 TFLOP/s bare, 110 with four in between), so the loop has as few as it
// can.  The wait for the next stage and the barrier sit in the middle of a stage, and a k-step's operands are
// requested one step (256 cycles of products) ahead, also across the border of a stage.
template <typename C, typename Issue>
__device__ __forceinline__ void nt_main_loop(f32x16_v (&acc)[C::WTM][C::WTN], uint32_t a_rel, uint32_t b_rel, int nk, Issue issue) {
  constexpr int S = C::STAGES;
  constexpr uint32_t STEP = 32u;   // from a k-step's piece to the next one's
  Frag<C> f[2];
  if constexpr (S == 2) {
    constexpr int READS = C::WTM + C::WTN;
    uint32_t so = 0;
    for (int t = 0; t < nk; ++t) {
      wait_vm<0>();      // this wave's share of stage t has landed
      block_barrier();   // everybody's has, and everybody is done reading stage t - 1
      if (t + 1 < nk) issue(t + 1, (t + 1) & 1);
      const uint32_t a = a_rel + so, b = b_rel + so;
      f[0].fetch(a, b);
      f[1].fetch(a ^ STEP, b ^ STEP);
      f[0].template wait<READS>();
      f[0].mma(acc);
      f[0].fetch(a ^ (2 * STEP), b ^ (2 * STEP));
      f[1].template wait<READS>();
      f[1].mma(acc);
      f[1].fetch(a ^ (3 * STEP), b ^ (3 * STEP));
      f[0].template wait<READS>();
      f[0].mma(acc);
      f[1].template wait<0>();
      f[1].mma(acc);
      so = C::STAGE_BYTES - so;
    }
  } else {
    wait_stages<C::PER_STAGE, S - 2>(nk - 1);
    block_barrier();
    f[0].fetch(a_rel, b_rel);
    f[0].template wait<0>();
    int stage = 0, fill = S - 1;
    for (int t = 0; t < nk; ++t) {
      const int next = stage + 1 == S ? 0 : stage + 1;
      const uint32_t so = (uint32_t)stage * C::STAGE_BYTES, a = a_rel + so, b = b_rel + so;
      f[1].fetch(a ^ STEP, b ^ STEP);
      f[0].mma(acc);
      f[1].template wait<0>();
      f[0].fetch(a ^ (2 * STEP), b ^ (2 * STEP));
      f[1].mma(acc);
      f[0].template wait<0>();
      if (t + 1 < nk) {
        wait_stages<C::PER_STAGE, S - 3>(nk - 2 - t);   // this wave's share of stage t + 1 has landed
        block_barrier();                                // everybody's has, and everybody is done reading stage t - 1
        if (t + S - 1 < nk) issue(t + S - 1, fill);
      }
      f[1].fetch(a ^ (3 * STEP), b ^ (3 * STEP));
      f[0].mma(acc);
      f[1].template wait<0>();
      // the first step of the next stage; behind the last stage it reads what is left in the ring and is not used
      f[0].fetch(a_rel + (uint32_t)next * C::STAGE_BYTES, b_rel + (uint32_t)next * C::STAGE_BYTES);
      f[1].mma(acc);
      f[0].template wait<0>();
      stage = next;
      fill = fill + 1 == S ? 0 : fill + 1;
    }
  }
}

// fp32 results, stored from the accumulator layout: element e of a 32 x 32 tile sits at row
// 8 (e / 4) + 4 (lane / 32) + e % 4, column lane % 32.  colsum[j] gathers what is stored of column j's tile.
// EPI_F32, whose results (the stand-in's rows for a cache, say) are many times its operands, is bound by these stores:
// 65536 x 1024 x 64 took 133 us on one three-stage tile per CU, 107 on two tiles of two stages, 100 with stores past the L2.
template <int EPI, typename C, int NB, int NM>
__device__ __forceinline__ void store_f32(const f32x16_v (&acc)[C::WTM][C::WTN], int m_first, int n_first, int lane, int M,
                                          int N, const float (&bias)[NB], const float (&mask)[NM][16],
                                          const float *__restrict__ aux, float *__restrict__ out, int split,
                                          float (&colsum)[C::WTN]) {
  const int c = lane & 31, g = lane >> 5;
  const bool whole = m_first + 32 * C::WTM <= M;   // all rows exist: no test per row
#pragma unroll
  for (int j = 0; j < C::WTN; ++j) {
    const int n = n_first + j * 32 + c;
    colsum[j] = 0.0f;
    if (n >= N) continue;
    // where this column goes: below `split` into out [M x split], the rest into aux [M x (N - split)]
    float *dst = out + n;
    int ld = N;
    if constexpr (EPI == EPI_DX) {
      dst = n < split ? out + n : const_cast<float *>(aux) + (n - split);
      ld = n < split ? split : N - split;
    }
#pragma unroll
    for (int i = 0; i < C::WTM; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = m_first + i * 32 + 8 * (e / 4) + 4 * g + (e % 4);
        float v = acc[i][j][e];
        if constexpr (EPI == EPI_BIAS_RELU) {
          v += bias[j];
          v = v > 0.0f ? v : 0.0f;
        }
        if constexpr (EPI == EPI_MASK) v = mask[i * C::WTN + j][e] > 0.0f ? v : 0.0f;
        if (whole || m < M) {
          if constexpr (EPI == EPI_F32)
            __builtin_nontemporal_store(v, &dst[(size_t)m * ld]);
          else
            dst[(size_t)m * ld] = v;
          if constexpr (EPI == EPI_MASK) colsum[j] += v;
        }
      }
  }
}

// SIDE: the first workgroups do a link of the grouping (group_device.hpp); workgroups then have kSortBlock threads, of which
// the products of a smaller shape leave the rest idle.
template <int EPI, typename C, bool SIDE = false>
__global__ void __launch_bounds__(SIDE ? kSortBlock : C::THREADS)
k_gemm_nt_tile(const typename C::T *__restrict__ A, const typename C::T *__restrict__ B, int M, int N, int K,
               const float *__restrict__ bias, const typename C::T *__restrict__ aux, void *__restrict__ out, int split,
               float *__restrict__ colpart, uint8_t *__restrict__ relu_bits, const int32_t *__restrict__ status,
               std::conditional_t<SIDE, SideTask, NoTask> side) {
  using T = typename C::T;
  if (status && *status != 0) return;
  constexpr bool kBf16 = sizeof(T) == 2;
  constexpr int kPatchBytes = kBf16 ? C::WAVES * 32 * PATCH_LD * 2 : 0;
  constexpr int kSumFloats = C::WAVES * 32 * C::WTN;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[C::STAGES * C::STAGE_BYTES];   // [stage][A rows | B rows]
  static_assert(kPatchBytes + kSumFloats * 4 <= C::STAGES * C::STAGE_BYTES, "patches and column sums fit");

  const int tid = threadIdx.x, lane = tid & 63;
  int block = blockIdx.x, blocks = gridDim.x;
  if constexpr (SIDE) {
    static_assert(C::THREADS <= kSortBlock && C::STAGES * C::STAGE_BYTES >= 12 << kSideDigitBits, "side work fits");
    if (block < side.blocks) return side_work(side, block, lds);
    block -= side.blocks;
    blocks -= side.blocks;
    if (tid >= C::THREADS) return;   // a barrier waits for wavefronts that are still there
  }
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
  const int n_tiles = (N + C::BN - 1) / C::BN;
  const int tile = xcd_remap(block, blocks);
  const int m0 = (tile / n_tiles) * C::BM, n0 = (tile % n_tiles) * C::BN;

  // this lane's piece of the rows it copies: LDS slot lane % 8 of row lane / 8 receives piece (lane % 8) ^ (row % 8)
  const int piece = (lane & 7) ^ (lane >> 3);
  const unsigned char *src[C::PER_STAGE];
#pragma unroll
  for (int i = 0; i < C::DMA_A; ++i)
    src[i] = reinterpret_cast<const unsigned char *>(A + (size_t)min(m0 + (i * C::WAVES + wave) * 8 + (lane >> 3), M - 1) * K) + piece * 16;
#pragma unroll
  for (int i = 0; i < C::DMA_B; ++i)
    src[C::DMA_A + i] =
        reinterpret_cast<const unsigned char *>(B + (size_t)min(n0 + (i * C::WAVES + wave) * 8 + (lane >> 3), N - 1) * K) + piece * 16;
  // What the epilogue needs from global memory is requested first and arrives while the products run.
  const int r = lane & 31, g = lane >> 5;
  const int wave_m0 = m0 + wm * C::WTM * 32, wave_n0 = n0 + wn * C::WTN * 32;
  float bias_reg[kBf16 ? 1 : C::WTN];
  if constexpr (EPI == EPI_BIAS_RELU) {
    if constexpr (kBf16) {
      static_assert(C::BN <= C::THREADS, "a thread fetches one bias");
      bias_reg[0] = tid < C::BN && n0 + tid < N ? bias[n0 + tid] : 0.0f;
    } else {
#pragma unroll
      for (int j = 0; j < C::WTN; ++j) bias_reg[j] = wave_n0 + j * 32 + r < N ? bias[wave_n0 + j * 32 + r] : 0.0f;
    }
  }
  uint32_t hbits[C::WTM][4];
#pragma unroll
  for (int i = 0; i < C::WTM; ++i)
#pragma unroll
    for (int it = 0; it < 4; ++it) hbits[i][it] = 0u;
  if constexpr (EPI == EPI_MASK_BITS) {
    const uint8_t *bits = reinterpret_cast<const uint8_t *>(aux);
    const int n_vec = n0 + wn * WN + (lane & 7) * 8;
#pragma unroll
    for (int i = 0; i < C::WTM; ++i)
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int m = wave_m0 + i * 32 + it * 8 + (lane >> 3);
        if (m < M && n_vec < N) hbits[i][it] = bits[(size_t)m * (N >> 3) + (n_vec >> 3)];
      }
  }
  float mask[EPI == EPI_MASK && !kBf16 ? C::WTM * C::WTN : 1][16];
  if constexpr (EPI == EPI_MASK && !kBf16) {
#pragma unroll
    for (int i = 0; i < C::WTM; ++i)
#pragma unroll
      for (int j = 0; j < C::WTN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int m = wave_m0 + i * 32 + 8 * (e / 4) + 4 * g + (e % 4), n = wave_n0 + j * 32 + r;
          mask[i * C::WTN + j][e] = aux[(size_t)min(m, M - 1) * N + min(n, N - 1)];
        }
  }

  const int nk = (K + C::KS - 1) / C::KS;
  const uint64_t zero = zero_address();
  auto issue = [&](int t, int stage) {
    unsigned char *a = lds + stage * C::STAGE_BYTES + wave * 1024, *b = a + C::BM * 128;
    if ((t + 1) * C::KS <= K) {
#pragma unroll
      for (int i = 0; i < C::PER_STAGE; ++i)
        copy_piece(src[i] + (size_t)t * 128, i < C::DMA_A ? a + i * C::WAVES * 1024 : b + (i - C::DMA_A) * C::WAVES * 1024);
    } else {
      const bool in = t * C::KS + piece * C::VEC < K;   // K is a multiple of a piece
#pragma unroll
      for (int i = 0; i < C::PER_STAGE; ++i)
        copy_piece_or_zero(src[i] + (size_t)t * 128, in, zero,
                           i < C::DMA_A ? a + i * C::WAVES * 1024 : b + (i - C::DMA_A) * C::WAVES * 1024);
    }
  };
#pragma unroll
  for (int p = 0; p < C::STAGES - 1; ++p)
    if (p < nk) issue(p, p);

  f32x16_v acc[C::WTM][C::WTN];
#pragma unroll
  for (int i = 0; i < C::WTM; ++i)
#pragma unroll
    for (int j = 0; j < C::WTN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
  const uint32_t in_row = (uint32_t)((g ^ (r & 7)) << 4);
  const uint32_t a_rel = lds_base + (uint32_t)(wm * C::WTM * 32 + r) * 128u + in_row;
  const uint32_t b_rel = lds_base + (uint32_t)(C::BM + wn * C::WTN * 32 + r) * 128u + in_row;
  nt_main_loop<C>(acc, a_rel, b_rel, nk, issue);

  if constexpr (kBf16) {
    static_assert(C::WTN == TN, "the patch epilogue takes wave tiles of 64 columns");
    __shared__ float s_bias[EPI == EPI_BIAS_RELU ? C::BN : 1];
    if constexpr (EPI == EPI_BIAS_RELU) {
      if (tid < C::BN) s_bias[tid] = bias_reg[0];
    }
    __syncthreads();   // every wave is done with the operand tiles: they become the output patches
    float colacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    epilogue_patch<EPI, C::WTM>(acc, reinterpret_cast<bf16_t *>(lds) + wave * 32 * PATCH_LD, m0, n0, wm, wn, lane, M, N, bias,
                                aux, out, split, relu_bits, colacc, s_bias, hbits);
    if constexpr (EPI == EPI_MASK || EPI == EPI_MASK_BITS) {
      if (colpart) {   // column sums of what was stored, per row tile: lanes, then the waves that share the columns
        float *s_col = reinterpret_cast<float *>(lds + kPatchBytes);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          float v = colacc[e];
          v += __shfl_xor(v, 8, kWave);
          v += __shfl_xor(v, 16, kWave);
          v += __shfl_xor(v, 32, kWave);
          if (lane < 8) s_col[wave * WN + lane * 8 + e] = v;
        }
        __syncthreads();
        if (wm == 0 && n0 + wn * WN + lane < N) {
          float v = s_col[wn * WN + lane];
#pragma unroll
          for (int w = 1; w < C::WAVES_M; ++w) v += s_col[(w * C::WAVES_N + wn) * WN + lane];
          colpart[(size_t)(m0 / C::BM) * N + n0 + wn * WN + lane] = v;
        }
      }
    }
  } else {
    // one wait for what was requested ahead, not one before every store
    if constexpr (EPI == EPI_BIAS_RELU) {
#pragma unroll
      for (int j = 0; j < C::WTN; ++j) landed(bias_reg[j]);
    }
    if constexpr (EPI == EPI_MASK) {
#pragma unroll
      for (int i = 0; i < C::WTM * C::WTN; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) landed(mask[i][e]);
    }
    float colsum[C::WTN];
    store_f32<EPI, C>(acc, wave_m0, wave_n0, lane, M, N, bias_reg, mask, reinterpret_cast<const float *>(aux), static_cast<float *>(out), split, colsum);
    if constexpr (EPI == EPI_MASK) {
      if (colpart) {
        float *s_col = reinterpret_cast<float *>(lds);
        __syncthreads();   // the operand tiles are not needed any more
#pragma unroll
        for (int j = 0; j < C::WTN; ++j) {
          const float v = colsum[j] + __shfl_xor(colsum[j], 32, kWave);
          if (lane < 32) s_col[(wave * C::WTN + j) * 32 + lane] = v;
        }
        __syncthreads();
        for (int k = tid; k < C::BN; k += C::THREADS) {
          const int w0 = k / (32 * C::WTN), at = k % (32 * C::WTN);
          float v = s_col[w0 * C::WTN * 32 + at];
#pragma unroll
          for (int w = 1; w < C::WAVES_M; ++w) v += s_col[(w * C::WAVES_N + w0) * C::WTN * 32 + at];
          if (n0 + k < N) colpart[(size_t)(m0 / C::BM) * N + n0 + k] = v;
        }
      }
    }
  }
}

// ---- TN: partial[z] = A[rows z]^T B[rows z] (tn_tile.hpp) -----------------------------------------------------
template <typename C>
__global__ void __launch_bounds__(C::THREADS)
k_gemm_tn_tile(TnTileArgs args, int K, int splits, const int32_t *__restrict__ status, const int32_t *__restrict__ k_dev) {
  if (status && *status != 0) return;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[C::STAGES * C::STAGE_BYTES];
  tn_tile<C>(args, K, splits, k_dev, xcd_remap(blockIdx.x, gridDim.x), lds);
}

// bf16: what the ranges leave is written, read again and added by the parameter update, so two workgroups of a CU that would walk
// neighbouring ranges of one tile are one of twice the wavefronts instead, which leaves one partial: of 576 -> 512 -> 256 15 MB and not 31.
// us a step, single / pairs, in blocks: 16 384 views 153.4 / 150.0, with Adam 158.5 / 154.9, 10 001 127.4 / 125.6 (on the same batch
// over and over, whose rows are in the caches, 138.8 / 138.5, 142.7 / 141.0, 118.3 / 117.3); layer by layer on two
// streams, with the accumulation beside them: 8193 of 1024 -> 256 168.3 / 164.5, 12 000 of 704 -> 640 -> 128 212.6 / 209.5, 16 384 of 1024 ->
// 1024 304.6 / 298.5, 32 736 of 576 -> 512 -> 256 327.6 / 321.3; on one, 2000 of 576 -> 512 -> 256 108.5 / 106.7.  Where whole ranges of pairs
// leave more of the CUs out than those of single ones do, they are not taken (26 tiles, 234 of 256 against 494 of 512: 184.9 / 186.9), nor
// where there are as many ranges either way, so that no partial is left out (a range has 64 rows at least, and there are 64 at most: 600
// views of 320 -> 256 91.6 / 92.1, 1500 of 128 -> 64 82.7 / 83.4, 16 384 of 128 -> 128 134.0 / 135.1, wider ones the same), nor in fp32, whose
// 64 x 64 tiles leave little (16 384 views 157.3 / 158.0).
template <typename C>
__global__ void __launch_bounds__(2 * C::THREADS)
k_gemm_tn_pair(TnTileArgs args, int K, int splits, const int32_t *__restrict__ status, const int32_t *__restrict__ k_dev) {
  if (status && *status != 0) return;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * C::STAGES * C::STAGE_BYTES];
  tn_tile<C, true>(args, K, splits, k_dev, xcd_remap(blockIdx.x, gridDim.x), lds);
}

// ---- tile shapes -----------------------------------------------------------------------------------------
using F32Small = NtTile<float, 1, 1, 2, 2, 4>;      //  64 x  64, 64 KB
using F32Big = NtTile<float, 2, 2, 2, 2, 3>;        // 128 x 128, 96 KB
using F32Pair = NtTile<float, 2, 2, 2, 2, 2>;       // 128 x 128, 64 KB: two on a CU, one stores while the other multiplies
using Bf16Small = NtTile<bf16_t, 1, 2, 2, 1, 3>;    //  64 x  64, two waves, 48 KB
using Bf16Tall = NtTile<bf16_t, 1, 2, 4, 1, 2>;     // 128 x  64, 48 KB
using Bf16Mid = NtTile<bf16_t, 2, 2, 2, 2, 2>;      // 128 x 128, 64 KB
using TnF32 = TnTile<float, 1, 1, 4>;               //  64 x  64, 64 KB
using TnBf16 = TnTile<bf16_t, 2, 2, 4>;             // 128 x 128, 64 KB

long long tiles_of(int M, int N, int bm, int bn) { return (long long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); }

template <int EPI, typename C>
hipError_t run_nt(const void *A, const void *B, int M, int N, int K, const float *bias, const void *aux, void *out, int split,
                  float *colpart, uint8_t *relu_bits, const int32_t *status, hipStream_t s, const SideTask *side, hipEvent_t stop) {
  using T = typename C::T;
  const unsigned tiles = (unsigned)tiles_of(M, N, C::BM, C::BN);
  if constexpr (EPI == EPI_BIAS_RELU || EPI == EPI_DX) {
    if (side) {
      launch_leaving(stop, k_gemm_nt_tile<EPI, C, true>, dim3(tiles + side->blocks), kSortBlock, 0, s, (const T *)A, (const T *)B, M, N, K,
                     bias, (const T *)aux, out, split, colpart, relu_bits, status, *side);
      return hipGetLastError();
    }
  }
  if (side) return hipErrorInvalidValue;
  launch_leaving(stop, k_gemm_nt_tile<EPI, C>, dim3(tiles), C::THREADS, 0, s, (const T *)A, (const T *)B, M, N, K, bias, (const T *)aux,
                 out, split, colpart, relu_bits, status, NoTask{});
  return hipGetLastError();
}

template <typename C>
hipError_t run_nt_any(const void *A, const void *B, int M, int N, int K, int epi, const float *bias, const void *aux, void *out,
                      int split, float *colpart, uint8_t *relu_bits, const int32_t *status, hipStream_t s, const SideTask *side, hipEvent_t stop) {
#define GEAR_NT(E) run_nt<E, C>(A, B, M, N, K, bias, aux, out, split, colpart, relu_bits, status, s, side, stop)
  switch (epi) {
    case EPI_BIAS_RELU: return GEAR_NT(EPI_BIAS_RELU);
    case EPI_MASK: return GEAR_NT(EPI_MASK);
    case EPI_DX: return GEAR_NT(EPI_DX);
    case EPI_F32: return run_nt<EPI_F32, std::conditional_t<std::is_same_v<C, F32Big>, F32Pair, C>>(A, B, M, N, K, bias, aux, out, split, colpart, relu_bits, status, s, side, stop);
    case EPI_MASK_BITS:
      if constexpr (sizeof(typename C::T) == 2) return GEAR_NT(EPI_MASK_BITS);
  }
#undef GEAR_NT
  return hipErrorInvalidValue;
}

// The shape a product of M x N takes.
enum NtShape { kSmall, kTall, kWide };   // 64 x 64, 128 x 64 (bf16 only), 128 x 128
int rows_of(NtShape shape) { return shape == kSmall ? 64 : 128; }

// bf16: two 128 x 128 tiles or three of 128 x 64 fit on a CU.  A 128 x 128 tile moves a quarter fewer bytes for its
// products (16384 x 512 x 576: 14.2 us against 17.0), as long as whole rounds of them fill the chip; where the last
// round is mostly empty the half-sized tiles end sooner (16384 x 576 x 512, 640 tiles: 18.8 against 17.6; 10001 x 512
// x 576, 316 tiles: 13.2 against 12.7).  Below one 128 x 64 tile per CU, 64 x 64 reaches more CUs.
// fp32: a CU holds one 128 x 128 tile or two of 64 x 64, and both shapes run at the rate of its matrix unit, so what decides
// is how full the last round is: 40 us a round of large tiles at K = 512, 10.4 us a half round of small ones and 2 us more
// to begin with (K = 512, bias + ReLU, us, 128 x 128 / 64 x 64: 16384 x 256 43.3 / 45.5, 16384 x 320 81 / 57, 8192 x 320
// 42 / 36, 20000 x 384 82 / 86, 24000 x 320 121 / 86, 32768 x 64 43 / 25).
// dLoss/dx keeps the large tiles from one per CU on: alone 16384 x 320 x 256 is 13 us shorter on small ones, but a step of two
// streams (139 000 ids) was 2 us longer with them; what takes the time back is not known.
// EPI_F32 has two large tiles on a CU as well, a half round of them 19 us at K = 256 where one of small ones is 5.3 (16384 x
// 384 39 / 35, 20000 x 320 39 / 40, 24000 x 576 76 / 78).
// `coarse` (column sums of more, narrower row tiles would not fit their region) rules 64 x 64 out.
NtShape nt_shape(int dtype, int M, int N, bool coarse, int epi = EPI_MASK) {
  const long long big = tiles_of(M, N, 128, 128);
  if (dtype != GEAR_BF16) {
    const long long rounds = (big + 255) / 256, halves = (tiles_of(M, N, 64, 64) + 255) / 256;
    if (epi == EPI_DX) return big >= 256 ? kWide : kSmall;
    if (epi == EPI_F32) return 29 * halves > 100 * rounds ? kWide : kSmall;
    return coarse || 26 * halves + 5 > 100 * rounds ? kWide : kSmall;
  }
  const long long tall = tiles_of(M, N, 128, 64);
  if (tall < 256) return coarse ? kTall : kSmall;
  return 2 * ((big + 511) / 512) <= (tall + 767) / 768 ? kWide : kTall;
}

template <typename C>
hipError_t run_tn(const TnProblem *p, int count, int K, int splits, bool pairs, const int32_t *status, hipStream_t s, const int32_t *k_dev) {
  TnTileArgs args;
  static_assert(C::BM == C::BN, "square tiles");
  (void)tn_tile_args(p, count, C::BM, &args);
  if (pairs && sizeof(typename C::T) == 2 && !k_dev && args.tiles * splits <= 256)
    hipLaunchKernelGGL((k_gemm_tn_pair<C>), dim3((unsigned)(args.tiles * splits)), dim3(2 * C::THREADS), 0, s, args, K, splits, status, k_dev);
  else
    hipLaunchKernelGGL((k_gemm_tn_tile<C>), dim3((unsigned)(args.tiles * splits)), dim3(C::THREADS), 0, s, args, K, splits, status, k_dev);
  return hipGetLastError();
}

}  // namespace

int nt_tile_colsum_parts(int dtype, int M, int N, bool coarse) {
  const int rows = rows_of(nt_shape(dtype, M, N, coarse));
  return (M + rows - 1) / rows;
}

hipError_t launch_gemm_nt_tile(int dtype, const void *A, const void *B, int M, int N, int K, int epi, const float *bias,
                               const void *aux, void *out, int split, float *colpart, uint8_t *relu_bits,
                               const int32_t *status, hipStream_t s, bool coarse, const SideTask *side, hipEvent_t stop) {
  const NtShape shape = nt_shape(dtype, M, N, coarse, epi);
#define GEAR_NT(C) run_nt_any<C>(A, B, M, N, K, epi, bias, aux, out, split, colpart, relu_bits, status, s, side, stop)
  if (dtype == GEAR_BF16) return shape == kWide ? GEAR_NT(Bf16Mid) : shape == kTall ? GEAR_NT(Bf16Tall) : GEAR_NT(Bf16Small);
  return shape == kWide ? GEAR_NT(F32Big) : GEAR_NT(F32Small);
#undef GEAR_NT
}

static long long tn_tiles(int dtype, const TnProblem *p, int count) {
  long long tiles = 0;
  const int edge = dtype == GEAR_BF16 ? TnBf16::BM : TnF32::BM;
  for (int i = 0; i < count; ++i) tiles += tiles_of(p[i].M, p[i].N, edge, edge);
  return tiles;
}

// Ranges of the inner length: `slots` for all CUs, as long as each keeps at least 64 rows.
static int tn_splits(int dtype, const TnProblem *p, int count, int K, int slots) {
  const long long tiles = tn_tiles(dtype, p, count);
  long long s = tiles > 0 ? slots / tiles : 1;
  if (s > K / 64) s = K / 64;
  if (s > 64) s = 64;
  return s < 1 ? 1 : (int)s;
}
int tn_tile_splits(int dtype, const TnProblem *p, int count, int K, bool *pairs) {
  const int all = tn_splits(dtype, p, count, K, 512), half = tn_splits(dtype, p, count, K, 256);
  *pairs = *pairs && dtype == GEAR_BF16 && half < all && 200 * half >= 97 * all;
  return *pairs ? half : all;
}

long long tn_tile_rows(int dtype, const TnProblem *p, int count, int K) {
  const int splits = tn_splits(dtype, p, count, K, 512);
  return (tn_tiles(dtype, p, count) * splits + 511) / 512 * ((K + splits - 1) / splits);
}

hipError_t launch_gemm_tn_tile(int dtype, const TnProblem *p, int count, int K, int splits, bool pairs, const int32_t *status, hipStream_t s,
                               const int32_t *k_dev) {
  return dtype == GEAR_BF16 ? run_tn<TnBf16>(p, count, K, splits, pairs, status, s, k_dev)
                            : run_tn<TnF32>(p, count, K, splits, pairs, status, s, k_dev);
}

}  // namespace gear
