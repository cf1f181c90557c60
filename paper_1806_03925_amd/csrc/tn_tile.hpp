// Device code of the weight gradients on tiles of moderate size (gemm_tile.hip has the products' own launches, accum_wgrad.hip
// has these beside the accumulation), and the copies, LDS reads and waits that all products on such tiles use.
#pragma once

#include "gemm_common.hpp"

namespace gear {
namespace {

__device__ uint4 g_zero_piece;   // sixteen zero bytes, the source of every piece beyond an operand's end

template <int N> __device__ __forceinline__ void wait_lgkm() { asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory"); }
template <typename V> __device__ __forceinline__ void landed(V &r) { asm volatile("" : "+v"(r)); }
template <int OFF> __device__ __forceinline__ void lds_read16(u32x4_v &dst, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
}
template <int OFF> __device__ __forceinline__ void lds_read4(float &dst, uint32_t addr) {
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
}
template <int OFF> __device__ __forceinline__ void lds_read_tr(u32x2_v &dst, uint32_t addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
}

// One 16-byte piece per lane from global memory to LDS (lane i's goes to dst + 16 i), or zeros where `in` is false.
// The choice of source is hidden from the compiler, which would otherwise copy under two execution masks in turn.
__device__ __forceinline__ void copy_piece(const void *src, unsigned char *dst) {
  __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)dst, 16, 0, 0);
}
__device__ __forceinline__ void copy_piece_or_zero(const void *src, bool in, uint64_t zero, unsigned char *dst) {
  uint64_t at = in ? (uint64_t)(uintptr_t)src : zero;
  asm volatile("" : "+v"(at));
  __builtin_amdgcn_global_load_lds((const void *)(uintptr_t)at, (lds_ptr_t)dst, 16, 0, 0);
}
__device__ __forceinline__ uint64_t zero_address() {   // fetched once, not before every use
  uint64_t z = (uint64_t)(uintptr_t)&g_zero_piece;
  asm volatile("" : "+s"(z));
  return z;
}

// wait until at most `stages` later stages of PER copies each are outstanding (0 <= stages <= MAX)
template <int PER, int MAX> __device__ __forceinline__ void wait_stages(int stages) {
  if constexpr (MAX == 0) {
    wait_vm<0>();
  } else {
    if (stages >= MAX)
      wait_vm<PER * MAX>();
    else
      wait_stages<PER, MAX - 1>(stages);
  }
}

// ---- TN: partial[z] = A[rows z]^T B[rows z], a stage is 32 rows of the batch --------------------------------
template <typename T_, int WTM_, int WTN_, int STAGES_> struct TnTile {
  using T = T_;
  static constexpr int WTM = WTM_, WTN = WTN_, STAGES = STAGES_, WAVES = 4, THREADS = 256;   // 2 x 2 waves
  static constexpr int BM = 64 * WTM, BN = 64 * WTN, KD = 32, ROUND = sizeof(T) == 2 ? 32 : 16;   // rows of a stage; a range is a multiple of ROUND
  static constexpr int ROW = BM * (int)sizeof(T);                 // bytes of a k-row of either operand
  static constexpr int PIECES = ROW / 16, ROWS_PER_DMA = 64 / PIECES;
  static constexpr int OPERAND_BYTES = KD * ROW, STAGE_BYTES = 2 * OPERAND_BYTES;
  static constexpr int DMA = KD / ROWS_PER_DMA / WAVES;           // instructions of a wave per operand and stage
  static_assert(BM == BN && PIECES == 16, "256-byte k-rows: a DMA instruction copies four of them");
};

// fp32: the k-row order in LDS is what v_mfma_f32_32x32x2_f32 wants (half a wave reads 32 neighbouring values).
// bf16: ds_read_b64_tr_b16 assembles eight k-values of a row per lane (sixteen lanes hand in a 4(k) x 16 block);
// pieces are XOR-ed by 4 (k % 4), so that the four k-rows a read touches lie in different quarters of the banks.
template <typename C>
__device__ __forceinline__ void mma_stage_rows(f32x16_v (&acc)[C::WTM][C::WTN], const uint32_t (&a_addr)[C::WTM],
                                               const uint32_t (&b_addr)[C::WTN], uint32_t so) {
  if constexpr (sizeof(typename C::T) == 4) {
    static_assert(C::WTM == 1 && C::WTN == 1, "one tile per wave in fp32");
    constexpr int STEPS = C::KD / 2;
    float a[STEPS], b[STEPS];
    const uint32_t aa = a_addr[0] + so, bb = b_addr[0] + so;
#define GEAR_ROW(K)                                   \
  lds_read4<(K) * 2 * C::ROW>(a[K], aa);              \
  lds_read4<(K) * 2 * C::ROW>(b[K], bb);
    GEAR_ROW(0) GEAR_ROW(1) GEAR_ROW(2) GEAR_ROW(3) GEAR_ROW(4) GEAR_ROW(5) GEAR_ROW(6) GEAR_ROW(7)
    wait_lgkm<8>();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      landed(a[k]);
      landed(b[k]);
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[k], b[k], acc[0][0], 0, 0, 0);
    }
    GEAR_ROW(8) GEAR_ROW(9) GEAR_ROW(10) GEAR_ROW(11)
    wait_lgkm<8>();
#pragma unroll
    for (int k = 4; k < 8; ++k) {
      landed(a[k]);
      landed(b[k]);
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[k], b[k], acc[0][0], 0, 0, 0);
    }
    GEAR_ROW(12) GEAR_ROW(13) GEAR_ROW(14) GEAR_ROW(15)
#undef GEAR_ROW
    wait_lgkm<8>();
#pragma unroll
    for (int k = 8; k < 12; ++k) {
      landed(a[k]);
      landed(b[k]);
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[k], b[k], acc[0][0], 0, 0, 0);
    }
    wait_lgkm<0>();
#pragma unroll
    for (int k = 12; k < 16; ++k) {
      landed(a[k]);
      landed(b[k]);
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[k], b[k], acc[0][0], 0, 0, 0);
    }
  } else {
    static_assert(C::WTM == 2 && C::WTN == 2, "2 x 2 tiles per wave in bf16");
    u32x2_v a[2][2][2], b[2][2][2];   // [k-step][tile][k-rows +0..3 | +4..7 of the lane's eight]
#define GEAR_TR(KK)                                                      \
  lds_read_tr<(KK) * 16 * C::ROW>(a[KK][0][0], a_addr[0] + so);          \
  lds_read_tr<(KK) * 16 * C::ROW + 4 * C::ROW>(a[KK][0][1], a_addr[0] + so); \
  lds_read_tr<(KK) * 16 * C::ROW>(a[KK][1][0], a_addr[1] + so);          \
  lds_read_tr<(KK) * 16 * C::ROW + 4 * C::ROW>(a[KK][1][1], a_addr[1] + so); \
  lds_read_tr<(KK) * 16 * C::ROW>(b[KK][0][0], b_addr[0] + so);          \
  lds_read_tr<(KK) * 16 * C::ROW + 4 * C::ROW>(b[KK][0][1], b_addr[0] + so); \
  lds_read_tr<(KK) * 16 * C::ROW>(b[KK][1][0], b_addr[1] + so);          \
  lds_read_tr<(KK) * 16 * C::ROW + 4 * C::ROW>(b[KK][1][1], b_addr[1] + so);
    GEAR_TR(0)
    GEAR_TR(1)
#undef GEAR_TR
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      if (kk == 0)
        wait_lgkm<8>();
      else
        wait_lgkm<0>();
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          landed(a[kk][i][h]);
          landed(b[kk][i][h]);
        }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const u32x4_v av = {a[kk][i][0].x, a[kk][i][0].y, a[kk][i][1].x, a[kk][i][1].y};
          const u32x4_v bv = {b[kk][j][0].x, b[kk][j][0].y, b[kk][j][1].x, b[kk][j][1].y};
          MFMA_BF16(acc[i][j], av, bv);
        }
    }
  }
}

struct TnTileArgs {
  int count, tiles;
  TnProblem p[GEAR_MAX_LAYERS];
  int first_tile[GEAR_MAX_LAYERS];
};

// the arguments of `count` problems on tiles of edge x edge; returns the number of tiles
inline int tn_tile_args(const TnProblem *p, int count, int edge, TnTileArgs *args) {
  args->count = count;
  args->tiles = 0;
  for (int i = 0; i < GEAR_MAX_LAYERS; ++i) {
    args->p[i] = i < count ? p[i] : TnProblem{nullptr, nullptr, nullptr, 0, 0};
    args->first_tile[i] = args->tiles;
    if (i < count) args->tiles += ((p[i].M + edge - 1) / edge) * ((p[i].N + edge - 1) / edge);
  }
  return args->tiles;
}

// `work`: one of k-ranges x (all tiles of all problems).  k_dev (may be NULL): the real inner length, at most K, only
// known on the device; the ranges are then cut there, and one beyond the end leaves zeros.
// lds: C::STAGES * C::STAGE_BYTES, aligned to 1024.
// PAIR: 512 threads and twice the LDS; either half of the wavefronts walks one half of the range, and the first adds the second's result
// to its own.
template <typename C, bool PAIR = false>
__device__ __forceinline__ void tn_tile(const TnTileArgs &args, int K, int splits, const int32_t *__restrict__ k_dev, int work,
                                        unsigned char *lds) {
  using T = typename C::T;
  if (k_dev) K = min(max(*k_dev, 0), K);
  const int k_chunk = max(((K + splits - 1) / splits + C::ROUND - 1) / C::ROUND * C::ROUND, C::ROUND);
  const int z = work / args.tiles, tile_all = work % args.tiles;
  int which = 0;
  for (int i = 1; i < args.count; ++i)
    if (tile_all >= args.first_tile[i]) which = i;
  const TnProblem &q = args.p[which];
  const int M = q.M, N = q.N, tile = tile_all - args.first_tile[which];
  const int n_tiles = (N + C::BN - 1) / C::BN;
  const int m0 = (tile / n_tiles) * C::BM, n0 = (tile % n_tiles) * C::BN;
  int k_begin = z * k_chunk, k_end = min(K, k_begin + k_chunk);

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & (C::WAVES - 1));
  const int half = PAIR ? __builtin_amdgcn_readfirstlane(threadIdx.x / C::THREADS) : 0;
  int rounds = k_end > k_begin ? (k_end - k_begin + C::KD - 1) / C::KD : 0;   // of the longer half
  if constexpr (PAIR) {
    lds += half * C::STAGES * C::STAGE_BYTES;
    rounds = (rounds + 1) / 2;
    const int middle = min(k_end, k_begin + rounds * C::KD);
    if (half == 0)
      k_end = middle;
    else
      k_begin = middle;
  }
  const int wm = wave >> 1, wn = wave & 1;
  constexpr int VEC = 16 / (int)sizeof(T);
  // a DMA instruction copies four k-rows; LDS slot lane % 16 of k-row lane / 16 receives this piece of the row
  const int krow = lane >> 4;
  const int piece = sizeof(T) == 2 ? (lane & 15) ^ (4 * krow) : (lane & 15);
  const T *a_src = static_cast<const T *>(q.A) + min(m0 + piece * VEC, M - VEC);
  const T *b_src = static_cast<const T *>(q.B) + min(n0 + piece * VEC, N - VEC);
  const int nk = k_end > k_begin ? (k_end - k_begin + C::KD - 1) / C::KD : 0;
  const uint64_t zero = zero_address();
  auto issue = [&](int t, int stage) {
    unsigned char *a = lds + stage * C::STAGE_BYTES + wave * 1024, *b = a + C::OPERAND_BYTES;
    const bool full = k_begin + (t + 1) * C::KD <= k_end;
#pragma unroll
    for (int i = 0; i < C::DMA; ++i) {
      const int k = k_begin + t * C::KD + (i * C::WAVES + wave) * C::ROWS_PER_DMA + krow;
      if (full) {
        copy_piece(a_src + (size_t)k * M, a + i * C::WAVES * 1024);
        copy_piece(b_src + (size_t)k * N, b + i * C::WAVES * 1024);
      } else {
        copy_piece_or_zero(a_src + (size_t)k * M, k < k_end, zero, a + i * C::WAVES * 1024);
        copy_piece_or_zero(b_src + (size_t)k * N, k < k_end, zero, b + i * C::WAVES * 1024);
      }
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
  uint32_t a_addr[C::WTM], b_addr[C::WTN];
  if constexpr (sizeof(T) == 4) {
    const uint32_t at = (uint32_t)(lane >> 5) * C::ROW + (uint32_t)(lane & 31) * 4u;
    a_addr[0] = lds_base + at + (uint32_t)wm * 128u;
    b_addr[0] = lds_base + C::OPERAND_BYTES + at + (uint32_t)wn * 128u;
  } else {
    const int j = lane & 15, h = (lane >> 4) & 1, g = lane >> 5;
    const uint32_t at = (uint32_t)(8 * g + (j >> 2)) * C::ROW + 32u * h + 8u * (j & 3);
#pragma unroll
    for (int i = 0; i < C::WTM; ++i) a_addr[i] = lds_base + at + (uint32_t)(((wm * C::WTM + i) ^ (j >> 2)) << 6);
#pragma unroll
    for (int i = 0; i < C::WTN; ++i)
      b_addr[i] = lds_base + C::OPERAND_BYTES + at + (uint32_t)(((wn * C::WTN + i) ^ (j >> 2)) << 6);
  }
  int stage = 0, fill = C::STAGES - 1;
  for (int t = 0; t < rounds; ++t) {
    if (!PAIR || t < nk) wait_stages<2 * C::DMA, C::STAGES - 2>(nk - 1 - t);
    block_barrier();
    if (PAIR && t >= nk) break;   // the second half's last round, if it has one less; no barrier of the first half's is behind it
    if (t + C::STAGES - 1 < nk) issue(t + C::STAGES - 1, fill);
    mma_stage_rows<C>(acc, a_addr, b_addr, (uint32_t)stage * C::STAGE_BYTES);
    stage = stage + 1 == C::STAGES ? 0 : stage + 1;
    fill = fill + 1 == C::STAGES ? 0 : fill + 1;
  }
  if constexpr (PAIR) {
    static_assert(C::WTM * C::WTN * 16 * C::THREADS * 4 <= C::STAGES * C::STAGE_BYTES, "a half's result fits in its stages");
    block_barrier();   // all reads of the stages are done
    float *other = reinterpret_cast<float *>(half == 0 ? lds + C::STAGES * C::STAGE_BYTES : lds) + threadIdx.x % C::THREADS;
    if (half == 1) {
#pragma unroll
      for (int i = 0; i < C::WTM; ++i)
#pragma unroll
        for (int j = 0; j < C::WTN; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) other[((i * C::WTN + j) * 16 + e) * C::THREADS] = acc[i][j][e];
      wait_lgkm<0>();
    }
    block_barrier();
    if (half == 1) return;
#pragma unroll
    for (int i = 0; i < C::WTM; ++i)
#pragma unroll
      for (int j = 0; j < C::WTN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] += other[((i * C::WTN + j) * 16 + e) * C::THREADS];
  }
  float *dst = q.partial + (size_t)z * M * N;
  const int c = lane & 31, g = lane >> 5;
#pragma unroll
  for (int i = 0; i < C::WTM; ++i)
#pragma unroll
    for (int j = 0; j < C::WTN; ++j) {
      const int n = n0 + (wn * C::WTN + j) * 32 + c;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = m0 + (wm * C::WTM + i) * 32 + 8 * (e / 4) + 4 * g + (e % 4);
        if (m < M && n < N) dst[(size_t)m * N + n] = acc[i][j][e];
      }
    }
}

}  // namespace
}  // namespace gear
