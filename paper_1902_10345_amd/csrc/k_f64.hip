// k_f64.hip -- binary64 GEMM on the FP64 matrix cores (gfx950).
//
// C <- alpha*A*B + beta*C in binary64 with v_mfma_f64_16x16x4f64 (every
// product and sum rounded in binary64).  The structure follows the paper's MM
// transformation chain (Sec. 6.2) the same way the binary32 kernels do:
//   MapTiling       BM x BN workgroup tile, waves of WM x WN, each a grid of
//                   16 x 16 MFMA blocks; K in 16-deep slabs.
//   LocalStorage /  A slab as [BM][16] and B slab transposed as [BN][16]
//   DoubleBuffering binary64 in LDS (128-byte rows, XOR-swizzled 16-byte
//                   chunks), two stages; slab t+1 is loaded while slab t is
//                   multiplied.
//   Vectorization   128-bit loads of A rows, 128-bit LDS writes and reads.
//   ReducePeeling   alpha/beta applied once in the epilogue.
// A batch of equally shaped problems at fixed element strides (the
// batched-strided product of the paper's quantum-transport case study,
// Sec. 6.4) runs the same tiles, or sub-tiles of one wave each straight from
// memory.
//
// MFMA operand layout (16x16x4, measured on gfx950): lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator element e of lane l
// is D[l / 16 + 4 e][l % 16].  Here lane group g = l / 16 owns k = 4g..4g+3
// of each slab and MFMA step q multiplies k = 4g + q, so each lane's k values
// are contiguous (two 16-byte LDS reads per 16 x 16 block and slab) and every
// k of the slab enters exactly once.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.hpp"
#include "f64_slabs.hpp"
#include "kernels.hpp"

namespace mm {
namespace f64 {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int CH = BK / 2;   // 16-byte chunks (two binary64) per LDS row
constexpr int kBufferFlags = 0x00020000;
enum { kFast, kGuarded, kMasked };  // how a tile loads a slab

// 128-byte rows: 16 consecutive rows at one logical chunk occupy 16 distinct
// 16-byte bank groups.
__device__ __forceinline__ int swz(int r) { return (r ^ (r >> 3)) & 7; }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const double *p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(p), (short)0,
                                           bytes > 0 ? (int)bytes : 0, kBufferFlags);
}

__device__ __forceinline__ double ld1(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}

__device__ __forceinline__ f64x2 ld2(__amdgpu_buffer_rsrc_t r, int voff) {
  return __builtin_bit_cast(f64x2, __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0));
}

template <int BM, int BN, int WM, int WN>
struct Cfg {
  static constexpr int NW = (BM / WM) * (BN / WN);   // waves of one k group
  static constexpr int NT = 64 * NW;
  static constexpr int WAVES_N = BN / WN;
  static constexpr int FM = WM / 16, FN = WN / 16;   // 16 x 16 blocks per wave
  static constexpr int A_ITEMS = BM * CH / NT;        // 16-byte items per lane
  static constexpr int B_ITEMS = BN * CH / NT;
  static_assert(A_ITEMS * NT == BM * CH && B_ITEMS * NT == BN * CH, "even split");
  // a wave's 64 lanes cover 64 consecutive B columns at one chunk index, so
  // the chunk's k-row offset is wave-uniform (a scalar offset)
  static_assert(BN % 64 == 0, "B chunk index must be wave-uniform");
  static constexpr int MIN_WG = NW >= 8 ? 1 : 2;   // workgroups per CU to plan registers for
  static constexpr int STAGE = (BM + BN) * BK;        // binary64 elements per stage
};

// One output tile of one problem.  A rows are read in 128-bit loads whatever
// lda, K and the base (a 128-bit buffer load needs only 4-byte alignment).
// The launcher guarantees that the byte extents of an A row panel (BM rows, or M
// where that is less) and of a B slab (16 rows, or K) stay below 2^31.
//
// KG = 2: two groups of NW waves share the workgroup, each with its own half
// of the slabs and its own LDS stages; the second group's partial tile is
// added to the first's through LDS, and two slabs of global loads are in flight
// per lane instead of one.  For products with one tile per CU at most, where
// nothing else hides a workgroup's latency (64 x 64 tiles, 1024^3: 50 -> 43 us;
// one of the two changes alone 48).  With more tiles per CU it is slower
// (1999 x 1501 x 1003: 106 -> 112).
template <int BM, int BN, int WM, int WN, int KG, bool BETA>
__device__ __forceinline__ void tile(int M, int N, int K, double alpha, const double *__restrict__ A,
                                     int64_t lda, const double *__restrict__ B, int64_t ldb,
                                     double beta, double *__restrict__ C, int64_t ldc, int m0,
                                     int n0, double *lds) {
  using G = Cfg<BM, BN, WM, WN>;
  constexpr int NT = G::NT;
  const int group = KG > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT) : 0;
  const int tid = KG > 1 ? (int)threadIdx.x % NT : (int)threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  lds += group * 2 * G::STAGE;
  const int Mr = M - m0, Nr = N - n0;
  const bool interior = Mr >= BM && Nr >= BN;
  const int rowsA = Mr < BM ? Mr : BM;
  const int colsB = Nr < BN ? Nr : BN;
  // A row panel: valid bytes end with the last valid row's K elements
  const __amdgpu_buffer_rsrc_t rA = rsrc(A + (int64_t)m0 * lda, ((int64_t)(rowsA - 1) * lda + K) * 8);
  int a_off[G::A_ITEMS];
#pragma unroll
  for (int i = 0; i < G::A_ITEMS; ++i) {
    const int idx = tid + NT * i;
    a_off[i] = idx / CH < rowsA ? ((idx / CH) * (int)lda + (idx % CH) * 2) * 8 : (int)0x80000000;
  }
  // B: this lane's column (out-of-range columns get an offset past any slab)
  // and the item's first k row (wave-uniform)
  int b_col[G::B_ITEMS], b_row[G::B_ITEMS];
  const int ldb8 = (int)ldb * 8;
#pragma unroll
  for (int i = 0; i < G::B_ITEMS; ++i) {
    const int idx = tid + NT * i;
    const int n = idx % BN;
    b_col[i] = n < colsB ? n * 8 : (int)0x80000000;
    b_row[i] = __builtin_amdgcn_readfirstlane(2 * (idx / BN)) * ldb8;
  }

  constexpr int DEPTH = KG;  // slabs of global loads in flight
  double ra_[DEPTH][G::A_ITEMS][2], rb_[DEPTH][G::B_ITEMS][2];
  // FAST: the slab lies inside [0, K) or, GUARD, begins before k = 0 and is not
  // multiplied; otherwise k outside [0, K) read as 0.
  auto gload = [&](auto F, auto SET, int k0) {
    constexpr bool FAST = decltype(F)::value != kMasked, GUARD = decltype(F)::value == kGuarded;
    auto &ra = ra_[decltype(SET)::value];
    auto &rb = rb_[decltype(SET)::value];
#pragma unroll
    for (int i = 0; i < G::A_ITEMS; ++i) {
      if (FAST) {
        const f64x2 v = ld2(rA, a_off[i] + k0 * 8);
        ra[i][0] = v.x;
        ra[i][1] = v.y;
      } else {
        const int k = k0 + ((tid + NT * i) % CH) * 2;
#pragma unroll
        for (int e = 0; e < 2; ++e)
          ra[i][e] = ld1(rA, (k + e >= 0 && k + e < K) ? a_off[i] + (k0 + e) * 8 : (int)0x80000000, 0);
      }
    }
    if (FAST) {
      const __amdgpu_buffer_rsrc_t rB =
          rsrc(B + (int64_t)(unsigned)(GUARD && k0 < 0 ? 0 : k0) * ldb + n0,
               (GUARD ? slab_extent(k0, ldb, colsB) : (int64_t)(BK - 1) * ldb + colsB) * 8);
#pragma unroll
      for (int i = 0; i < G::B_ITEMS; ++i)
#pragma unroll
        for (int e = 0; e < 2; ++e) rb[i][e] = ld1(rB, b_col[i], b_row[i] + e * ldb8);
    } else {
#pragma unroll
      for (int i = 0; i < G::B_ITEMS; ++i) {
        const int idx = tid + NT * i;
        const int c = __builtin_amdgcn_readfirstlane(idx / BN);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int k = k0 + 2 * c + e;
          const bool kin = k >= 0 && k < K;
          const __amdgpu_buffer_rsrc_t r = rsrc(B + (int64_t)(kin ? k : 0) * ldb + n0, kin ? colsB * 8 : 0);
          rb[i][e] = ld1(r, (idx % BN) * 8, 0);
        }
      }
    }
  };
  auto sstore = [&](auto SET, int stage) {
    auto &ra = ra_[decltype(SET)::value];
    auto &rb = rb_[decltype(SET)::value];
    double *sA = lds + stage * G::STAGE;
    double *sB = sA + BM * BK;
#pragma unroll
    for (int i = 0; i < G::A_ITEMS; ++i) {
      const int idx = tid + NT * i;
      const int r = idx / CH, c = idx % CH;
      *reinterpret_cast<f64x2 *>(sA + r * BK + ((c ^ swz(r)) << 1)) = f64x2{ra[i][0], ra[i][1]};
    }
#pragma unroll
    for (int i = 0; i < G::B_ITEMS; ++i) {
      const int idx = tid + NT * i;
      const int n = idx % BN, c = idx / BN;
      *reinterpret_cast<f64x2 *>(sB + n * BK + ((c ^ swz(n)) << 1)) = f64x2{rb[i][0], rb[i][1]};
    }
  };

  const int wm0 = (wave / G::WAVES_N) * WM, wn0 = (wave % G::WAVES_N) * WN;
  const int lr = lane & 15, lg = lane >> 4;
  f64x4 acc[G::FM][G::FN];
#pragma unroll
  for (int i = 0; i < G::FM; ++i)
#pragma unroll
    for (int j = 0; j < G::FN; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};

  // One slab: per half h, each lane reads its chunk 2 lg + h (k = 4 lg + 2 h,
  // +1) of every block and runs MFMA steps q = 2 h and 2 h + 1.
  auto mfma_stage = [&](int stage) {
    const double *sA = lds + stage * G::STAGE;
    const double *sB = sA + BM * BK;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      f64x2 a[G::FM], b[G::FN];
#pragma unroll
      for (int j = 0; j < G::FN; ++j) {
        const int n = wn0 + 16 * j + lr;
        b[j] = *reinterpret_cast<const f64x2 *>(sB + n * BK + (((2 * lg + h) ^ swz(n)) << 1));
      }
#pragma unroll
      for (int i = 0; i < G::FM; ++i) {
        const int r = wm0 + 16 * i + lr;
        a[i] = *reinterpret_cast<const f64x2 *>(sA + r * BK + (((2 * lg + h) ^ swz(r)) << 1));
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int i = 0; i < G::FM; ++i)
#pragma unroll
          for (int j = 0; j < G::FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][q], b[j][q], acc[i][j], 0, 0, 0);
    }
  };

  // Slab 0 of the first group is loaded masked in the prologue; the loads of the
  // loop, which takes two turns, lie inside [0, K).
  using Fast = std::integral_constant<int, kFast>;
  using Guarded = std::integral_constant<int, kGuarded>;
  using Masked = std::integral_constant<int, kMasked>;
  using R0 = std::integral_constant<int, 0>;
  using R1 = std::integral_constant<int, DEPTH - 1>;
  const Slabs sl(K, KG, group);
  const int KT = sl.turns, own = sl.own;
  if (group == 0) gload(Masked{}, R0{}, sl.base);
  else gload(Guarded{}, R0{}, sl.k(0));
  if (DEPTH == 2) gload(Guarded{}, R1{}, sl.k(1));
  sstore(R0{}, 0);
  __syncthreads();
  int t = 0;
  for (; t + 2 <= KT; t += 2) {
    gload(Fast{}, R0{}, sl.k(t + DEPTH));
    __builtin_amdgcn_sched_barrier(0);
    mfma_stage(0);
    sstore(R1{}, 1);
    __syncthreads();
    gload(Fast{}, R1{}, sl.k(t + 1 + DEPTH));
    __builtin_amdgcn_sched_barrier(0);
    if (KG == 1 || t + 1 < own) mfma_stage(1);
    sstore(R0{}, 0);
    __syncthreads();
  }
  if (t < KT && (KG == 1 || t < own)) mfma_stage(0);

  if constexpr (KG > 1) {
    double *part = lds - group * 2 * G::STAGE;
    __syncthreads();  // the last fragment reads
    if (group) {
#pragma unroll
      for (int i = 0; i < G::FM; ++i)
#pragma unroll
        for (int j = 0; j < G::FN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) part[((i * G::FN + j) * 4 + e) * NT + tid] = acc[i][j][e];
    }
    __syncthreads();
    if (group) return;
#pragma unroll
    for (int i = 0; i < G::FM; ++i)
#pragma unroll
      for (int j = 0; j < G::FN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][e] += part[((i * G::FN + j) * 4 + e) * NT + tid];
  }

  // Epilogue: element e of lane l is row lg + 4 e, column lr of its block.
  // With beta != 0 a row of blocks of C is read in one go, ahead of the stores
  // of the row before it: element by element each read waited for its
  // predecessor's store (1999 x 1501 x 1003 108 -> 103 us).
  auto inside = [&](int i, int j, int e) {
    return interior || (wn0 + 16 * j + lr < Nr && wm0 + 16 * i + lg + 4 * e < Mr);
  };
  double *const cp = C + (int64_t)(m0 + wm0 + lg) * ldc + (n0 + wn0 + lr);
  double cold[2][G::FN][4];
  auto cread = [&](int i) {
#pragma unroll
    for (int j = 0; j < G::FN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        cold[i & 1][j][e] = inside(i, j, e) ? cp[(int64_t)(16 * i + 4 * e) * ldc + 16 * j] : 0.0;
  };
  if (BETA) cread(0);
#pragma unroll
  for (int i = 0; i < G::FM; ++i) {
    if (BETA && i + 1 < G::FM) cread(i + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < G::FN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (inside(i, j, e)) {
          const double v = alpha * acc[i][j][e];
          cp[(int64_t)(16 * i + 4 * e) * ldc + 16 * j] = BETA ? fma(beta, cold[i & 1][j][e], v) : v;
        }
  }
}

// Grid: the output tiles of every problem of the batch (element strides sa, sb,
// sc between consecutive problems) in one XCD-aware order.
template <int BM, int BN, int WM, int WN, int KG, bool BETA>
__global__ __launch_bounds__((KG * Cfg<BM, BN, WM, WN>::NT), (Cfg<BM, BN, WM, WN>::MIN_WG)) void gemm_f64_kernel(
    int M, int N, int K, double alpha, const double *__restrict__ A, int64_t lda, int64_t sa,
    const double *__restrict__ B, int64_t ldb, int64_t sb, double beta, double *__restrict__ C,
    int64_t ldc, int64_t sc, int tiles_m, int tiles_n) {
  using G = Cfg<BM, BN, WM, WN>;
  __shared__ __attribute__((aligned(16))) double lds[KG * 2 * G::STAGE];
  const int tiles = tiles_m * tiles_n;
  const int wg = tiles > 1 ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int64_t b = wg / tiles;
  int tm, tn;
  tile_coords(wg - (int)b * tiles, tiles_m, tiles_n, 8, tm, tn);
  tile<BM, BN, WM, WN, KG, BETA>(M, N, K, alpha, A + b * sa, lda, B + b * sb, ldb, beta, C + b * sc,
                                  ldc, tm * BM, tn * BN, lds);
}

static bool tile_reaches(const GemmArgsF64 &g, int64_t bm) {
  const int64_t lim = ((int64_t)1 << 31) / 8;
  return std::min(bm, g.M) * g.lda + g.K < lim && std::min<int64_t>(BK, g.K) * g.ldb + g.N < lim;
}

template <int BM, int BN, int WM, int WN, int KG = 1>
gemm_status launch(const GemmArgsF64 &g, hipStream_t s) {
  using G = Cfg<BM, BN, WM, WN>;
  const int tiles_m = (int)((g.M + BM - 1) / BM);
  const int tiles_n = (int)((g.N + BN - 1) / BN);
  const int64_t nwg = (int64_t)tiles_m * tiles_n * g.batch;
  if (nwg > kMaxLanes / (KG * G::NT)) {
    set_error("gemm_f64: too many tiles or problems for one launch");
    return GEMM_STATUS_UNSUPPORTED;
  }
  if (!tile_reaches(g, BM)) {
    set_error("gemm_f64: lda or ldb too large for 32-bit tile offsets");
    return GEMM_STATUS_UNSUPPORTED;
  }
  const bool beta = g.beta != 0.0;
  const dim3 grid((unsigned)nwg), block(KG * G::NT);
#define MM_LAUNCH(BT)                                                                        \
  hipLaunchKernelGGL((gemm_f64_kernel<BM, BN, WM, WN, KG, BT>), grid, block, 0, s, (int)g.M,      \
                     (int)g.N, (int)g.K, g.alpha, g.A, g.lda, g.sa, g.B, g.ldb, g.sb, g.beta, g.C, \
                     g.ldc, g.sc, tiles_m, tiles_n)
  if (beta) MM_LAUNCH(true); else MM_LAUNCH(false);
#undef MM_LAUNCH
  return check_launch("gemm_f64_kernel");
}

// Batched small problems: one wave per 16 F x 16 F sub-tile of a problem, four
// waves per workgroup, the sub-tiles of a problem on consecutive waves.
// Operands go from memory straight into MFMA fragments (each element is used
// by few waves, so staging through LDS would only add traffic and barriers).
// The k range is walked in chunks of 16: lane group g takes four k of every
// block (two 128-bit loads of an A row when the chunk lies inside [0, K), else
// four 64-bit loads) and the four B values of its column at those k (64-bit
// loads, consecutive lanes on consecutive columns); MFMA step q multiplies the
// group's q-th k.  Rows past M and columns past N read zero through the buffer
// range check, k past K is masked per element, and memory instructions that no
// lane needs are skipped wave by wave.
// C stores are non-temporal (a cache hint): 32^3 x 29 297 134.2 -> 131.0 us.
constexpr int kStoreNT = 2;

template <int F, bool BETA>
__global__ __launch_bounds__(256, 2) void small_batched_kernel(
    int M, int N, int K, double alpha, const double *__restrict__ A, int64_t lda, int64_t sa,
    const double *__restrict__ B, int64_t ldb, int64_t sb, double beta, double *__restrict__ C,
    int64_t ldc, int64_t sc, int batch, int tiles_m, int tiles_n) {
  const int lane = threadIdx.x & 63;
  // the wave index is uniform across the wave; saying so keeps the problem's
  // buffer resources in scalar registers (no per-lane resource loops)
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int tiles = tiles_m * tiles_n;
  int prob = (int)blockIdx.x * 4 + wv, m0 = 0, n0 = 0;
  if (tiles > 1) {  // XCD-aware order where a problem spans workgroups: its panels meet in one L2
    const int unit = (tiles > 4 || tiles == 3 ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x) * 4 + wv;
    prob = unit / tiles;
    const int sub = unit - prob * tiles, tm = sub / tiles_n;
    m0 = tm * 16 * F;
    n0 = (sub - tm * tiles_n) * 16 * F;
  }
  if (prob >= batch) return;
  const int Mr = M - m0, Nr = N - n0;
  const int lr = lane & 15, lg = lane >> 4;
  const __amdgpu_buffer_rsrc_t rA =
      rsrc(A + prob * sa + m0 * lda, ((int64_t)(Mr - 1) * lda + K) * 8);
  const __amdgpu_buffer_rsrc_t rB = rsrc(B + prob * sb + n0, ((int64_t)(K - 1) * ldb + Nr) * 8);
  const __amdgpu_buffer_rsrc_t rC =
      rsrc(C + prob * sc + m0 * ldc + n0, ((int64_t)(Mr - 1) * ldc + Nr) * 8);
  int bcol[F], arow[F];
#pragma unroll
  for (int i = 0; i < F; ++i) {
    const int x = 16 * i + lr;
    bcol[i] = x < Nr ? x * 8 : (int)0x80000000;
    arow[i] = x < Mr ? x * (int)lda * 8 : (int)0x80000000;
  }
  const int ldb8 = (int)ldb * 8;
  f64x4 acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  double a[F][4], b[F][4];
  // lane group g takes k = k0 + 2g, +1 (q = 0, 1) and k0 + 8 + 2g, +1
  // (q = 2, 3): one 128-bit load of the four groups reads 64 contiguous
  // bytes of each A row
  auto load = [&](int k0) {
    auto kq = [&](int q) { return k0 + 2 * lg + (q & 1) + 8 * (q >> 1); };
    if (k0 + 16 <= K) {
#pragma unroll
      for (int i = 0; i < F; ++i) {
        const f64x2 v0 = ld2(rA, arow[i] + kq(0) * 8), v1 = ld2(rA, arow[i] + kq(2) * 8);
        a[i][0] = v0.x; a[i][1] = v0.y; a[i][2] = v1.x; a[i][3] = v1.y;
      }
#pragma unroll
      for (int j = 0; j < F; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) b[j][q] = ld1(rB, bcol[j] + kq(q) * ldb8, 0);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool any = k0 + (q & 1) + 8 * (q >> 1) < K;  // some lane group has a k here
        const bool kin = kq(q) < K;
#pragma unroll
        for (int i = 0; i < F; ++i)
          a[i][q] = any ? ld1(rA, kin ? arow[i] + kq(q) * 8 : (int)0x80000000, 0) : 0.0;
#pragma unroll
        for (int j = 0; j < F; ++j)
          b[j][q] = any ? ld1(rB, kin ? bcol[j] + kq(q) * ldb8 : (int)0x80000000, 0) : 0.0;
      }
    }
  };
  for (int k0 = 0; k0 < K; k0 += 16) {
    load(k0);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][q], b[j][q], acc[i][j], 0, 0, 0);
  }
  // element e of lane l is row lg + 4 e, column lr of its block; columns past
  // N get an out-of-range offset, rows past M fall beyond the resource.  With
  // beta != 0 every read of C is issued before the first store.
  const int ldc8 = (int)ldc * 8;
  int vb[F];
#pragma unroll
  for (int j = 0; j < F; ++j) {
    const int col = 16 * j + lr;
    vb[j] = col < Nr ? lg * ldc8 + col * 8 : (int)0x80000000;
  }
  double cold[F][F][4];
  if (BETA) {
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (16 * i + 4 * e < Mr) {
#pragma unroll
          for (int j = 0; j < F; ++j) cold[i][j][e] = ld1(rC, vb[j], (16 * i + 4 * e) * ldc8);
        }
  }
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (16 * i + 4 * e < Mr) {
#pragma unroll
        for (int j = 0; j < F; ++j) {
          double v = alpha * acc[i][j][e];
          if (BETA) v = fma(beta, cold[i][j][e], v);
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rC, vb[j],
                                                (16 * i + 4 * e) * ldc8, kStoreNT);
        }
      }
}

// 32-bit offsets of the small-problem kernel: M rows of A, K rows of B, the rows of
// C in whole groups of four (those past M are dropped by the range check).
static bool small_fits(const GemmArgsF64 &g) {
  const int64_t lim = (int64_t)1 << 31, rows = (g.M + 3) / 4 * 4;
  return (g.M * g.lda + g.K) * 8 < lim && (g.K * g.ldb + g.N) * 8 < lim &&
         (rows * g.ldc + g.N) * 8 < lim;
}

template <int F>
gemm_status launch_small(const GemmArgsF64 &g, hipStream_t s) {
  const int64_t tiles_m = (g.M + 16 * F - 1) / (16 * F), tiles_n = (g.N + 16 * F - 1) / (16 * F);
  const int64_t units = tiles_m * tiles_n * g.batch;
  if (units > kMaxLanes / 64) { set_error("gemm_f64: batch too large"); return GEMM_STATUS_UNSUPPORTED; }
#define MM_LAUNCH(BT)                                                                               \
  hipLaunchKernelGGL((small_batched_kernel<F, BT>), dim3((unsigned)((units + 3) / 4)),        \
                     dim3(256), 0, s, (int)g.M, (int)g.N, (int)g.K, g.alpha, g.A, g.lda, g.sa, g.B, \
                     g.ldb, g.sb, g.beta, g.C, g.ldc, g.sc, (int)g.batch, (int)tiles_m,             \
                     (int)tiles_n)
  if (g.beta != 0.0) MM_LAUNCH(true); else MM_LAUNCH(false);
#undef MM_LAUNCH
  return check_launch("small_batched_kernel");
}

// Products with too few output tiles to fill the machine: one 16 F x 16 F tile
// per workgroup of eight waves, each accumulating the whole tile over its own
// run of 16-deep chunks (two chunks of operands in flight per wave, straight
// from memory into MFMA fragments as in the batched kernel; no barrier in the
// k loop); the eight partial tiles are added in wave order through LDS.
// Bound: a wave's chain of loads while CUs are idle (0.5 us a chunk for F = 1,
// 1.45 for F = 2), the L2 beyond that (about 11 TB/s at 2048^3, where LDS tiles
// are 1.5 times as fast).  Against 64 x 64 tiles, us: 160 x 48 x 1888 84 -> 13,
// 32 x 2016 x 759 37 -> 7, 166 x 1036 x 1857 84 -> 24, 576 x 1136 x 1512 71 ->
// 51.  Three chunks in flight were no faster (13.6, 7.5; F = 2: 26, 56).
constexpr int KW = 8;

template <int F, bool BETA>
__global__ __launch_bounds__(64 * KW) void split_kernel(
    int M, int N, int K, double alpha, const double *__restrict__ A, int64_t lda, int64_t sa,
    const double *__restrict__ B, int64_t ldb, int64_t sb, double beta, double *__restrict__ C,
    int64_t ldc, int64_t sc, int tiles_m, int tiles_n) {
  constexpr int OUT = 16 * F * 16 * F;
  __shared__ double part[KW][OUT];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wg = xcd_remap(blockIdx.x, gridDim.x), tiles = tiles_m * tiles_n;
  const int64_t prob = wg / tiles;
  int tm, tn;
  tile_coords(wg - (int)prob * tiles, tiles_m, tiles_n, 8, tm, tn);
  const int m0 = tm * 16 * F, n0 = tn * 16 * F;
  const int Mr = M - m0, Nr = N - n0;
  const int lr = lane & 15, lg = lane >> 4;
  const __amdgpu_buffer_rsrc_t rA =
      rsrc(A + prob * sa + (int64_t)m0 * lda, ((int64_t)(Mr - 1) * lda + K) * 8);
  const __amdgpu_buffer_rsrc_t rB = rsrc(B + prob * sb + n0, ((int64_t)(K - 1) * ldb + Nr) * 8);
  // lane group g takes k = 2g, 2g + 1, 8 + 2g, 9 + 2g of a chunk; its part of
  // the offsets is fixed, the chunk's is wave-uniform
  const int ldb8 = (int)ldb * 8;
  int arow[F], bcol[F];
#pragma unroll
  for (int i = 0; i < F; ++i) {
    const int x = 16 * i + lr;
    arow[i] = x < Mr ? (x * (int)lda + 2 * lg) * 8 : (int)0x80000000;
    bcol[i] = x < Nr ? x * 8 + 2 * lg * ldb8 : (int)0x80000000;
  }
  f64x4 acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  // the chunk grid ends at K: only chunk 0 can be partial
  const int KC = (K + 15) / 16, kbase = K - 16 * KC;
  const int c0 = wave * KC / KW, c1 = (wave + 1) * KC / KW;
  double a[2][F][4], b[2][F][4];
  auto load = [&](auto S, int c) {
    constexpr int st = decltype(S)::value;
    // chunks past the wave's last are read again at an offset in range, unused
    const int k = kbase + 16 * (c < c1 ? c : c1 - 1), k0 = k > 0 ? k : 0;
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f64x2 v = __builtin_bit_cast(
            f64x2, __builtin_amdgcn_raw_buffer_load_b128(rA, arow[i], (k0 + 8 * h) * 8, 0));
        a[st][i][2 * h] = v.x;
        a[st][i][2 * h + 1] = v.y;
      }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int j = 0; j < F; ++j) b[st][j][q] = ld1(rB, bcol[j], (k0 + (q & 1) + 8 * (q >> 1)) * ldb8);
  };
  auto load_partial = [&]() {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = kbase + (q & 1) + 8 * (q >> 1);  // of lane group 0
      const bool in = k + 2 * lg >= 0;
#pragma unroll
      for (int i = 0; i < F; ++i)
        a[0][i][q] = ld1(rA, in && 16 * i + lr < Mr ? arow[i] + k * 8 : (int)0x80000000, 0);
      // (bcol alone may lie beyond 2^31 where K < 8; the sum does not)
#pragma unroll
      for (int j = 0; j < F; ++j)
        b[0][j][q] = ld1(rB, in && 16 * j + lr < Nr ? bcol[j] + k * ldb8 : (int)0x80000000, 0);
    }
  };
  auto multiply = [&](auto S) {
    constexpr int st = decltype(S)::value;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[st][i][q], b[st][j][q], acc[i][j], 0, 0, 0);
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  if (c0 < c1) {
    if (c0 == 0 && kbase < 0) load_partial();
    else load(S0{}, c0);
    for (int c = c0;;) {
      load(S1{}, c + 1);
      __builtin_amdgcn_sched_barrier(0);
      multiply(S0{});
      if (++c >= c1) break;
      load(S0{}, c + 1);
      __builtin_amdgcn_sched_barrier(0);
      multiply(S1{});
      if (++c >= c1) break;
    }
  }
  // element e of lane l is row lg + 4 e, column lr of its block
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[wave][((i * F + j) * 4 + e) * 64 + lane] = acc[i][j][e];
  double *const Cb = C + prob * sc + (int64_t)m0 * ldc + n0;
  double cold[(OUT + 64 * KW - 1) / (64 * KW)];
  auto at = [&](int idx, int &row, int &col) {
    const int blk = idx >> 8, e = (idx >> 6) & 3, l = idx & 63;
    row = 16 * (blk / F) + (l >> 4) + 4 * e;
    col = 16 * (blk % F) + (l & 15);
  };
  int row, col;
  if (BETA) {
#pragma unroll
    for (int x = 0; x * 64 * KW < OUT; ++x) {
      const int idx = x * 64 * KW + (int)threadIdx.x;
      at(idx, row, col);
      cold[x] = idx < OUT && row < Mr && col < Nr ? Cb[(int64_t)row * ldc + col] : 0.0;
    }
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x * 64 * KW < OUT; ++x) {
    const int idx = x * 64 * KW + (int)threadIdx.x;
    at(idx, row, col);
    if (idx < OUT && row < Mr && col < Nr) {
      double v = part[0][idx];
#pragma unroll
      for (int w = 1; w < KW; ++w) v += part[w][idx];
      v *= alpha;
      Cb[(int64_t)row * ldc + col] = BETA ? fma(beta, cold[x], v) : v;
    }
  }
}

template <int F>
gemm_status launch_split(const GemmArgsF64 &g, hipStream_t s) {
  const int64_t tiles_m = (g.M + 16 * F - 1) / (16 * F), tiles_n = (g.N + 16 * F - 1) / (16 * F);
  const int64_t units = tiles_m * tiles_n * g.batch;
  if (units > kMaxLanes / (64 * KW)) { set_error("gemm_f64: batch too large"); return GEMM_STATUS_UNSUPPORTED; }
#define MM_LAUNCH(BT)                                                                                \
  hipLaunchKernelGGL((split_kernel<F, BT>), dim3((unsigned)units), dim3(64 * KW), 0, s,        \
                     (int)g.M, (int)g.N, (int)g.K, g.alpha, g.A, g.lda, g.sa, g.B, g.ldb, g.sb,      \
                     g.beta, g.C, g.ldc, g.sc, (int)tiles_m, (int)tiles_n)
  if (g.beta != 0.0) MM_LAUNCH(true); else MM_LAUNCH(false);
#undef MM_LAUNCH
  return check_launch("split_kernel");
}

// C <- beta*C over a batch (alpha == 0 or K == 0).
template <bool BETA>
__global__ __launch_bounds__(256) void scale_kernel(int64_t M, int64_t N, double beta,
                                                    double *__restrict__ C, int64_t ldc,
                                                    int64_t sc) {
  double *Cb = C + (int64_t)blockIdx.y * sc;
  const int64_t total = M * N;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * 256) {
    const int64_t i = e / N, j = e - i * N;
    double *p = Cb + i * ldc + j;
    *p = BETA ? beta * *p : 0.0;
  }
}

}  // namespace f64

struct F64Config {
  TileConfig t;
};
static const F64Config kF64Configs[] = {
    {{128, 128, 16, "f64_128x128x16_4w64x64", 256}},
    {{256, 128, 16, "f64_256x128x16_8w64x64", 512}},
    {{64, 64, 16, "f64_64x64x16_4w32x32", 256}},
    // one wave per output tile, operands straight into MFMA fragments (as a
    // configuration: problems of one tile, M, N <= 16 / 32 / 64)
    {{16, 16, 16, "f64_small_16", 64}},
    {{32, 32, 16, "f64_small_32", 64}},
    {{64, 64, 16, "f64_small_64", 64}},
    // one tile per workgroup of 8 waves, its k range split over the waves
    {{16, 16, 16, "f64_16x16x16_8wk", 512}},
    {{32, 32, 16, "f64_32x32x16_8wk", 512}},
    // 64 x 64 tiles, the k range split between two groups of four waves
    {{64, 64, 16, "f64_64x64x16_2x4w32x32_kg2", 512}},
};

int f64_num_configs() { return (int)(sizeof(kF64Configs) / sizeof(kF64Configs[0])); }
const TileConfig &f64_config(int i) { return kF64Configs[i].t; }

// Sub-tile codes of a batch (beyond the configurations): one wave per 16 x 16,
// 32 x 32 or 64 x 64 outputs.
constexpr int kDirect16 = 100, kDirect32 = 101, kDirect64 = 102;

// The split kernels' modelled time in us (fitted on 33 products from 32 to 2048
// per dimension): the chain of one wave's chunks, or a cost per tile and per
// tile and chunk, whichever is longer.
static double split_time(int f, double tiles, double kc) {
  const double chain = std::ceil(kc / 8.0);
  return f == 1 ? std::max(1.5 + 0.5 * chain, 3.0 + tiles * (0.0022 + 0.00029 * kc))
                : std::max(1.5 + 1.45 * chain, 3.0 + tiles * (0.008 + 0.00073 * kc));
}

// A batch: the tile with the least modelled time beyond the operands' traffic
// (`fixed` ns per output tile, `step` ns per tile and 16 k, whole machine;
// fitted on 26 batches whose inputs change from call to call).   Against one wave per problem up to 64 x 64 and
// 128 x 128 LDS tiles beyond, us at beta = 0: 76 x 48 x 32 x 1134 36 -> 16, 9 x
// 112 x 48 x 770 33 -> 9, 159 x 112 x 64 x 429 52 -> 33, 96^3 x 700 58 -> 43.
static int f64_batch_config(int64_t M, int64_t N, int64_t K, int64_t batch) {
  // 64 x 64 per wave only for batches of nearly full 64 x 64 problems that
  // fill the machine (64^3 x 2000 41 us against 45 for 32 x 32)
  if (M > 48 && N > 48 && M <= 64 && N <= 64 && K >= 32 && batch >= 6 * (int64_t)num_cus())
    return kDirect64;
  struct Tile {
    int cfg, b, per_cu;
    double fixed, step;
  };
  constexpr Tile kTiles[] = {{kDirect16, 16, 20, 0.05, 0.22},
                             {kDirect32, 32, 12, 0.10, 0.45},
                             {2, 64, 3, 2.5, 1.30},
                             {0, 128, 2, 4.0, 6.0}};
  int best = 2;
  double best_cost = -1.0;
  for (const Tile &t : kTiles) {
    const bool lds = t.cfg < kDirect16;
    const double tiles = (double)((M + t.b - 1) / t.b) * (double)((N + t.b - 1) / t.b) * (double)batch;
    const double slots = (double)num_cus() * t.per_cu, r = tiles / slots;
    // the sub-tiles re-read their panels too often in problems beyond 256, and
    // three waves of an LDS tile idle in problems up to 32 x 32 (32 x 32 x 512
    // x 300 43 us, 32 with sub-tiles)
    if (lds ? M <= 32 && N <= 32 : M > 256 || N > 256) continue;
    if (lds && kF64Configs[t.cfg].t.per_launch(M, N) < 1) continue;
    // LDS tiles that do not fill the machine come one or two to a CU
    const double part = lds ? 0.58 + 0.42 * std::ceil(r * t.per_cu) / t.per_cu : 0.7 + 0.3 * r;
    const double rounds = r > 4.0 ? r : r >= 1.0 ? std::ceil(r) : part;
    const double cost = rounds * slots * (t.fixed + t.step * (double)((K + 15) / 16));
    if (best_cost < 0.0 || cost < best_cost) { best = t.cfg; best_cost = cost; }
  }
  // few long problems: the k range split over a workgroup's waves (64 x 64 x 512
  // x 100 26 -> 19 us, 64 x 64 x 256 x 50 15 -> 7.5)
  for (int f = 1; f <= 2; ++f) {
    const int b = 16 * f;
    const double tiles = (double)((M + b - 1) / b) * (double)((N + b - 1) / b) * (double)batch;
    const double cost = 1e3 * (2.0 + split_time(f, tiles, (double)((K + 15) / 16)));
    if (cost < best_cost) { best = 5 + f; best_cost = cost; }
  }
  return best;
}

int f64_default_config(int64_t M, int64_t N, int64_t K, int64_t batch) {
  if (batch > 1) return f64_batch_config(M, N, K, batch);
  // 128 x 128 tiles once there are two per CU.  Measured on one box: the kernel
  // is matrix-core bound and the tiles tie within 1 % at 4096^3, but 64 x 64
  // tiles read 10x the minimum HBM bytes there (5.3 against 1.9 GB per launch),
  // which costs clock under the power limit; at 2048^3 (one 128 x 128 tile per
  // CU) 64 x 64 tiles are 11 % faster.
  const double cus = num_cus();
  auto tiles = [&](int b) { return (double)((M + b - 1) / b) * (double)((N + b - 1) / b); };
  if (tiles(128) >= 2 * cus) return 0;
  // Below that the least modelled time in us.  64 x 64 tiles: a CU with n of
  // them takes 0.25 + 0.46 n per slab (the matrix cores' own time is 0.48 n);
  // the two-group form where n is 1.
  const double kc = (double)((K + 15) / 16), r = tiles(64) / cus, n = std::ceil(r);
  const struct { int cfg; double us; } c[] = {
      {2, 3.5 + kc * (n <= 1.0 ? 0.71 : n <= 4.0 ? 0.25 + 0.46 * n : 0.5 * r)},
      {8, n <= 1.0 ? 4.5 + 0.6 * kc : 1e30},
      {6, split_time(1, tiles(16), kc)},
      {7, split_time(2, tiles(32), kc)}};
  int best = 0;
  for (int i = 1; i < 4; ++i)
    if (c[i].us < c[best].us) best = i;
  return c[best].cfg;
}

static gemm_status f64_launch(const GemmArgsF64 &g, int cfg, hipStream_t s) {
  switch (cfg) {
    case 0: return f64::launch<128, 128, 64, 64>(g, s);
    case 1: return f64::launch<256, 128, 64, 64>(g, s);
    case 2: return f64::launch<64, 64, 32, 32>(g, s);
    case 6: return f64::launch_split<1>(g, s);
    case 7: return f64::launch_split<2>(g, s);
    case 8: return f64::launch<64, 64, 32, 32, 2>(g, s);
    case kDirect16: return f64::launch_small<1>(g, s);
    case kDirect32: return f64::launch_small<2>(g, s);
    case kDirect64: return f64::launch_small<4>(g, s);
    default: set_error("gemm_f64: bad tile config"); return GEMM_STATUS_UNSUPPORTED;
  }
}

gemm_status f64_run(const GemmArgsF64 &g, int cfg, bool batched, hipStream_t s) {
  if (cfg >= 3 && cfg <= 5) {
    const int lim = cfg == 3 ? 16 : cfg == 4 ? 32 : 64;
    if (g.M > lim || g.N > lim) {
      set_error("gemm_f64: problem larger than the small-problem configuration");
      return GEMM_STATUS_UNSUPPORTED;
    }
    cfg = kDirect16 + (cfg - 3);
  }
  if (cfg >= kDirect16) {
    const int lim = cfg == kDirect16 ? 16 : cfg == kDirect32 ? 32 : 64;
    if (g.M <= 64 && g.N <= 64 &&
        ((lim * g.lda + g.K) * 8 >= ((int64_t)1 << 31) || (g.K * g.ldb + g.N) * 8 >= ((int64_t)1 << 31))) {
      set_error("gemm_f64: lda or ldb too large for 32-bit offsets of the small-problem kernel");
      return GEMM_STATUS_UNSUPPORTED;
    }
  }
  // other operands that 32-bit offsets cannot reach take the 64 x 64 tile, whose
  // panels are the smallest (so do those of a batch, whose rule may take 128 x 128
  // tiles for few problems)
  if ((cfg >= kDirect16 || cfg == 6 || cfg == 7) && !f64::small_fits(g)) cfg = 2;
  if (cfg == 0 && batched && !f64::tile_reaches(g, 128)) cfg = 2;
  // as many problems to a launch as its lanes allow
  const int tile = cfg >= kDirect16 ? cfg - kDirect16 + 3 : cfg;
  if (tile < 0 || tile >= f64_num_configs()) {
    set_error("gemm_f64: bad tile config");
    return GEMM_STATUS_UNSUPPORTED;
  }
  const int64_t most = std::max<int64_t>(1, kF64Configs[tile].t.per_launch(g.M, g.N));
  for (int64_t b = 0; b < g.batch; b += most) {
    GemmArgsF64 part = g;
    part.A += b * g.sa;
    part.B += b * g.sb;
    part.C += b * g.sc;
    part.batch = std::min(most, g.batch - b);
    if (gemm_status st = f64_launch(part, cfg, s)) return st;
  }
  return GEMM_STATUS_OK;
}

gemm_status scale_c_f64(int64_t M, int64_t N, double beta, double *C, int64_t ldc, int64_t sc,
                        int64_t batch, hipStream_t s) {
  const int64_t want = (M * N + 255) / 256;
  const unsigned gx = (unsigned)(want < 4096 ? (want > 0 ? want : 1) : 4096);
  const dim3 grid(gx, (unsigned)batch);
  if (beta != 0.0)
    hipLaunchKernelGGL(f64::scale_kernel<true>, grid, dim3(256), 0, s, M, N, beta, C, ldc, sc);
  else
    hipLaunchKernelGGL(f64::scale_kernel<false>, grid, dim3(256), 0, s, M, N, beta, C, ldc, sc);
  return check_launch("scale_kernel_f64");
}

}  // namespace mm
