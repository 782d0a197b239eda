// k_small.hip -- products too small to fill the machine with output tiles.
//
// One BM x BN output tile per workgroup of KW waves.  The tile's k range is
// cut into KW consecutive ranges of whole chunks, one per wave: every wave
// accumulates the whole tile over its own range on the matrix cores, with its
// own loads (a wave touches each element it loads once; nothing is shared
// between waves, so the k loop has no barrier).  The KW partial tiles are then
// summed in wave order through LDS and the epilogue applies alpha
// and beta.  This is the k-reduction of the matrix product split into
// independent partial reductions whose write conflict on C is resolved by a
// sum (Sec. 3.3, write-conflict resolution; App. A, the wcr attribute), here
// an ordered sum inside the workgroup: deterministic for a given shape and
// configuration, no workspace, one launch.
//
// Three arithmetic modes share the kernel:
//   NP == 1  binary32 products on v_mfma_f32_32x32x2f32 (the plain path);
//   NP == 2  the split-precision path, 3 bf16 products (a0b0 + a0b1 + a1b0);
//   NP == 3  the split-precision path, 6 bf16 products.
// TA / TB: A stored K x M / B stored N x K (op(A) = A^T, op(B) = B^T).
#include "bf16x3.hpp"
#include "common.hpp"
#include "kernels.hpp"

namespace mm {
namespace small {

using bx3::bf16x2;
using bx3::f32x2;
using bx3::kBufferFlags;

constexpr int KW = 8;  // waves per workgroup (k ranges per output tile)

// One operand of a wave: NF blocks of 32 rows of op(A) (columns of op(B)), CK
// k per chunk (the unit of loading), SETS chunks of loads in flight, E
// consecutive k per lane and MFMA k-step (a k-step is 2E deep: lanes 0-31 hold
// its first E k, lanes 32-63 the others).  A row index outside the matrix reads
// as zero: its lane offset lies beyond the resource.  Lane offsets are fixed
// for the whole product and the chunk moves in the wave-uniform offset, so a
// chunk costs no vector address arithmetic.  How it is read:
enum class Read {
  // row index contiguous in memory (row-major B, transposed A): one 32-bit
  // load per k, consecutive lanes on consecutive addresses
  kRows,
  // k contiguous (row-major A, transposed B): 128-bit loads, at any alignment,
  // each lane from its own row
  kDirect,
  // k contiguous, long products: a direct read touches 32 rows per
  // instruction, which the L1 serves one row at a time.  Instead consecutive
  // lanes read consecutive 16-byte pieces of a row (CK k per row: 8 or 4
  // lanes), and the wave turns the chunk through an LDS area of its own
  // (pieces XOR-swizzled by the row; no barrier: one wave's LDS instructions
  // execute in order)
  kStaged,
};

template <Read R, int NF, int CK, int SETS, int E>
struct Operand;

template <int NF, int CK, int SETS, int E>
struct Operand<Read::kStaged, NF, CK, SETS, E> {
  static constexpr int NI = NF * CK / 8;        // 128-bit loads per chunk
  static constexpr int LPR = CK / 4;            // lanes (16-byte pieces) per row
  static constexpr int LDS_FLOATS = NF * 32 * CK;
  __amdgpu_buffer_rsrc_t rs;
  int voff[NI];
  f32x4 raw[SETS][NI];
  float *lds;
  int lane;
  __device__ static __forceinline__ int swz(int r) { return LPR == 8 ? r & 7 : (r >> 1) & 3; }
  __device__ __forceinline__ int row(int j) const { return j * (64 / LPR) + lane / LPR; }
  __device__ __forceinline__ void init(const float *P, int bytes, int ld, int i0, int lim, int lane_,
                                       float *lds_) {
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(P), (short)0, bytes, kBufferFlags);
    lane = lane_;
    lds = lds_;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int i = i0 + row(j);
      voff[j] = i < lim ? (int)(((unsigned)i * (unsigned)ld + (lane % LPR) * 4) * 4u) : (int)0x80000000;
    }
  }
  template <int S>
  __device__ __forceinline__ void load(int k0) {
#pragma unroll
    for (int j = 0; j < NI; ++j)
      raw[S][j] = __builtin_bit_cast(
          f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff[j], k0 * 4, 0));
  }
  // the chunk that begins before k = 0
  template <int S>
  __device__ __forceinline__ void load_masked(int k0) {
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = voff[j] >= 0 && k0 + (lane % LPR) * 4 + e >= 0;
        const int off = in ? voff[j] + (k0 + e) * 4 : (int)0x80000000;
        raw[S][j][e] =
            __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
      }
  }
  template <int S>
  __device__ __forceinline__ void stage() {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int r = row(j);
      *reinterpret_cast<f32x4 *>(lds + r * CK + (((lane % LPR) ^ swz(r)) << 2)) = raw[S][j];
    }
  }
  template <int S>
  __device__ __forceinline__ void frag(float (&v)[NF][E], int u) const {
    const int lr = lane & 31, lg = lane >> 5;
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int q = 0; q < E / 4; ++q) {
        const int r = 32 * i + lr;
        const f32x4 x = *reinterpret_cast<const f32x4 *>(
            lds + r * CK + ((((2 * u + lg) * (E / 4) + q) ^ swz(r)) << 2));
        v[i][4 * q] = x.x; v[i][4 * q + 1] = x.y; v[i][4 * q + 2] = x.z; v[i][4 * q + 3] = x.w;
      }
  }
};

template <int NF, int CK, int SETS, int E>
struct Operand<Read::kRows, NF, CK, SETS, E> {
  static constexpr int LDS_FLOATS = 0;
  __amdgpu_buffer_rsrc_t rs;
  int voff[NF];
  float raw[SETS][NF][CK / 2];  // element x: k-step x / E, k x % E of the lane's E
  int ld, lg;
  __device__ __forceinline__ void init(const float *P, int bytes, int ld_, int i0, int lim, int lane,
                                       float *) {
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(P), (short)0, bytes, kBufferFlags);
    ld = ld_;
    lg = lane >> 5;
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      const int n = i0 + 32 * i + (lane & 31);
      voff[i] = n < lim ? n * 4 : (int)0x80000000;
    }
  }
  template <int S>
  __device__ __forceinline__ void load(int k0) {
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      const int off = voff[i] + lg * E * ld * 4;
#pragma unroll
      for (int x = 0; x < CK / 2; ++x)
        raw[S][i][x] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                     rs, off, (k0 + x / E * 2 * E + x % E) * ld * 4, 0));
    }
  }
  template <int S>
  __device__ __forceinline__ void load_masked(int k0) {
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int x = 0; x < CK / 2; ++x) {
        const int k = k0 + x / E * 2 * E + lg * E + x % E;
        const int off = voff[i] >= 0 && k >= 0 ? voff[i] + k * ld * 4 : (int)0x80000000;
        raw[S][i][x] =
            __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
      }
  }
  template <int S>
  __device__ __forceinline__ void stage() {}
  template <int S>
  __device__ __forceinline__ void frag(float (&v)[NF][E], int u) const {
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int e = 0; e < E; ++e) v[i][e] = raw[S][i][u * E + e];
  }
};

template <int NF, int CK, int SETS, int E>
struct Operand<Read::kDirect, NF, CK, SETS, E> {
  static constexpr int LDS_FLOATS = 0;
  __amdgpu_buffer_rsrc_t rs;
  int voff[NF];
  float raw[SETS][NF][CK / 2];
  int lg;
  __device__ __forceinline__ void init(const float *P, int bytes, int ld, int i0, int lim, int lane,
                                       float *) {
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(P), (short)0, bytes, kBufferFlags);
    lg = lane >> 5;
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      const int m = i0 + 32 * i + (lane & 31);
      voff[i] = m < lim ? (int)(((unsigned)m * (unsigned)ld + lg * E) * 4u) : (int)0x80000000;
    }
  }
  template <int S>
  __device__ __forceinline__ void load(int k0) {
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int q = 0; q < CK / 8; ++q) {
        const float4 x = __builtin_bit_cast(
            float4, __builtin_amdgcn_raw_buffer_load_b128(
                        rs, voff[i], (k0 + 4 * q / E * 2 * E + 4 * q % E) * 4, 0));
        raw[S][i][4 * q + 0] = x.x; raw[S][i][4 * q + 1] = x.y;
        raw[S][i][4 * q + 2] = x.z; raw[S][i][4 * q + 3] = x.w;
      }
  }
  template <int S>
  __device__ __forceinline__ void load_masked(int k0) {
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int x = 0; x < CK / 2; ++x) {
        const int kr = k0 + x / E * 2 * E + x % E;  // the k of lane group 0
        const int off = voff[i] >= 0 && kr + lg * E >= 0 ? voff[i] + kr * 4 : (int)0x80000000;
        raw[S][i][x] =
            __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
      }
  }
  template <int S>
  __device__ __forceinline__ void stage() {}
  template <int S>
  __device__ __forceinline__ void frag(float (&v)[NF][E], int u) const {
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int e = 0; e < E; ++e) v[i][e] = raw[S][i][u * E + e];
  }
};

template <int NP>
constexpr int kE = NP == 1 ? 4 : 8;

// k per chunk: one MFMA k-step, or staged 32 (16 for 64 x 64 tiles, whose
// blocks need the registers).
template <int BM, int NP>
constexpr int chunk_k(bool staged) {
  return staged ? (BM == 32 ? 32 : 16) : 2 * kE<NP>;
}

// Bound: a wave's chain of chunks (two to four waves per SIMD), each wanting
// its loads to arrive and its share of the L1's address rate; SETS - 1 chunks
// of loads are in flight while one is multiplied.
// FEW: row-major A of at most eight rows is read directly also where B is staged: its
// rows are few enough for the L1, and turning them through LDS is a detour.
template <int BM, int BN, int NP, bool STAGED, bool FEW, bool TA, bool TB, bool BETA>
__global__ __launch_bounds__(64 * KW) void gemm_small_kernel(
    int M, int N, int K, float alpha, const float *__restrict__ A, int lda, int bytes_a,
    const float *__restrict__ B, int ldb, int bytes_b, float beta, float *__restrict__ C,
    int64_t ldc, int tiles_m, int tiles_n, bool deal) {
  constexpr int FM = BM / 32, FN = BN / 32;
  constexpr int E = kE<NP>;
  constexpr int CK = chunk_k<BM, NP>(STAGED);
  constexpr int KS = CK / (2 * E);              // MFMA k-steps per chunk
  constexpr int SETS = STAGED ? (BM == 32 ? 2 : 3) : (FM * CK > 16 ? 3 : 4);
  constexpr int BLK = 16 * 64;  // floats of one 32 x 32 accumulator block
  constexpr Read kc = STAGED ? Read::kStaged : Read::kDirect;
  using OpA = Operand<TA ? Read::kRows : FEW ? Read::kDirect : kc, FM, CK, SETS, E>;
  using OpB = Operand<TB ? kc : Read::kRows, FN, CK, SETS, E>;
  constexpr int TOT = FM * FN * BLK;            // floats of a partial tile
  constexpr int STG = OpA::LDS_FLOATS + OpB::LDS_FLOATS;
  constexpr int PERW = TOT > STG ? TOT : STG;   // a wave's LDS: staging, then its partial tile
  __shared__ __attribute__((aligned(16))) float smem[KW * PERW];

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // XCD-aware order, groups of 8 tile rows walked down a column of tiles: the
  // tiles that share an operand panel, and the cache lines that unaligned
  // neighbours have in common, meet in one L2 (900^2 x 3000 73 -> 58 us in
  // binary32, 48 x 2993 x 5248 38 -> 25).  `deal`: the columns of tiles go to
  // the XCDs one by one instead -- rows of B that lie a multiple of 4 KB apart
  // put the 8-column run of one XCD on few of its L2 channels (64 x 4096 x
  // 4096 19.4 us in runs, 17.2 dealt).
  int tm, tn;
  const int w0 = blockIdx.x, dealt = tiles_n / 8 * 8;
  if (deal && w0 < dealt * tiles_m) {
    const int c = (w0 >> 3) / tiles_m;
    tm = (w0 >> 3) - c * tiles_m;
    tn = c * 8 + (w0 & 7);
  } else if (deal) {
    const int r = w0 - dealt * tiles_m;
    tm = r % tiles_m;
    tn = dealt + r / tiles_m;
  } else {
    tile_coords(xcd_remap(w0, gridDim.x), tiles_m, tiles_n, 8, tm, tn);
  }
  const int m0 = tm * BM, n0 = tn * BN;
  OpA opa;
  OpB opb;
  opa.init(A, bytes_a, lda, m0, M, lane, smem + w * PERW);
  opb.init(B, bytes_b, ldb, n0, N, lane, smem + w * PERW + OpA::LDS_FLOATS);

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  // the grid of chunks ends at K: only chunk 0 can be partial
  const int total = (K + CK - 1) / CK;
  const int kbase = K - total * CK;
  // equal ranges to within a chunk (whole multiples would leave the last wave
  // short and the other sums longer)
  const int c0 = (int)((int64_t)w * total / KW);
  const int n = (int)((int64_t)(w + 1) * total / KW) - c0;

  auto load = [&](auto SET, int c) {
    constexpr int S = decltype(SET)::value;
    const int k0 = kbase + c * CK;
    opa.template load<S>(k0);
    opb.template load<S>(k0);
  };
  auto load_masked = [&](auto SET) {
    constexpr int S = decltype(SET)::value;
    opa.template load_masked<S>(kbase);
    opb.template load_masked<S>(kbase);
  };
  auto multiply = [&](auto SET) {
    constexpr int S = decltype(SET)::value;
    if constexpr (STG > 0) {
      // the previous chunk's reads are done before its area is rewritten, and
      // this chunk's writes before its reads (order within the wave)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      opa.template stage<S>();
      opb.template stage<S>();
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
#pragma unroll
    for (int u = 0; u < KS; ++u) {
      float fa[FM][E], fb[FN][E];
      opa.template frag<S>(fa, u);
      opb.template frag<S>(fb, u);
      if constexpr (NP == 1) {
        // MFMA q sums k = q of the lower half-wave's four and of the upper
        // half-wave's four: every k of the step exactly once
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
              acc[i][j] =
                  __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][q], fb[j][q], acc[i][j], 0, 0, 0);
      } else {
        bf16x8 a[NP][FM], b[NP][FN];
        // split of E = 8 binary32 values into NP bf16 planes, two at a time
        auto split8 = [&](const float (&x)[E], bf16x8 &p0, bf16x8 &p1, bf16x8 &p2) {
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            bf16x2 x0, x1, x2;
            if constexpr (NP == 2) bx3::split2(f32x2{x[e], x[e + 1]}, x0, x1);
            else bx3::split3(f32x2{x[e], x[e + 1]}, x0, x1, x2);
            p0[e] = x0.x; p0[e + 1] = x0.y;
            p1[e] = x1.x; p1[e + 1] = x1.y;
            if constexpr (NP == 3) { p2[e] = x2.x; p2[e + 1] = x2.y; }
          }
        };
#pragma unroll
        for (int i = 0; i < FM; ++i) split8(fa[i], a[0][i], a[1][i], a[NP - 1][i]);
#pragma unroll
        for (int j = 0; j < FN; ++j) split8(fb[j], b[0][j], b[1][j], b[NP - 1][j]);
        auto prod = [&](int qa, int qb) {
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[qa][i], b[qb][j], acc[i][j],
                                                                  0, 0, 0);
        };
        // small products first, the leading product last
        if constexpr (NP == 3) {
          prod(2, 0);
          prod(1, 1);
          prod(0, 2);
        }
        prod(1, 0);
        prod(0, 1);
        prod(0, 0);
      }
    }
  };

  if (n > 0) {
    if (c0 == 0 && kbase < 0) load_masked(std::integral_constant<int, 0>{});
    else load(std::integral_constant<int, 0>{}, c0);
    bx3::static_for<SETS - 2>([&](auto I) {
      constexpr int i = decltype(I)::value + 1;
      if (i < n) load(std::integral_constant<int, i>{}, c0 + i);
    });
    for (int s = 0; s < n; s += SETS)
      bx3::static_for<SETS>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if (s + i < n) {
          if (s + i + SETS - 1 < n)
            load(std::integral_constant<int, (i + SETS - 1) % SETS>{}, c0 + s + i + SETS - 1);
          multiply(I);
        }
      });
  }

  // partial tiles to LDS (lane-contiguous: no bank conflicts; each wave's own
  // area, after its staging), then the ordered sum over the waves and the
  // epilogue (every read of C before the first store)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        smem[w * PERW + (i * FN + j) * BLK + e * 64 + lane] = acc[i][j][e];
  constexpr int PER = TOT / (64 * KW);
  float cold[PER];
  float *p[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int idx = tid + r * 64 * KW;
    const int l = idx & 63, e = (idx >> 6) & 15, blk = idx >> 10;
    const int row = m0 + (blk / FN) * 32 + 8 * (e >> 2) + 4 * (l >> 5) + (e & 3);
    const int col = n0 + (blk % FN) * 32 + (l & 31);
    p[r] = row < M && col < N ? C + (int64_t)row * ldc + col : nullptr;
    if (BETA) cold[r] = p[r] ? *p[r] : 0.0f;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int idx = tid + r * 64 * KW;
    float s = smem[idx];
#pragma unroll
    for (int v = 1; v < KW; ++v) s += smem[v * PERW + idx];
    const float v = alpha * s;
    if (p[r]) *p[r] = BETA ? fmaf(beta, cold[r], v) : v;
  }
}

// Byte extent of a stored operand (rows x row stride, the last row cut at
// cols); the kernel addresses it with 32-bit offsets from its base.
static inline int64_t extent_bytes(int64_t rows, int64_t ld, int64_t cols) {
  return rows <= 0 || cols <= 0 ? 0 : ((rows - 1) * ld + cols) * 4;
}

template <int BM, int BN, int NP>
gemm_status launch(const GemmArgs &g, hipStream_t s) {
  const int64_t tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const int64_t ea = g.ta ? extent_bytes(g.K, g.lda, g.M) : extent_bytes(g.M, g.lda, g.K);
  const int64_t eb = g.tb ? extent_bytes(g.N, g.ldb, g.K) : extent_bytes(g.K, g.ldb, g.N);
  // every element offset (and the out-of-range marker) must fit in 31 bits
  if (tiles_m * tiles_n > kMaxLanes / (64 * KW) || ea >= ((int64_t)1 << 31) || eb >= ((int64_t)1 << 31)) {
    set_error("small-product configuration: operands too large for 32-bit offsets or one launch");
    return GEMM_STATUS_UNSUPPORTED;
  }
  // Staged where a wave's range is long (direct -> staged, us): 32 x 32 tiles
  // NN K 3761 16.1 -> 12.6, 1500 12.2 -> 11.1, 1100 8.8 -> 8.2, 349 8.1 -> 10.1;
  // TT K 1440 11.0 -> 9.7, 571 13.7 -> 14.4; 64 x 64 tiles K 3712 84 -> 75, 1500
  // 24.4 -> 23.6.  The rule looks at K alone: the ranges of the waves, and with
  // them the bits of the result, are the same for every transpose flag (TN,
  // which has nothing to turn, takes the same chunks).
  const bool staged = g.K >= 1024;
  // (the same ranges with A read directly: 3 x 6816 x 1920 10.9 -> 10.6 us, 1 x 4000 x 1500 7.5
  // -> 7.1; at sixteen rows 11.3 -> 11.5, 7.9 -> 8.3)
  const bool few = BM == 32 && staged && !g.ta && g.M <= 8;
  const bool deal = tiles_m <= 8 && !g.tb && g.ldb % 1024 == 0;
  const bool beta = g.beta != 0.0f;
  const dim3 grid((unsigned)(tiles_m * tiles_n)), block(64 * KW);
#define MM_SMALL(ST, FEW, TA, TB, BT)                                                             \
  hipLaunchKernelGGL((gemm_small_kernel<BM, BN, NP, ST, FEW, TA, TB, BT>), grid, block, 0, s,     \
                     (int)g.M, (int)g.N, (int)g.K, g.alpha, g.A, (int)g.lda, (int)ea, g.B,         \
                     (int)g.ldb, (int)eb, g.beta, g.C, g.ldc, (int)tiles_m, (int)tiles_n, deal)
#define MM_SMALL_BETA(ST, FEW, TA, TB) \
  do { if (beta) MM_SMALL(ST, FEW, TA, TB, true); else MM_SMALL(ST, FEW, TA, TB, false); } while (0)
#define MM_SMALL_ST(TA, TB)                                       \
  do {                                                            \
    if (few) MM_SMALL_BETA(true, (BM == 32 && !TA), TA, TB);      \
    else if (staged) MM_SMALL_BETA(true, false, TA, TB);          \
    else MM_SMALL_BETA(false, false, TA, TB);                     \
  } while (0)
  if (g.ta) { if (g.tb) MM_SMALL_ST(true, true); else MM_SMALL_ST(true, false); }
  else      { if (g.tb) MM_SMALL_ST(false, true); else MM_SMALL_ST(false, false); }
#undef MM_SMALL_ST
#undef MM_SMALL_BETA
#undef MM_SMALL
  return check_launch("gemm_small_kernel");
}

}  // namespace small

// which: 0 = 32 x 32 tiles, 1 = 64 x 64 tiles; np: 1 (binary32), 2 or 3
// (bf16 planes per operand).
gemm_status small_run(const GemmArgs &g, int which, int np, hipStream_t s) {
  if (np == 1) return which == 0 ? small::launch<32, 32, 1>(g, s) : small::launch<64, 64, 1>(g, s);
  if (np == 2) return which == 0 ? small::launch<32, 32, 2>(g, s) : small::launch<64, 64, 2>(g, s);
  return which == 0 ? small::launch<32, 32, 3>(g, s) : small::launch<64, 64, 3>(g, s);
}

}  // namespace mm
