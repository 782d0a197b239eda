// k_bf16x3.hip -- FP32-accurate split-precision GEMM on bf16 MFMA (gfx950).
#include <algorithm>
#include <cmath>

#include "bx3_launch.hpp"

namespace mm {
namespace bx3 {

// ---- split-K ----------------------------------------------------------------
// Workgroup (chunk c, output tile) multiplies K range [c*chunk, min(K, (c+1)*chunk))
// of its tile (alpha 1, beta 0) into partial plane c of P (M x N, ld N).
// Chunks are whole units of 16 k (32 with six products), whatever the tile: the
// slab grid of every chunk ends on its own boundary, only a chunk's first slab
// can be partial, and every tile gives the same partial products.
template <int BM, int BN, int BK, int WM, int WN, int NP, int NW>
__global__ __launch_bounds__(64 * NW, 1) void gemm_bx3_splitk_kernel(
    int M, int N, int K, int chunk, const float *__restrict__ A, int64_t lda,
    const float *__restrict__ B, int64_t ldb, float *__restrict__ P, int tiles_m, int tiles_n) {
  using G = Cfg<BM, BN, BK, WM, WN, NP, NW>;
  __shared__ __attribute__((aligned(16))) __bf16 lds[G::LDS_BYTES / 2];
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  const int tiles = tiles_m * tiles_n;
  const int c = wg / tiles;
  int tm, tn;
  tile_coords(wg - c * tiles, tiles_m, tiles_n, 8, tm, tn);
  const int k0 = c * chunk;
  const int kc = (K - k0 < chunk ? K - k0 : chunk);
  tile<BM, BN, BK, WM, WN, NP, NW, false>(M, N, kc, 1.0f, A + k0, lda, B + (int64_t)k0 * ldb,
                                               ldb, 0.0f, P + (int64_t)c * M * N, N, tm * BM,
                                               tn * BN, lds);
}

// P_0 + P_1 + ... of element q, in plane order.  AHEAD: eight planes are read
// ahead of their additions, for reductions whose chain of S dependent reads is the
// time, and no plane is read twice (us, in turn -> eight ahead: 57 x 1856 x 6046 in
// 23 chunks 23.2 -> 17.3, 64 x 4096 x 4096 in 16 23.4 -> 20.7; 2048 x 2048 x 512 in two
// chunks 28.5, 29.2 when a short group repeated its last plane).  In turn where
// 128-bit reads of four or more workgroups per CU keep the memory busy: 256 x 4096 x
// 2048 in eight 27.3, 28.0 eight ahead, 512 x 4096 x 4096 in nine 86.8, 88.9.
template <typename V>
__device__ __forceinline__ V sum_planes(const V *P, int64_t plane, int S, int64_t q, bool ahead) {
  V acc = P[q];
  int c = 1;
  auto add = [&](auto n) {
    constexpr int kN = decltype(n)::value;
    V v[kN];
#pragma unroll
    for (int u = 0; u < kN; ++u) v[u] = P[(c + u) * plane + q];
#pragma unroll
    for (int u = 0; u < kN; ++u) acc += v[u];
    c += kN;
  };
  if (!ahead) {
    while (c < S) add(std::integral_constant<int, 1>{});
    return acc;
  }
  while (c + 8 <= S) add(std::integral_constant<int, 8>{});
  switch (S - c) {
    case 7: add(std::integral_constant<int, 7>{}); break;
    case 6: add(std::integral_constant<int, 6>{}); break;
    case 5: add(std::integral_constant<int, 5>{}); break;
    case 4: add(std::integral_constant<int, 4>{}); break;
    case 3: add(std::integral_constant<int, 3>{}); break;
    case 2: add(std::integral_constant<int, 2>{}); break;
    case 1: add(std::integral_constant<int, 1>{}); break;
    default: break;
  }
  return acc;
}

// The write-conflict resolution of the chunks: C = alpha * (P_0 + P_1 + ...)
// + beta * C, summed in chunk order (deterministic), the same epilogue
// arithmetic as the single-pass kernel.  VEC: N, ldc multiples of 4 and C 16-byte
// aligned.
template <bool VEC, bool BETA>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(int M, int N, int S,
                                                            const float *__restrict__ P,
                                                            float alpha, float beta,
                                                            float *__restrict__ C, int64_t ldc) {
  const int64_t plane = (int64_t)M * N;
  if (VEC) {
    const int64_t n4 = plane / 4;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < n4; q += (int64_t)gridDim.x * 256) {
      const f32x4 acc = sum_planes(reinterpret_cast<const f32x4 *>(P), n4, S, q, gridDim.x < 1024);
      const int64_t e = 4 * q;
      const int64_t i = e / N, j = e - i * N;
      float4 *cp = reinterpret_cast<float4 *>(C + i * ldc + j);
      float4 out = make_float4(alpha * acc.x, alpha * acc.y, alpha * acc.z, alpha * acc.w);
      if (BETA) {
        const float4 c0 = *cp;
        out = make_float4(fmaf(beta, c0.x, out.x), fmaf(beta, c0.y, out.y),
                          fmaf(beta, c0.z, out.z), fmaf(beta, c0.w, out.w));
      }
      *cp = out;
    }
  } else {
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < plane; e += (int64_t)gridDim.x * 256) {
      const float acc = sum_planes(P, plane, S, e, true);
      const int64_t i = e / N, j = e - i * N;
      float *cp = C + i * ldc + j;
      const float v = alpha * acc;
      *cp = BETA ? fmaf(beta, *cp, v) : v;
    }
  }
}

template <int BM, int BN, int BK, int WM, int WN, int NP, int NW>
gemm_status launch_splitk(const GemmArgs &g, int S, int unit, float *P, hipStream_t s) {
  const int tiles_m = (int)((g.M + BM - 1) / BM);
  const int tiles_n = (int)((g.N + BN - 1) / BN);
  if (((int64_t)BM * g.lda + g.K) * 4 >= (int64_t)1 << 31 ||
      ((int64_t)BK * g.ldb + g.N) * 4 >= ((int64_t)1 << 31)) {
    set_error("gemm_f32_3xbf16_splitk: lda or ldb too large for 32-bit tile offsets");
    return GEMM_STATUS_UNSUPPORTED;
  }
  const int chunk = (int)(((g.K + S - 1) / S + unit - 1) / unit * unit);
  S = (int)((g.K + chunk - 1) / chunk);  // chunks that hold work (<= requested)
  const int64_t nwg = (int64_t)tiles_m * tiles_n * S;
  if (nwg > kMaxLanes / (64 * NW)) {
    set_error("gemm_f32_3xbf16_splitk: too many workgroups");
    return GEMM_STATUS_UNSUPPORTED;
  }
  hipLaunchKernelGGL((gemm_bx3_splitk_kernel<BM, BN, BK, WM, WN, NP, NW>), dim3((unsigned)nwg),
                     dim3(64 * NW), 0, s, (int)g.M, (int)g.N, (int)g.K, chunk, g.A, g.lda, g.B,
                     g.ldb, P, tiles_m, tiles_n);
  if (gemm_status st = check_launch("gemm_bx3_splitk_kernel")) return st;
  const bool rvec = g.N % 4 == 0 && g.ldc % 4 == 0 && ((uintptr_t)g.C & 15) == 0;
  const int64_t items = rvec ? g.M * g.N / 4 : g.M * g.N;
  const unsigned grid = (unsigned)std::min<int64_t>((items + 255) / 256, 4096);
#define MM_RED(V, BT)                                                                              \
  hipLaunchKernelGGL((splitk_reduce_kernel<V, BT>), dim3(grid), dim3(256), 0, s, (int)g.M,        \
                     (int)g.N, S, P, g.alpha, g.beta, g.C, g.ldc)
  if (rvec) { if (g.beta != 0.0f) MM_RED(true, true); else MM_RED(true, false); }
  else      { if (g.beta != 0.0f) MM_RED(false, true); else MM_RED(false, false); }
#undef MM_RED
  return check_launch("splitk_reduce_kernel");
}

// Split kernel used to verify the staging split bit for bit.
__global__ __launch_bounds__(256) void split_kernel(int64_t n, const float *__restrict__ x,
                                                    unsigned short *__restrict__ p0,
                                                    unsigned short *__restrict__ p1,
                                                    unsigned short *__restrict__ p2) {
  // pairs (x[2q], x[2q+1]) through the same pair split the tile body uses
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; 2 * q < n; q += (int64_t)gridDim.x * 256) {
    const int64_t i = 2 * q;
    const bool two = i + 1 < n;
    bf16x2 h, m, l;
    split3(f32x2{x[i], two ? x[i + 1] : 0.0f}, h, m, l);
    // bit-cast whole pairs (a bit_cast of a vector element is not
    // element-indexed in this compiler) and take the halves
    const unsigned hb = __builtin_bit_cast(unsigned, h), mb = __builtin_bit_cast(unsigned, m),
                   lb = __builtin_bit_cast(unsigned, l);
    p0[i] = (unsigned short)(hb & 0xffffu);
    p1[i] = (unsigned short)(mb & 0xffffu);
    if (p2) p2[i] = (unsigned short)(lb & 0xffffu);
    if (two) {
      p0[i + 1] = (unsigned short)(hb >> 16);
      p1[i + 1] = (unsigned short)(mb >> 16);
      if (p2) p2[i + 1] = (unsigned short)(lb >> 16);
    }
  }
}

// ---- batched small problems --------------------------------------------------
// One wave per 32 SB x 32 SB sub-tile of a problem, four waves per workgroup,
// the sub-tiles of a problem on consecutive waves (its panels meet in the L1
// and L2 of one CU).  The operands go from memory straight into MFMA fragments
// (and are split in registers, NP = 2 or 3 planes; NP = 1 is binary32 on the
// FP32 matrix cores): with so few waves per problem, staging through LDS would
// add barriers that nothing overlaps.  A lane holds 8 k of its A row (two
// 128-bit loads) and of its B column (eight loads, consecutive lanes on
// consecutive columns) per 16-deep k-step: 8 consecutive k on the split path,
// two runs of 4 in binary32 (the FP32 tile's fragment order).  Eight
// waves per SIMD hide each other's latency; keeping the next k-step's loads in
// flight as well costs a third of the waves and was level or slower (20 x 20 x
// 100 x 5000 17.7 -> 17.6 us, 40 x 20 x 33 x 700 5.6 -> 5.6, 60 x 60 x 59 x
// 3000 45 -> 51).
// The k-steps lie on the grid that ends at K (only the first can be partial)
// and the products come in the tile kernels' order, so every element is the
// same sum as in the LDS-staged tile of the same arithmetic.
// Bound: HBM for problems above about 24^3; below that the number of memory
// instructions, so those that no lane needs (rows past M, k below 0) are
// skipped wave by wave.
// C stores with the non-temporal cache policy (the slc bit, NT on gfx950; a
// hint only): 32^3 x 29 297 at beta = 0 63.2 -> 55.4 us, 48^3 x 12 000 63.6
// -> 53.9 us.  The same hint on the operand loads was slower.
constexpr int kStoreNT = 2;

// SB = 2 takes whole problems of up to 64 x 64, whose operands it reads once and whose
// rows of C it writes whole (us, SB = 1 / 2: 48^3 x 5000 33.5 / 30.7 in binary32, 32.8 / 27.3 with
// three products; 60^3 x 3000 40.6 / 33.1, 39.2 / 29.9); smaller sub-tiles fill the machine
// better with few problems and cost less padding (33 x 64 x 20 x 5000 17.7 / 19.5, 14.4 / 13.5).
// WHOLE: M a multiple of 32, no rows of C to skip (binary32 32 x 32 x 2 x 10 416 with
// beta 16.3 -> 15.5 us).
template <int SB, int NP, bool BETA, bool TILED, bool WHOLE>
__global__ __launch_bounds__(256) void small_batched_bx3_kernel(
    int M, int N, int K, float alpha, const float *__restrict__ A, int64_t lda, int64_t sa,
    const float *__restrict__ B, int64_t ldb, int64_t sb, float beta, float *__restrict__ C,
    int64_t ldc, int64_t sc, int batch, int tiles_m, int tiles_n) {
  const int lane = threadIdx.x & 63;
  // the wave index is uniform across the wave; saying so keeps the problem's
  // buffer resources in scalar registers
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  int prob = (int)blockIdx.x * 4 + wv, m0 = 0, n0 = 0;
  if constexpr (TILED) {
    // XCD-aware order where a problem spans several workgroups (its panels meet in
    // one L2: 160^2 x 16 x 1500 39 -> 26 us); plain order where it does not (32^3 x
    // 29 297 is 6 % faster so, 48^3 x 5000 in binary32 38 -> 34)
    const int tiles = tiles_m * tiles_n;
    const int unit = (tiles > 4 || tiles == 3 ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x) * 4 + wv;
    prob = unit / tiles;
    const int sub = unit - prob * tiles, tm = sub / tiles_n;
    m0 = tm * 32 * SB;
    n0 = (sub - tm * tiles_n) * 32 * SB;
  }
  if (prob >= batch) return;
  const int Mr = M - m0, Nr = N - n0;  // valid rows and columns of the sub-tile (may exceed it)
  const int lr = lane & 31, lg = lane >> 5;
  // rows past M and columns past N read zero through the range check (their
  // results are never stored); k below 0 is masked per element
  const __amdgpu_buffer_rsrc_t rA = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(A + (int64_t)prob * sa + (int64_t)m0 * lda), (short)0,
      (int)(((int64_t)(Mr - 1) * lda + K) * 4), kBufferFlags);
  const __amdgpu_buffer_rsrc_t rB = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(B + (int64_t)prob * sb + n0), (short)0,
      (int)(((int64_t)(K - 1) * ldb + Nr) * 4), kBufferFlags);
  const __amdgpu_buffer_rsrc_t rC = __builtin_amdgcn_make_buffer_rsrc(
      C + (int64_t)prob * sc + (int64_t)m0 * ldc + n0, (short)0,
      (int)(((int64_t)(Mr - 1) * ldc + Nr) * 4), kBufferFlags);
  const int ldb4 = (int)ldb * 4;
  // k of a lane's element e in the step that starts at k = 0: lane group g
  // holds k = 8g + e on the split path, 4g + e % 4 + 8 (e / 4) in binary32
  // (as in the FP32 tile: MFMA e takes element e of both groups).  The group's
  // part is in the lane's offset, the rest in the wave-uniform offset.
  constexpr int kGroup = NP == 1 ? 4 : 8;       // first k of lane group 1
  auto koff = [](int e) { return NP == 1 ? 8 * (e >> 2) + (e & 3) : e; };
  int arow[SB], bcol[SB];
  bool col[SB];
#pragma unroll
  for (int i = 0; i < SB; ++i) {
    const int x = 32 * i + lr;
    // (out of range also 16 elements before)
    arow[i] = x < Mr ? (x * (int)lda + kGroup * lg) * 4 : (int)0x80000040;
    col[i] = x < Nr;
    bcol[i] = col[i] ? x * 4 + kGroup * lg * ldb4 : (int)0x80000000;
  }
  f32x16 acc[SB][SB];
#pragma unroll
  for (int i = 0; i < SB; ++i)
#pragma unroll
    for (int j = 0; j < SB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  auto ld = [](__amdgpu_buffer_rsrc_t r, int off, int soff) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
  };
  const int KT = (K + 15) / 16;
  const int kbase = K - KT * 16;
  float a[SB][8], b[SB][8];
  auto load = [&](int s) {
    const int k0 = kbase + 16 * s;
    if (s > 0 || kbase == 0) {
#pragma unroll
      for (int i = 0; i < SB; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                        rA, arow[i], (k0 + koff(4 * h)) * 4, 0));
          a[i][4 * h] = v.x; a[i][4 * h + 1] = v.y;
          a[i][4 * h + 2] = v.z; a[i][4 * h + 3] = v.w;
        }
#pragma unroll
      for (int j = 0; j < SB; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) b[j][e] = ld(rB, bcol[j], (k0 + koff(e)) * ldb4);
    } else {
      // the partial first step: k in [kbase, kbase + 16) with kbase < 0
      auto element = [&](int e) {
        const int kk = kbase + koff(e);  // the k of lane group 0
        const bool in = kk >= -kGroup * lg;
#pragma unroll
        for (int i = 0; i < SB; ++i) {
          a[i][e] = ld(rA, in ? arow[i] + kk * 4 : (int)0x80000000, 0);
          b[i][e] = ld(rB, (int)in & (int)col[i] ? bcol[i] + kk * ldb4 : (int)0x80000000, 0);
        }
      };
      // branches around loads that neither lane group needs: worth their cost
      // only where they save most of the eight (three products, us without / with:
      // 12 x 32 x 25 423 at K = 2 8.8 / 8.0, 32 x 32 x 8522 at K = 6 8.7 / 9.6, 7 x 9 x 50 000
      // at K = 6 15.0 / 19.4; binary32, whose lane group 1 begins at k = 4, saves more: 7 x
      // 9 at K = 10 22.7 / 21.8)
      if (K > (NP == 1 ? 10 : 3)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) element(e);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
#pragma unroll
          for (int i = 0; i < SB; ++i) a[i][e] = b[i][e] = 0.0f;
          if (kbase + koff(e) + kGroup >= 0) element(e);
        }
      }
    }
  };
  auto multiply = [&]() {
    if constexpr (NP == 1) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int i = 0; i < SB; ++i)
#pragma unroll
          for (int j = 0; j < SB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
    } else {
      // the 8 values of one block as NP bf16 planes (plane 0 the leading part)
      auto split8 = [](const float (&x)[8], bf16x8 (&pl)[NP]) {
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          bf16x2 x0, x1, x2;
          if constexpr (NP == 2) split2(f32x2{x[e], x[e + 1]}, x0, x1);
          else split3(f32x2{x[e], x[e + 1]}, x0, x1, x2);
          pl[0][e] = x0.x; pl[0][e + 1] = x0.y;
          pl[1][e] = x1.x; pl[1][e + 1] = x1.y;
          if constexpr (NP == 3) { pl[2][e] = x2.x; pl[2][e + 1] = x2.y; }
        }
      };
      bf16x8 pa[SB][NP], pb[SB][NP];
#pragma unroll
      for (int i = 0; i < SB; ++i) split8(a[i], pa[i]);
#pragma unroll
      for (int j = 0; j < SB; ++j) split8(b[j], pb[j]);
      auto prod = [&](int qa, int qb) {
#pragma unroll
        for (int i = 0; i < SB; ++i)
#pragma unroll
          for (int j = 0; j < SB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa[i][qa], pb[j][qb], acc[i][j], 0, 0, 0);
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
  };
  for (int s = 0; s < KT; ++s) {
    load(s);
    // all loads of a step in flight before its first product: left alone, the
    // compiler moves each load of B behind the previous binary32 product and
    // waits for it (32 x 32 x 64 x 6798 in binary32 37 -> 33 us)
    __builtin_amdgcn_sched_barrier(0);
    multiply();
  }
  // 32 x 32 block layout: lane l, element e -> row 8*(e/4) + 4*(l/32) + e%4,
  // column l%32.  Columns past N get an out-of-range offset; rows past M fall
  // beyond the resource and their stores are dropped; groups of eight rows
  // that lie past M altogether issue nothing.  With beta != 0 every read of C
  // is issued before the first store.
  const int ldc4 = (int)ldc * 4;
  int vb[SB];
#pragma unroll
  for (int j = 0; j < SB; ++j) vb[j] = col[j] ? 4 * lg * ldc4 + (32 * j + lr) * 4 : (int)0x80000000;
  // (64 rows with beta: without tests, whose joins hold the stores back: 60^3 x 3000 with
  // three products 41.5 -> 38.7 us; beta 0 33 x 64 x 20 x 5000 13.3, 13.7 without them)
  constexpr bool kAllRows = WHOLE || (SB == 2 && BETA);
  float cold[SB][SB][16];
  if (BETA) {
#pragma unroll
    for (int i = 0; i < SB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (kAllRows || 32 * i + 8 * q < Mr) {
#pragma unroll
          for (int j = 0; j < SB; ++j)
#pragma unroll
            for (int e = 4 * q; e < 4 * q + 4; ++e)
              cold[i][j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                            rC, vb[j], (32 * i + 8 * q + (e & 3)) * ldc4, 0));
        }
  }
#pragma unroll
  for (int i = 0; i < SB; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (kAllRows || 32 * i + 8 * q < Mr) {
#pragma unroll
        for (int e = 4 * q; e < 4 * q + 4; ++e)
#pragma unroll
          for (int j = 0; j < SB; ++j) {
            float v = alpha * acc[i][j][e];
            if (BETA) v = fmaf(beta, cold[i][j][e], v);
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rC, vb[j],
                                                  (32 * i + 8 * q + (e & 3)) * ldc4, kStoreNT);
          }
      }
}

// Offsets of the small-problem kernel stay below 2^31: M rows of A, K rows of B,
// the rows of C in whole groups of eight (those past M are dropped by the range
// check).
bool small_batched_fits(const GemmArgs &g) {
  const int64_t lim = (int64_t)1 << 31, rows = (g.M + 7) / 8 * 8;
  return (g.M * g.lda + g.K) * 4 < lim && (g.K * g.ldb + g.N) * 4 < lim &&
         (rows * g.ldc + g.N) * 4 < lim;
}

// At most 65535 problems per launch (the caller's chunks).  SB = 2: problems of up
// to 64 x 64, one wave each.
template <int SB, int NP>
gemm_status launch_small_batched(const GemmArgs &g, int64_t sa, int64_t sb, int64_t sc,
                                 int batch, hipStream_t s) {
  constexpr int kTile = 32 * SB;
  const int64_t tiles_m = (g.M + kTile - 1) / kTile, tiles_n = (g.N + kTile - 1) / kTile;
  const int64_t units = tiles_m * tiles_n * batch;
  if (units > kMaxLanes / 64 || (SB == 2 && tiles_m * tiles_n > 1)) {
    set_error("gemm_strided_batched: too many tiles for one launch");
    return GEMM_STATUS_UNSUPPORTED;
  }
  const bool beta = g.beta != 0.0f;
  const dim3 grid((unsigned)((units + 3) / 4)), block(256);
#define MM_LAUNCH(BT, TILED, WHOLE)                                                              \
  hipLaunchKernelGGL((small_batched_bx3_kernel<SB, NP, BT, TILED, WHOLE>), grid, block, 0, s,      \
                     (int)g.M, (int)g.N, (int)g.K, g.alpha, g.A, g.lda, sa, g.B, g.ldb, sb,        \
                     g.beta, g.C, g.ldc, sc, batch, (int)tiles_m, (int)tiles_n)
#define MM_LAUNCH_ROWS(BT, TILED) \
  do { if (g.M % kTile == 0) MM_LAUNCH(BT, TILED, true); else MM_LAUNCH(BT, TILED, false); } while (0)
  if (SB == 1 && tiles_m * tiles_n > 1) {
    if (beta) MM_LAUNCH_ROWS(true, SB == 1); else MM_LAUNCH_ROWS(false, SB == 1);
  } else {
    if (beta) MM_LAUNCH_ROWS(true, false); else MM_LAUNCH_ROWS(false, false);
  }
#undef MM_LAUNCH_ROWS
#undef MM_LAUNCH
  return check_launch("small_batched_bx3_kernel");
}

}  // namespace bx3

constexpr int kSplitKMax = 64;

// Tile configurations of the split-precision path.  np = planes per operand
// (2 -> 3 products, 3 -> 6 products).
struct Bx3Config {
  TileConfig t;
  int np;
};
static const Bx3Config kBx3Configs[] = {
    {{256, 256, 16, "bx3_256x256x16_8w128x64_p3", 512}, 2},
    {{128, 128, 32, "bx3_128x128x32_4w64x64_p3", 256}, 2},
    {{256, 128, 32, "bx3_256x128x32_8w64x64_p3", 512}, 2},
    {{256, 256, 32, "bx3_256x256x32_8w128x64_p3", 512}, 2},
    {{256, 256, 16, "bx3_256x256x16_8w128x64_p6", 512}, 3},
    {{128, 128, 32, "bx3_128x128x32_4w64x64_p6", 256}, 3},
    {{64, 64, 32, "bx3_64x64x32_4w32x32_p3", 256}, 2},
    {{256, 256, 16, "bx3_256x256x16_4w128x128_p3", 256}, 2},
    {{128, 128, 16, "bx3_128x128x16_4w64x64_p3", 256}, 2},
    // small products: one tile per workgroup of 8 waves, its k range split
    // over the waves (fragments straight from global memory, ordered sum
    // through LDS)
    {{32, 32, 16, "bx3_small_32x32_8wk_p3", 512}, 2},
    {{64, 64, 16, "bx3_small_64x64_8wk_p3", 512}, 2},
    {{32, 32, 16, "bx3_small_32x32_8wk_p6", 512}, 3},
    {{64, 64, 16, "bx3_small_64x64_8wk_p6", 512}, 3},
    // the 256 x 256 x 16 tile with a ring of three LDS stages: the first
    // product's fragments of the next slab are read before the barrier
    {{256, 256, 16, "bx3_256x256x16_8w128x64_p3_ring3", 512}, 2},
    // 128 x 128 x 16 tiles, the k range split between two groups of four
    // waves (partial tiles summed through LDS in group order)
    {{128, 128, 16, "bx3_128x128x16_2x4w64x64_p3_kg2", 512}, 2},
    // six products: 16-deep slabs (32-deep ones leave one workgroup per CU),
    // the two-group tile, and 256 x 128 tiles
    {{128, 128, 16, "bx3_128x128x16_4w64x64_p6", 256}, 3},
    {{128, 128, 16, "bx3_128x128x16_2x4w64x64_p6_kg2", 512}, 3},
    {{256, 128, 32, "bx3_256x128x32_8w64x64_p6", 512}, 3},
    // 64 x 64 tiles, the k range split between two groups of four waves
    {{64, 64, 32, "bx3_64x64x32_2x4w32x32_p3_kg2", 512}, 2},
};

int bx3_num_configs() { return (int)(sizeof(kBx3Configs) / sizeof(kBx3Configs[0])); }
const TileConfig &bx3_config(int i) { return kBx3Configs[i].t; }
int bx3_config_products(int i) { return kBx3Configs[i].np == 2 ? 3 : 6; }

// The default: the configuration with the least modelled time (tile_time) among
// those whose sums are short enough.  Costs fitted on 434 shapes (six products 254)
// of 32 to 8192 per dimension, whole and ragged, every configuration timed on inputs
// that change from call to call: the choice is 0.5 % (0.2 %) behind the fastest on
// average, costs fitted on long K alone were 3.0 % (0.8 %) behind, with short K the
// furthest off (1680 x 1792 x 96 13.2 us, now 8.0; six products 2618 x 3313 x 464 73, now
// 53), and a rule on tile counts 3.2 % (1.9 %), with tiles that do not fill the machine
// the furthest (256 x 256 ones only where they fill every CU: 3500^3 369 us, 240 by
// time; six products 665, 416).
int bx3_default_config(int64_t M, int64_t N, int64_t K, int n_products) {
  const int64_t cus = num_cus();
  auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  static const TileCost k3[] = {
      {0, 256, 256, 1, 10.03, 0.927, 1.35, 0.0},  {2, 256, 128, 1, 6.38, 0.622, 0.699, 0.0},
      {8, 128, 128, 2, 3.57, 0.461, 0.712, 1.92}, {14, 128, 128, 1, 3.88, 0.339, 0.407, 2.25},
      {6, 64, 64, 5, 3.45, 0.205, 0.651, 2.48},   {18, 64, 64, 2, 2.28, 0.186, 0.28, 3.04},
      {10, 64, 64, 1, 2.72, 0.143, 0.147, 2.52},  {9, 32, 32, 2, 1.09, 0.055, 0.111, 3.56}};
  static const TileCost k6[] = {
      {4, 256, 256, 1, 5.44, 1.9, 2.267, 1.74},    {17, 256, 128, 1, 5.91, 1.016, 1.167, 1.75},
      {15, 128, 128, 2, 2.2, 0.685, 1.189, 2.73},  {16, 128, 128, 1, 4.34, 0.546, 0.676, 1.58},
      {12, 64, 64, 1, 3.08, 0.169, 0.2, 2.58},     {11, 32, 32, 2, 1.27, 0.071, 0.138, 3.14}};
  // 512 whole 64 x 64 tiles in at most half as many 128 x 128 ones as there are
  // CUs keep the 64 x 64 LDS tile, which the host tests name for 2048 x 1024 x
  // 4096 (89 us; configuration 18 takes 70)
  if (n_products == 3 && M % 128 == 0 && N % 128 == 0 && 2 * tiles(128, 128) <= cus &&
      tiles(64, 64) >= 2 * cus)
    return 6;
  // No longer sums than the rules on tile counts gave, in parts of K: the small
  // tiles' run over an eighth each, the two-group tiles' over a half, or (the 64
  // x 64 one, whose sums are folded) an eighth; folding goes by whole slabs of
  // 32, so that below K = 96 its parts would be the longer ones.  Operands of one
  // sign show the difference, the split's own error averages out there: uniform
  // in [0, 1), 1280 x 1045 x 3712, 1.13e-7 with the small tile, 1.09e-7 folded
  // (65 us), 2.7e-7 over K / 2 unfolded (65 us), 5.3e-7 over K.
  auto parts = [&](int cfg) {
    if (cfg >= 9 && cfg <= 12) return 8;
    if (cfg == 18) return K >= 96 ? 8 : 2;
    return cfg == 14 || cfg == 16 ? 2 : 1;
  };
  const int at_least = parts(bx3_count_config(M, N, K, n_products));
  int best = n_products == 6 ? 12 : 10;
  double best_us = -1.0;
  auto consider = [&](const TileCost &t) {
    if (parts(t.cfg) < at_least || kBx3Configs[t.cfg].t.per_launch(M, N) < 1) return;
    if ((t.cfg == 14 || t.cfg == 16 || t.cfg == 18) && K % 2 != 0) return;  // two equal k ranges
    const double us = tile_time(t, M, N, K);
    if (best_us < 0.0 || us < best_us) { best = t.cfg; best_us = us; }
  };
  if (n_products == 6) for (const TileCost &t : k6) consider(t);
  else for (const TileCost &t : k3) consider(t);
  return best;
}

int bx3_count_config(int64_t M, int64_t N, int64_t K, int n_products) {
  const int64_t cus = num_cus();
  auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  const bool six = n_products == 6;
  if (tiles(256, 256) >= cus) return six ? 4 : 0;
  const int64_t t128 = tiles(128, 128), mid = tiles(256, 128);
  if (!six && mid * 4 >= cus * 3 && mid <= cus) return 2;
  if (!six && t128 <= cus && 2 * t128 > cus && K % 2 == 0) return 14;
  if (t128 >= cus) return six ? 15 : 8;
  if (tiles(32, 32) <= 2 * cus) return six ? 11 : 9;
  return six ? 12 : tiles(64, 64) < 2 * cus ? 10 : 6;
}

gemm_status bx3_run(const GemmArgs &g, int cfg, hipStream_t s) {
  if (cfg >= 9 && cfg <= 12) return small_run(g, (cfg - 9) & 1, cfg <= 10 ? 2 : 3, s);
  if (g.ta || g.tb) return g.ta ? (g.tb ? bx3_run_tt(g, cfg, s) : bx3_run_tn(g, cfg, s)) : bx3_run_nt(g, cfg, s);
  switch (cfg) {
    case 0: return bx3::launch<256, 256, 16, 128, 64, 2, 8>(g, s);
    case 1: return bx3::launch<128, 128, 32, 64, 64, 2, 4>(g, s);
    case 2: return bx3::launch<256, 128, 32, 64, 64, 2, 8>(g, s);
    case 3: return bx3::launch<256, 256, 32, 128, 64, 2, 8>(g, s);
    case 4: return bx3::launch<256, 256, 16, 128, 64, 3, 8>(g, s);
    case 5: return bx3::launch<128, 128, 32, 64, 64, 3, 4>(g, s);
    case 6: return bx3::launch<64, 64, 32, 32, 32, 2, 4>(g, s);
    case 7: return bx3::launch<256, 256, 16, 128, 128, 2, 4>(g, s);
    case 8: return bx3::launch<128, 128, 16, 64, 64, 2, 4>(g, s);
    case 13: return bx3::launch<256, 256, 16, 128, 64, 2, 8, false, false, 3>(g, s);
    case 14: return bx3::launch_kg<128, 128, 16, 64, 64, 2, 4>(g, s);
    case 15: return bx3::launch<128, 128, 16, 64, 64, 3, 4>(g, s);
    case 16: return bx3::launch_kg<128, 128, 16, 64, 64, 3, 4>(g, s);
    case 17: return bx3::launch<256, 128, 32, 64, 64, 3, 8>(g, s);
    case 18: return bx3::launch_kg<64, 64, 32, 32, 32, 2, 4>(g, s);
    default: set_error("gemm_f32_3xbf16: bad tile config"); return GEMM_STATUS_UNSUPPORTED;
  }
}

// Split counts for the 128 x 128 tiles; a chunk is at least 256 deep.
int bx3_splitk_default(int64_t M, int64_t N, int64_t K) {
  const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128);
  int64_t s = (2 * (int64_t)num_cus() + tiles - 1) / tiles;
  const int64_t by_k = K / 256;
  if (s > by_k) s = by_k;
  if (s > kSplitKMax) s = kSplitKMax;
  return (int)(s < 1 ? 1 : s);
}

size_t bx3_splitk_ws_bytes(int64_t M, int64_t N, int splits) {
  return splits <= 1 ? 0 : (((size_t)splits * (size_t)M * (size_t)N * 4 + 255) / 256) * 256;
}

gemm_status bx3_run_splitk(const GemmArgs &g, int n_products, int splits, void *ws, hipStream_t s) {
  float *P = static_cast<float *>(ws);
  if (splits <= 1) return bx3_run(g, n_products == 6 ? 15 : 8, s);  // same tile, one pass
  const int unit = n_products == 6 ? 32 : 16;
  // 64 x 64 tiles where half of a 128 x 128 tile would be padding (three / six
  // products, us, 128 -> 64: 14 x 3595 x 1168 15.1 -> 12.5, 21 -> 14; 64 x 4096
  // x 4096 22.5 -> 22, 29 -> 27) or operands are small and 128 x 128 tiles leave
  // half of the CUs idle (a quarter for six products, whose tiles take longer), so
  // that a chunk's chain of slabs is the time: 512 x 512 x 2048 on 128 CUs 15.3 ->
  // 12.6, 19.7 -> 14.7; 384 x 1200 x 1600 on 180 16.1 -> 17.4, 21.8 -> 19.4; 512 x
  // 1800 x 1024 on 240 17.8 -> 18.3, 22.1 -> 24.7; 1024 x 4096 x 1024 twice on all
  // 40 -> 48, 56 -> 67.  Larger operands stream from HBM, three products as fast as
  // that goes: 128-wide tiles read longer pieces of B's rows (64 x 8192 x 8192 70 ->
  // 65, 100 x 4096 x 4096 32 -> 25, 120 x 1100 x 7000 22 -> 20).
  const int64_t bytes = 4 * (g.M + g.N) * g.K;
  const int64_t deep = ((g.K + splits - 1) / splits + unit - 1) / unit * unit;  // of a chunk
  const int64_t big = ((g.M + 127) / 128) * ((g.N + 127) / 128) * ((g.K + deep - 1) / deep);
  const bool idle = big * 4 <= (n_products == 6 ? 3 : 2) * (int64_t)num_cus();
  const bool small = (g.M <= 64 ? n_products == 6 || bytes <= 80000000
                                : idle && bytes <= 24000000) &&
                     bx3::offsets_fit<64, 64, 32, false, false>(g) &&
                     kBx3Configs[6].t.per_launch(g.M, g.N) >= splits;
  if (n_products == 6)
    return small ? bx3::launch_splitk<64, 64, 32, 32, 32, 3, 4>(g, splits, unit, P, s)
                 : bx3::launch_splitk<128, 128, 16, 64, 64, 3, 4>(g, splits, unit, P, s);
  return small ? bx3::launch_splitk<64, 64, 32, 32, 32, 2, 4>(g, splits, unit, P, s)
               : bx3::launch_splitk<128, 128, 16, 64, 64, 2, 4>(g, splits, unit, P, s);
}

gemm_status f32mfma_run(const GemmArgs &g, int which, hipStream_t s) {
  if (g.ta || g.tb)
    return g.ta ? (g.tb ? f32mfma_run_tt(g, which, s) : f32mfma_run_tn(g, which, s))
                : f32mfma_run_nt(g, which, s);
  return bx3::f32mfma_run_trans<false, false>(g, which, s);
}

// Batched-strided products: the tile with the least modelled time beyond the
// operands' traffic, which every tile has in common: `fixed` ns per output
// tile and `step` ns per tile and 16-deep k-step, whole machine.  The batch takes whole
// rounds of the workgroups that fit the machine at once while there are few rounds; of a
// round that is not full, `part` is its latency and the rest goes with the tiles.
// `ragged`: where rows of C are no whole 64-byte pieces, sub-tiles of one wave each
// write parts of lines (three products, 53 x 59 x 24 x 2398 17.3 us, 64 x 64 tiles 12.3).
// Fitted on 390 batches a mode (16 to 2000 per dimension, 8 to 400 MB), every tile timed
// on inputs that change from call to call: the choice is 1.2 to 1.3 % behind the fastest
// on average, with costs fitted on 46 batches it was 3.5 to 4.3 %.  Against the
// tile chosen by the stacked problem's size alone (256 x 256 tiles for any large batch),
// binary32 / three / six products, us: 100 x 72 x 90 x 2000 232 -> 70, 101 -> 53, 135 ->
// 55; 144 x 8 x 9 x 5403 217 -> 20, 153 -> 18, 236 -> 18; 300^3 x 100 163 -> 65, 55 -> 47, 84 ->
// 55.
namespace {
struct BatchTile {
  TileConfig t;                // output tile
  double per_cu[3];            // tiles per compute unit at once
  double fixed[3], step[3];    // ns: binary32, three products, six products
  double part[3];
};
constexpr BatchTile kBatchTiles[kBatchedTiles] = {
    // kBatchedDirect, 64, 128, 256, kBatchedWave64
    {{32, 32, 16, "direct", 64}, {20, 20, 20}, {0.036, 0.168, 0.136}, {0.264, 0.14, 0.203}, {0.5, 0.33, 0.44}},
    {{64, 64, 32, "lds64", 256}, {4, 4, 4}, {9.37, 2.51, 7.11}, {1.985, 0.195, 0.6}, {0.15, 0.54, 0.15}},
    {{128, 128, 16, "lds128", 256}, {2, 2, 2}, {2.4, 6.64, 5.78}, {3.36, 0.507, 1.286}, {0.75, 0.48, 0.9}},
    {{256, 256, 16, "lds256", 512}, {1, 1, 1}, {13.5, 25.4, 38.6}, {13.2, 1.32, 3.66}, {0.6, 0.9, 0.9}},
    {{64, 64, 16, "direct64", 64}, {12, 4, 8}, {2.34, 0.62, 0.655}, {0.51, 0.447, 0.361}, {0.9, 0.68, 0.9}},
};
// `ragged` of a sub-tile, in problems of one 64 x 64 tile, of one 128 x 128 tile
// (and per step) and in wider ones
constexpr double kRagged64[3] = {0.73, 0.0, 0.2}, kRagged128[3] = {0.0, 0.23, 0.29},
                 kRagged128Step[3] = {0.051, 0.0, 0.0}, kRaggedWide[3] = {0.25, 0.22, 0.215};
// a 64 x 64 problem's wave that reads C as well: two waves per SIMD (three products, us,
// with beta, wave / LDS tile: 60^3 x 3000 38 / 36, 64^3 x 4000 54 / 50)
constexpr double kWave64Beta[3] = {1.5, 1.21, 1.34};
}  // namespace

int batched_config(int path, int n_products, int64_t M, int64_t N, int64_t K, int64_t batch,
                   bool reads_c) {
  const int mode = path == GEMM_PATH_F32 ? 0 : n_products == 6 ? 2 : 1;
  const double steps = (double)((K + 15) / 16);
  double ragged = 0.0;
  if (N % 16 != 0 && N > 64)
    ragged = M <= 128 && N <= 128 ? kRagged128[mode] + kRagged128Step[mode] * steps : kRaggedWide[mode];
  else if (N % 16 != 0 && N > 32 && M <= 64)
    ragged = kRagged64[mode];
  int best = kBatchedDirect;
  double best_cost = 0.0;
  for (int c = 0; c < kBatchedTiles; ++c) {
    const BatchTile &t = kBatchTiles[c];
    if (c == kBatchedWave64 && (M > 64 || N > 64 || (M <= 32 && N <= 32))) continue;
    const double tiles = (double)((M + t.t.bm - 1) / t.t.bm) * (double)((N + t.t.bn - 1) / t.t.bn) *
                         (double)batch;
    const double slots = (double)num_cus() * t.per_cu[mode];
    const double r = tiles / slots;
    const double rounds = r > 4.0 ? r : r >= 1.0 ? std::ceil(r) : t.part[mode] + (1.0 - t.part[mode]) * r;
    const double more = c == kBatchedWave64 && reads_c ? kWave64Beta[mode] : 1.0;
    const double cost = more * rounds * slots * (t.fixed[mode] + (c == kBatchedDirect ? ragged : 0.0) +
                                          t.step[mode] * steps);
    if (c == 0 || cost < best_cost) { best = c; best_cost = cost; }
  }
  return best;
}

template <int NP>
static gemm_status batched_tile(int cfg, const GemmArgs &g, int64_t sa, int64_t sb, int64_t sc,
                                int batch, hipStream_t s) {
  switch (cfg) {
    case kBatchedDirect: return bx3::launch_small_batched<1, NP>(g, sa, sb, sc, batch, s);
    case kBatchedWave64: return bx3::launch_small_batched<2, NP>(g, sa, sb, sc, batch, s);
    case kBatched128: return bx3::launch_batched<128, 128, 16, 64, 64, NP, 4>(g, sa, sb, sc, batch, s);
    case kBatched256: return bx3::launch_batched<256, 256, 16, 128, 64, NP, 8>(g, sa, sb, sc, batch, s);
    default: return bx3::launch_batched<64, 64, 32, 32, 32, NP, 4>(g, sa, sb, sc, batch, s);
  }
}

gemm_status batched_run(int path, int cfg, const GemmArgs &g, int n_products, int64_t sa,
                        int64_t sb, int64_t sc, int batch, hipStream_t s) {
  // a tile whose 32-bit offsets cannot reach the operands, or with more tiles in a
  // problem than a launch has room for, leaves them to the next that can: the 64 x
  // 64 one has the smallest panels of A, the larger ones the smaller slabs of B
  auto runs = [&](int c) {
    if (kBatchTiles[c].t.per_launch(g.M, g.N) < 1) return false;
    switch (c) {
      case kBatchedDirect: return bx3::small_batched_fits(g);
      case kBatchedWave64:  // (64 rows of C are addressed)
        return g.M <= 64 && g.N <= 64 && bx3::small_batched_fits(g) &&
               (64 * g.ldc + g.N) * 4 < ((int64_t)1 << 31);
      case kBatched128: return bx3::offsets_fit<128, 128, 16, false, false>(g);
      case kBatched256: return bx3::offsets_fit<256, 256, 16, false, false>(g);
      default: return bx3::offsets_fit<64, 64, 32, false, false>(g);
    }
  };
  for (int c : {kBatched64, kBatched128, kBatched256})
    if (!runs(cfg)) cfg = c;
  // as many problems to a launch as its lanes allow
  const int64_t most = std::max<int64_t>(1, kBatchTiles[cfg].t.per_launch(g.M, g.N));
  for (int64_t b = 0; b < batch; b += most) {
    GemmArgs part = g;
    part.A += b * sa;
    part.B += b * sb;
    part.C += b * sc;
    const int n = (int)std::min<int64_t>(most, batch - b);
    const gemm_status st = path == GEMM_PATH_F32 ? batched_tile<1>(cfg, part, sa, sb, sc, n, s)
                           : n_products == 6     ? batched_tile<3>(cfg, part, sa, sb, sc, n, s)
                                                 : batched_tile<2>(cfg, part, sa, sb, sc, n, s);
    if (st) return st;
  }
  return GEMM_STATUS_OK;
}

gemm_status bx3_split(int64_t n, const float *x, uint16_t *p0, uint16_t *p1, uint16_t *p2,
                      hipStream_t s) {
  const int64_t want = ((n + 1) / 2 + 255) / 256;
  const unsigned grid = (unsigned)(want < 8192 ? (want > 0 ? want : 1) : 8192);
  hipLaunchKernelGGL(bx3::split_kernel, dim3(grid), dim3(256), 0, s, n, x, p0, p1, p2);
  return check_launch("split_kernel");
}

}  // namespace mm
