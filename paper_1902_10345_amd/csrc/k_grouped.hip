// k_grouped.hip -- one launch for a batch of independent GEMMs of
// uneven sizes on the 3xBF16 split-precision MFMA path.
//
// The batch is flattened into one list of output tiles (problem p owns tiles
// [start[p], start[p+1])), one workgroup per tile, in an order that hands out
// the longest tiles first: the hardware's dispatcher then plays the part of the
// paper's consume scopes (Sec. 3.3), where workers take elements off a shared
// stream -- a workgroup starts as soon as a CU has room.  A workgroup finds its
// problem by a search over the prefix of tile counts and runs the same tile
// body as the single-GEMM kernel.  Each problem carries its own tile shape,
// chosen per problem (library heuristic or the autotuner).
//
// Nothing in the workspace is written on the device, so a launch can be
// captured into a HIP graph and replayed.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "bf16x3.hpp"
#include "grouped.hpp"
#include "kernels.hpp"

namespace mm {
namespace grp {

// Tile variants of the grouped kernel (256 lanes, 2 bf16 planes).
//   0: 128 x 128 x 16 (2 x 2 waves of 64 x 64)   1: 64 x 64 x 32 (2 x 2 of 32 x 32)
constexpr int kVariants = 2;
constexpr int kBM[kVariants] = {128, 64};
constexpr int kBN[kVariants] = {128, 64};
using G0 = bx3::Cfg<128, 128, 16, 64, 64, 2, 4>;
using G1 = bx3::Cfg<64, 64, 32, 32, 32, 2, 4>;
constexpr int kLdsBytes = G0::LDS_BYTES > G1::LDS_BYTES ? G0::LDS_BYTES : G1::LDS_BYTES;

template <int V, bool BETA>
__device__ __forceinline__ void run_tile(const Desc &d, int m0, int n0, __bf16 *lds) {
  if constexpr (V == 0)
    bx3::tile<128, 128, 16, 64, 64, 2, 4, BETA>(d.M, d.N, d.K, d.alpha, d.A, d.lda, d.B,
                                                     d.ldb, d.beta, d.C, d.ldc, m0, n0, lds);
  else
    bx3::tile<64, 64, 32, 32, 32, 2, 4, BETA>(d.M, d.N, d.K, d.alpha, d.A, d.lda, d.B, d.ldb,
                                                   d.beta, d.C, d.ldc, m0, n0, lds);
}

// Workgroups are dispatched round robin over the 8 XCDs.  Within each run of
// kRun * 8 consecutive ids, an XCD gets kRun consecutive tiles: neighbouring
// tiles of a problem -- which share A row panels and B column panels -- meet in
// one L2, and every XCD sees the list from its long end to its short one (512
// problems of 32 to 1024 per dimension: runs of 1 tile 167 us, 4 155, 16 152,
// 64 160; 204 unaligned problems 96, 91, 91, 104).
constexpr int kRun = 16;
__device__ __forceinline__ int dealt_tile(int wg, int total) {
  const int base = wg - wg % (8 * kRun);
  if (base + 8 * kRun > total) return base + xcd_remap(wg - base, total - base);
  const int in = wg - base;
  return base + (in % 8) * kRun + in / 8;
}

// Bound: HBM and the matrix cores' wait for it (a tile is 2 to 64 k-slabs, then
// done).  Three workgroups per CU (16-deep slabs: 32 KB of LDS, 142 registers
// per lane) overlap their start, loads and stores: 512 problems of
// 32 to 1024 per dimension 165 -> 152 us against two persistent workgroups per CU
// that took tiles from an atomic counter (cleared by a launch of its own); 204
// unaligned problems 139 -> 90.
__global__ __launch_bounds__(256, 3) void grouped_kernel(
    const Desc *__restrict__ descs, const int *__restrict__ starts, int count, int first) {
  __shared__ __attribute__((aligned(16))) __bf16 lds[kLdsBytes / 2];
  const int t = first + dealt_tile((int)blockIdx.x, (int)gridDim.x);
  // owning problem: the last p with starts[p] <= t, a search by 64 lanes (two
  // dependent loads for up to 4096 problems)
  const int lane = threadIdx.x & 63;
  int lo = 0, n = count;
  while (n > 1) {
    const int step = (n + 63) / 64, at = lane * step;
    const bool le = at < n && starts[lo + (at < n ? at : 0)] <= t;
    const int seg = __builtin_popcountll(__ballot(le)) - 1;
    lo += seg * step;
    n = min(step, n - seg * step);
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  const Desc d = descs[lo];
  const int local = t - starts[lo];
  const int bm = d.variant == 0 ? 128 : 64, bn = bm;
  // tiles of a problem in groups of 8 tile rows, as in the single-GEMM
  // kernels: consecutive tiles share A row panels and B column panels
  int tm, tn;
  tile_coords(local, (d.M + bm - 1) / bm, d.tiles_n, 8, tm, tn);
  const int m0 = tm * bm, n0 = tn * bn;
  if (d.beta != 0.0f) {
    if (d.variant == 0) run_tile<0, true>(d, m0, n0, lds);
    else run_tile<1, true>(d, m0, n0, lds);
  } else {
    if (d.variant == 0) run_tile<0, false>(d, m0, n0, lds);
    else run_tile<1, false>(d, m0, n0, lds);
  }
}

}  // namespace grp

int grouped_num_variants() { return grp::kVariants; }
int grouped_variant_bm(int v) { return grp::kBM[v]; }

// Library heuristic: the variant with the smaller padded work, where a 64 x 64
// tile is charged `small_cost` times a 128 x 128 tile's work per output
// element (it re-reads its operands twice as often).
int grouped_pick_variant(int64_t M, int64_t N, double small_cost) {
  const double w0 = (double)((M + 127) / 128) * ((N + 127) / 128) * 128.0 * 128.0;
  const double w1 = (double)((M + 63) / 64) * ((N + 63) / 64) * 64.0 * 64.0 * small_cost;
  return w1 < w0 ? 1 : 0;
}

size_t grouped_ws_bytes(int count) {
  const size_t head = 256;  // unused: the size that callers allocate stays as it was
  const size_t descs = ((sizeof(Desc) * (size_t)count + 255) / 256) * 256;
  const size_t starts = sizeof(int) * ((size_t)count + 1);
  return head + descs + starts;
}

gemm_status grouped_build(const gemm_problem *probs, int count, const int *variant,
                          std::vector<Desc> &descs, std::vector<int> &starts, int &total) {
  descs.resize(count);
  starts.resize((size_t)count + 1);
  const double small_cost = tuned_small_cost();
  // Longest tiles first: a tile's time grows with K, so handing out the
  // deepest problems' tiles first keeps the end of the queue short.  The
  // table order changes only the schedule, never a problem's result.
  std::vector<int> order(count);
  for (int p = 0; p < count; ++p) order[p] = p;
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return probs[a].K > probs[b].K; });
  int64_t t = 0;
  for (int slot = 0; slot < count; ++slot) {
    const int p = order[slot];
    const gemm_problem &q = probs[p];
    Desc &d = descs[slot];
    d.A = q.A; d.B = q.B; d.C = q.C;
    d.lda = q.lda; d.ldb = q.ldb; d.ldc = q.ldc;
    d.M = (int)q.M; d.N = (int)q.N; d.K = (int)q.K;
    d.alpha = q.alpha; d.beta = q.beta;
    d.variant = variant ? variant[p] : grouped_pick_variant(q.M, q.N, small_cost);
    const int bm = grp::kBM[d.variant], bn = grp::kBN[d.variant];
    // problems that need no MFMA work contribute no tiles; the host handles
    // them (no-op or C <- beta*C) before the launch
    const bool work = q.M > 0 && q.N > 0 && q.K > 0 && q.alpha != 0.0f;
    d.tiles_n = work ? (int)((q.N + bn - 1) / bn) : 0;
    const int64_t tiles = work ? ((q.M + bm - 1) / bm) * (int64_t)d.tiles_n : 0;
    starts[slot] = (int)t;
    t += tiles;
    if (t > 0x7fffffff) { set_error("grouped_gemm: too many tiles"); return GEMM_STATUS_UNSUPPORTED; }
  }
  starts[count] = (int)t;
  total = (int)t;
  return GEMM_STATUS_OK;
}

gemm_status grouped_enqueue(void *ws, int count, int total, hipStream_t s) {
  if (total == 0) return GEMM_STATUS_OK;
  const uint8_t *base = static_cast<const uint8_t *>(ws);
  const Desc *descs = reinterpret_cast<const Desc *>(base + 256);
  const int *starts = reinterpret_cast<const int *>(
      base + 256 + ((sizeof(Desc) * (size_t)count + 255) / 256) * 256);
  // (a launch holds less than 2^32 lanes)
  constexpr int kMaxGrid = 1 << 23;
  for (int first = 0; first < total; first += kMaxGrid) {
    const dim3 grid((unsigned)std::min(kMaxGrid, total - first));
    hipLaunchKernelGGL(grp::grouped_kernel, grid, dim3(256), 0, s, descs, starts, count, first);
    if (gemm_status st = check_launch("grouped_kernel")) return st;
    if (total - first <= kMaxGrid) break;
  }
  return GEMM_STATUS_OK;
}

gemm_status grouped_upload(void *ws, const std::vector<Desc> &descs, const std::vector<int> &starts,
                           hipStream_t s) {
  uint8_t *base = static_cast<uint8_t *>(ws);
  const size_t dbytes = sizeof(Desc) * descs.size();
  const size_t soff = 256 + ((dbytes + 255) / 256) * 256;
  hipError_t e = hipMemcpyAsync(base + 256, descs.data(), dbytes, hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return hip_fail("grouped_gemm: descriptor upload", e);
  e = hipMemcpyAsync(base + soff, starts.data(), sizeof(int) * starts.size(), hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return hip_fail("grouped_gemm: tile-prefix upload", e);
  // the host vectors are freed on return: make sure the copies have consumed them
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail("grouped_gemm: upload sync", e);
  return GEMM_STATUS_OK;
}

gemm_status grouped_upload_pinned(void *ws, void *pinned, const std::vector<Desc> &descs,
                                  const std::vector<int> &starts, hipStream_t s) {
  // the pinned staging buffer mirrors the workspace from byte 256 on; the
  // caller guarantees it is not rewritten before this copy has executed
  const size_t dbytes = sizeof(Desc) * descs.size();
  const size_t soff = ((dbytes + 255) / 256) * 256;
  uint8_t *h = static_cast<uint8_t *>(pinned);
  std::memcpy(h, descs.data(), dbytes);
  std::memcpy(h + soff, starts.data(), sizeof(int) * starts.size());
  hipError_t e = hipMemcpyAsync(static_cast<uint8_t *>(ws) + 256, h, soff + sizeof(int) * starts.size(),
                                hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return hip_fail("grouped: descriptor upload", e);
  return GEMM_STATUS_OK;
}

}  // namespace mm
