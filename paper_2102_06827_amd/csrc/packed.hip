// packed.hip -- gather product over any strides and extents: single elements
// are loaded, and packed along the summation on their way into LDS.
//
// The vector-load tiles of gett.hip need 16-byte aligned runs in both
// operands; orbital counts are as often odd as not, and then they have only
// a 64 x 64 tile that loads elements through 64-bit offset pairs.  This
// kernel loads nothing but single elements, so it needs no runs and no
// alignment, and makes them cheap instead:
//
//   * Offsets are 32-bit byte offsets (operands below 2 GiB).  An operand
//     contiguous along its rows has one row offset per thread, in a vector
//     register, and its summation offsets in scalar registers; one contiguous
//     along the summation has the summation offset in a vector register, one
//     per step.  Either way an element costs one 32-bit addition and one
//     buffer load: the sum is the load's vector offset, which its bounds check
//     sees whole.
//   * 64 lanes read 64 consecutive elements (or 64 / BK runs of BK), so the
//     loads are as coalesced as the operand allows.  Rows past the edge read
//     the last row (the tables are padded with it), whose products are never
//     stored; indices past the summation's end have offsets out of the
//     operand's bounds and load zeros.  Nothing is masked.
//   * Every LDS tile is stored [row][k] with a 16-byte pad, whatever the
//     operand's order: a thread that walks the summation writes its 16 bytes
//     of consecutive k at once.  A lane then reads 16 bytes of one row for 2
//     (FP64) or 4 (FP32) MFMAs: over a chunk of 4 * VL summation indices,
//     lane group g = lane / 16 holds indices g * VL .. g * VL + VL - 1, and
//     MFMA j of the chunk multiplies index g * VL + j of every group (A and B
//     agree on it, so the sum is the same up to order).  With a pitch of
//     BK + VL elements the 16 rows a lane group reads start in 16 different
//     groups of four banks.
//
// Bound: the matrix cores.  Software pipeline, one barrier a step: a step's
// products run while the next step moves from registers to LDS (during the
// first half) and the one after is asked for (during the second), the LDS
// writes and loads spread between the MFMAs, so that nothing waits for a load
// issued less than a step ago.  MI355X, against the tiles of gett.hip on the
// same box: a full round of 128 x 128 tiles over K = 8208, FP64 66-71 TFLOP/s
// (60-64), FP32 122-138 (103-107); 1725^3 in FP64 171 us (244; by TTGT's
// permutes and GEMM 286), in FP32 95 us (206); 256^3 in FP64 9.4 us (12.4).
//
// The tiles: 128 x 128 moves the fewest bytes per product; the smaller ones
// fill the chip and fit ragged edges better, down to half of a 64 x 64 tile
// for outputs with one side of at most 32 (98304 x 32, K = 96, FP64: 20 us
// against 27 on 64 x 64) and for latency (512^3: 15 us against 17).
//
// A launch is `whole` workgroups that compute one output tile each, then
// `shares` workgroups that split the summation steps of the remaining tiles
// equally; a share may run over tile boundaries.  Partial tiles go to the
// workspace and packed_fixup_kernel adds them in share order.
#include <array>
#include <climits>
#include <map>
#include <mutex>
#include <type_traits>

#include "packed.hpp"

namespace comet {
namespace {

using namespace packed;

// Workgroup tile BM x BN, summation step BK, a WGM x WGN grid of waves, and
// the waves per SIMD the register allocation leaves room for.
struct PackedTile {
  int bm, bn, bk, wgm, wgn, wpe;
};
constexpr PackedTile kPacked64[] = {
    {128, 128, 16, 4, 2, 4},
    {64, 64, 16, 2, 2, 4},
    {128, 64, 16, 4, 2, 4},
    {64, 32, 16, 2, 2, 4},
    {32, 64, 16, 2, 2, 4},
};
constexpr PackedTile kPacked32[] = {
    {128, 128, 32, 2, 2, 2},
    {64, 64, 32, 2, 2, 4},
    {128, 64, 32, 4, 2, 4},
    {64, 32, 32, 2, 2, 4},
    {32, 64, 32, 2, 2, 4},
};
static_assert(sizeof(kPacked64) / sizeof(PackedTile) == kPackedTiles, "tile count");
static_assert(sizeof(kPacked32) / sizeof(PackedTile) == kPackedTiles, "tile count");
template <typename T>
constexpr PackedTile packed_tile(int tile) {
  return sizeof(T) == 8 ? kPacked64[tile] : kPacked32[tile];
}

// FP32 accumulators of a tile (see PackedCore): eight sets on the tiles of
// small and mid-size products, a fold every 256 summation indices on 64 x 64
// and 128 x 64 and every 1024 on 128 x 128.  A whole tile would carry all of
// K in one accumulator, and its error grows by the root of that chain; a
// schedule that fills the chip with whole tiles is not to cost the accuracy
// that splitting the summation over workgroups had.  Relative error (uniform
// operands), split over workgroups / one accumulator / so: 256^3 1.5e-7,
// 2.9e-7, 1.1e-7; 512^3 1.5e-7, 4.1e-7, 1.5e-7; 960^3 2.1e-7, 5.6e-7, 2.0e-7;
// 1500^3 4.0e-7, 6.6e-7, 2.8e-7; 3072 x 600 x 1000 3.0e-7, 5.7e-7, 2.9e-7;
// 3072^3 8.4e-7, 9.5e-7, 5.7e-7.  us, one accumulator / so: 256^3 7.1 / 7.4,
// 512^3 11.1 / 11.5, 1200^3 44.3 / 44.7, 1725^3 108 / 109, 3072^3 430 / 434.
// (A fold every step or two on the small tiles: 512^3 11.6 to 12.2, 1200^3 45.3
// to 46.7; every 128 and 512 indices on the larger ones: 1900^3 144 / 146.)
// Summations of at most kPackedChain indices keep one accumulator: they are no
// longer than the chains of the small tiles, and clearing and adding the sets
// would be felt (4000 entries of 32^3 16.4 us, 19.9 with them; 98304 x 32 x 96
// 14.8 and 15.4).
constexpr int kSets32[] = {1, 1, 1, 8, 8}, kFold32[] = {32, 8, 8, 0, 0};
constexpr int kPackedChain = 128;
template <typename T>
constexpr bool packed_long(int K) { return sizeof(T) == 4 && K > kPackedChain; }
template <typename T, int TILE, int LA, int LB, bool LONG>
using PackedKernel = PackedCore<T, packed_tile<T>(TILE).bm, packed_tile<T>(TILE).bn, packed_tile<T>(TILE).bk,
                                packed_tile<T>(TILE).wgm, packed_tile<T>(TILE).wgn, LA, LB, LONG ? kSets32[TILE] : 1,
                                LONG ? kFold32[TILE] : 0>;

// The workspace slot of share s's piece of shared tile t.  Along the steps
// each piece has a larger s or a larger t than the one before, so s + t
// tells them apart; where tiles are more than the shares, each of which splits
// two tiles at most, its first or its last.
__device__ __forceinline__ int64_t piece_slot(int s, int t, bool begun_here, int tiles, int shares) {
  return tiles <= shares ? int64_t(s) + t : 2 * int64_t(s) + (begun_here ? 0 : 1);
}

// first step of share s of S over I steps
__device__ __forceinline__ int64_t share_begin(int64_t I, int S, int s) { return I * s / S; }

// STREAM: C is written with nontemporal stores.  LONG: the accumulators of
// packed_long.
template <typename T, int TILE, int LA, int LB, bool STREAM, bool LONG>
__global__ __launch_bounds__(64 * packed_tile<T>(TILE).wgm * packed_tile<T>(TILE).wgn, packed_tile<T>(TILE).wpe) void
packed_kernel(PackedLaunch g) {
  typedef PackedKernel<T, TILE, LA, LB, LONG> P;
  typedef typename P::WT WT;
  __shared__ __attribute__((aligned(16))) T smem[P::LDS];
  __shared__ int64_t ctab_s[P::BM + P::BN];
  lds_t<int64_t> *const ctab = to_lds(ctab_s);
  const int b = blockIdx.x;
  const int nk = (g.K + P::BK - 1) / P::BK;
  const bool is_whole = b < g.whole;
  const int share = is_whole ? 0 : xcd_remap(b - g.whole, g.shares);
  const int64_t I = int64_t(g.tilesM * g.tilesN - g.whole) * nk;
  int64_t it = 0, end = nk;
  if (!is_whole) {
    it = share_begin(I, g.shares, share);
    end = share_begin(I, g.shares, share + 1);
  }
  // batch labels: the entry's slices
  int64_t xa = 0, xb = 0, xc = 0;
  if (g.xa) {
    const int64_t x = g.first + blockIdx.y;
    xa = to_glb(g.xa)[x];
    xb = to_glb(g.xb)[x];
    xc = to_glb(g.xc)[x];
  }
  T *const C = static_cast<T *>(g.C) + xc;
  const __amdgpu_buffer_rsrc_t ra = buffer_of(static_cast<const T *>(g.A) + xa, g.bytesA - uint32_t(xa * sizeof(T)));
  const __amdgpu_buffer_rsrc_t rb = buffer_of(static_cast<const T *>(g.B) + xb, g.bytesB - uint32_t(xb * sizeof(T)));
  const int first = int(it / nk);
  while (it < end) {
    // (uniform values whose divisions run on the vector unit)
    const int tt = __builtin_amdgcn_readfirstlane(int(it / nk));
    const int s0 = __builtin_amdgcn_readfirstlane(int(it - int64_t(tt) * nk));
    const int s1 = __builtin_amdgcn_readfirstlane(int(end - it < nk - s0 ? s0 + (end - it) : nk));
    int tm, tn;
    group_coords(is_whole ? xcd_remap(b, g.whole) : g.whole + tt, g.tilesM, g.tilesN, &tm, &tn);
    const int m0 = __builtin_amdgcn_readfirstlane(tm * P::BM), n0 = __builtin_amdgcn_readfirstlane(tn * P::BN);
    // (What depends on the thread alone is the same for every piece: the
    // compiler works the epilogue's addresses out ahead of the loop, holds
    // them over the products and, in the FP64 128 x 128 kernels, spills 25 to
    // 32 of them.  Where registers are short a thread index it cannot see
    // through keeps them where they are used: FP64 3072^3 848 -> 828 us, no
    // scratch; elsewhere they are worked out while the loads are awaited, K =
    // 30, 3000 x 9000, FP64 59.2 us against 60.4.)
    int tid = threadIdx.x;
    if constexpr (TILE == 0 || LONG) asm volatile("" : "+v"(tid));
    WT w;
    typename P::COffsets co;
    co.load(tid, g.c, m0, n0, g.M, g.N);
    P::accumulate(w, ra, rb, g.am + m0, g.ak, g.bk, g.bn + n0, s0, s1, to_lds(smem), co, ctab, tid);
    if constexpr (TILE == 0 || LONG) asm volatile("" : "+v"(tid));
    if (s1 - s0 == nk) {
      gett_store_staged<T, T, P::BM, P::BN, P::WGM, P::WGN, false, STREAM>(
          w, C, ctab, ctab + P::BM, g.M, g.N, g.alpha, g.beta, m0, n0, nullptr, tid);
      __syncthreads();   // the C offsets are read before the next piece's are stored
    } else {
      constexpr int64_t kSlot = int64_t(WT::FM) * WT::FN * WT::NT;   // 4-vectors per slot
      gett_store_partial<T, P::BM, P::BN, P::WGM, P::WGN>(
          w, static_cast<typename WT::acc_t *>(g.ws) +
                 piece_slot(share, tt, tt == first, g.tilesM * g.tilesN - g.whole, g.shares) * kSlot);
    }
    it += s1 - s0;
  }
}

// Adds the pieces of each tile that shares split, in share order, and
// writes alpha * sum + beta * C.  Workgroup (x, y): tile x of those, and
// accumulator element y = i * FN + j of every thread.  Tiles that one share
// covered whole are already written.
template <typename T, int TILE, bool STREAM>
__global__ __launch_bounds__(64 * packed_tile<T>(TILE).wgm * packed_tile<T>(TILE).wgn) void packed_fixup_kernel(
    PackedLaunch g) {
  typedef PackedKernel<T, TILE, 0, 0, false> P;
  typedef typename P::WT WT;
  typedef typename WT::acc_t acc_t;
  const int nk = (g.K + P::BK - 1) / P::BK;
  const int tt = blockIdx.x, f = blockIdx.y;
  const int64_t I = int64_t(g.tilesM * g.tilesN - g.whole) * nk;
  // the shares holding the tile's first and last step: the largest s with
  // share_begin(s) <= x is floor(((x + 1) * S - 1) / I)
  const int64_t x0 = int64_t(tt) * nk, x1 = x0 + nk - 1;
  const int lo = int(((x0 + 1) * g.shares - 1) / I), hi = int(((x1 + 1) * g.shares - 1) / I);
  if (lo == hi) return;
  constexpr int64_t kSlot = int64_t(WT::FM) * WT::FN * WT::NT;
  const glb_t<const acc_t> *const ws = to_glb(static_cast<const acc_t *>(g.ws)) + int64_t(f) * WT::NT + threadIdx.x;
  // only the first share may have begun in an earlier tile
  const int tiles = g.tilesM * g.tilesN - g.whole;
  acc_t v = ws[piece_slot(lo, tt, share_begin(I, g.shares, lo) >= x0, tiles, g.shares) * kSlot];
  for (int s = lo + 1; s <= hi; ++s) v = v + ws[piece_slot(s, tt, true, tiles, g.shares) * kSlot];
  int tm, tn;
  group_coords(g.whole + tt, g.tilesM, g.tilesN, &tm, &tn);
  gett_store_fragment<T, T, P::BM, P::BN, P::WGM, P::WGN, STREAM>(v, f / WT::FN, f % WT::FN, static_cast<T *>(g.C),
                                                                  g.c, g.M, g.N, g.alpha, g.beta,
                                                                  int64_t(tm) * P::BM, int64_t(tn) * P::BN);
}

template <typename T, int TILE, int LA, int LB, bool STREAM, bool LONG>
hipError_t packed_s(const PackedLaunch &g, hipStream_t s) {
  typedef PackedKernel<T, TILE, LA, LB, LONG> P;
  const int64_t tiles = int64_t((g.M + P::BM - 1) / P::BM) * ((g.N + P::BN - 1) / P::BN);
  const int64_t nk = (g.K + P::BK - 1) / P::BK;
  if (g.tilesM != (g.M + P::BM - 1) / P::BM || g.tilesN != (g.N + P::BN - 1) / P::BN || g.whole < 0 ||
      g.whole > tiles || g.shares < 0 || (g.shares == 0) != (g.whole == tiles) ||
      int64_t(g.shares) > (tiles - g.whole) * nk || int64_t(g.whole) + g.shares > INT32_MAX || (g.shares && !g.ws) ||
      !packed_grid_fits(P::NT, tiles, g.whole, g.shares) || (g.xa && (g.shares || !g.xb || !g.xc)))
    return hipErrorInvalidValue;
  if (g.xa) {
    constexpr int64_t kMaxY = 65535;   // grid limit along y
    for (int64_t e0 = 0; e0 < g.entries; e0 += kMaxY) {
      PackedLaunch q = g;
      q.first = e0;
      hipLaunchKernelGGL((packed_kernel<T, TILE, LA, LB, STREAM, LONG>),
                         dim3(unsigned(g.whole), unsigned(g.entries - e0 < kMaxY ? g.entries - e0 : kMaxY)),
                         dim3(P::NT), 0, s, q);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  hipLaunchKernelGGL((packed_kernel<T, TILE, LA, LB, STREAM, LONG>), dim3(unsigned(g.whole + g.shares)), dim3(P::NT), 0, s,
                     g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || g.shares == 0) return e;
  hipLaunchKernelGGL((packed_fixup_kernel<T, TILE, STREAM>), dim3(unsigned(tiles - g.whole), P::WT::FM * P::WT::FN),
                     dim3(P::NT), 0, s, g);
  return hipGetLastError();
}

template <typename T, int TILE, int LA, int LB, bool LONG>
hipError_t packed_n(const PackedLaunch &g, int *occupancy, hipStream_t s) {
  if (occupancy)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(occupancy, packed_kernel<T, TILE, LA, LB, true, LONG>,
                                                        PackedKernel<T, TILE, LA, LB, LONG>::NT, 0);
  // C past the caches only where every store writes whole 64-byte segments.
  // Whole segments: streaming is faster (K = 32, FP64, 8192 x 16384 with
  // C in runs of 16: 266 us against 309).  Parts of one: the neighbours'
  // stores have to meet in the cache (K = 31, 6975 x 14415, runs of 15: 530
  // us streamed, 219 us plain; FP32 549 and 154 us).
  const bool stream = g.c_segments && reinterpret_cast<uintptr_t>(g.C) % 64 == 0;
  return stream ? packed_s<T, TILE, LA, LB, true, LONG>(g, s) : packed_s<T, TILE, LA, LB, false, LONG>(g, s);
}

template <typename T, int TILE, int LA, int LB>
hipError_t packed_l(const PackedLaunch &g, int *occupancy, hipStream_t s) {
  if constexpr (sizeof(T) == 4)
    if (packed_long<T>(g.K)) return packed_n<T, TILE, LA, LB, true>(g, occupancy, s);
  return packed_n<T, TILE, LA, LB, false>(g, occupancy, s);
}

template <typename T, int TILE>
hipError_t packed_t(const PackedLaunch &g, int *occupancy, hipStream_t s) {
  switch (g.layoutA * 2 + g.layoutB) {
    case 0: return packed_l<T, TILE, 0, 0>(g, occupancy, s);
    case 1: return packed_l<T, TILE, 0, 1>(g, occupancy, s);
    case 2: return packed_l<T, TILE, 1, 0>(g, occupancy, s);
    default: return packed_l<T, TILE, 1, 1>(g, occupancy, s);
  }
}

template <typename T>
hipError_t packed_d(const PackedLaunch &g, int *occupancy, hipStream_t s) {
  switch (g.tile) {
    case 0: return packed_t<T, 0>(g, occupancy, s);
    case 1: return packed_t<T, 1>(g, occupancy, s);
    case 2: return packed_t<T, 2>(g, occupancy, s);
    case 3: return packed_t<T, 3>(g, occupancy, s);
    case 4: return packed_t<T, 4>(g, occupancy, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

void packed_tile_shape(int tile, int dtype, int *bm, int *bn, int *bk, int *threads) {
  const PackedTile &p = dtype == 0 ? kPacked64[tile] : kPacked32[tile];
  *bm = p.bm;
  *bn = p.bn;
  *bk = p.bk;
  *threads = 64 * p.wgm * p.wgn;
}

hipError_t launch_packed(const PackedLaunch &g, hipStream_t s) {
  return g.dtype == 0 ? packed_d<double>(g, nullptr, s) : packed_d<float>(g, nullptr, s);
}

int packed_occupancy(int tile, int dtype, int layoutA, int layoutB, int K) {
  static std::mutex mu;
  static std::map<std::array<int, 6>, int> known;   // it depends on the kernel alone
  int device = 0;
  (void)hipGetDevice(&device);
  const std::array<int, 6> key = {device, tile, dtype, layoutA, layoutB, dtype == 1 && packed_long<float>(K)};
  std::lock_guard<std::mutex> lk(mu);
  const auto it = known.find(key);
  if (it != known.end()) return it->second;
  PackedLaunch g{};
  g.tile = tile;
  g.dtype = dtype;
  g.layoutA = layoutA;
  g.layoutB = layoutB;
  g.K = K;
  int n = 0;
  const hipError_t e = dtype == 0 ? packed_d<double>(g, &n, nullptr) : packed_d<float>(g, &n, nullptr);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    n = 0;
  }
  known[key] = n;
  return n;
}

}  // namespace comet
