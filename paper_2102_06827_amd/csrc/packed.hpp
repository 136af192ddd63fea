// packed.hpp -- the tile product of the packed gather kernels (packed.hip,
// and the native batch in batch.hip): operands loaded element by element
// through 32-bit byte offsets, and packed along the summation in LDS.  The
// reasons stand at the top of packed.hip.
#pragma once

#include "gather.hpp"
#include "kernels.hpp"

namespace comet {
namespace packed {

using namespace gather;

// a table read by wave-uniform indices only: scalar loads
typedef const __attribute__((address_space(4))) uint32_t *scalar_table;

__device__ __forceinline__ void buffer_element(double *v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  const u2 x = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
  *v = __builtin_bit_cast(double, x);
}
__device__ __forceinline__ void buffer_element(float *v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  *v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}

// `bytes` from p on; a load past them gives zero
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}

// One operand's tile: R rows by BK summation indices, PER elements a thread.
template <typename T, int R, int BK, int LAYOUT, int NT>
struct PackedLoader {
  static constexpr int VL = 16 / int(sizeof(T));
  static constexpr int LDK = BK + VL;
  static constexpr int ELEMS = R * LDK;
  static constexpr int PER = R * BK / NT;
  static_assert(PER * NT == R * BK && PER % VL == 0, "tile does not split evenly over the workgroup");
  static_assert(LAYOUT == 0 ? NT % BK == 0 : NT % R == 0, "thread mapping");
  // a wave's lanes share their summation indices: scalar offsets
  static constexpr bool UNIFORM = LAYOUT == 1 && R % 64 == 0;
  typedef T vec_t __attribute__((ext_vector_type(VL)));

  T v[PER];
  uint32_t ro[LAYOUT == 0 ? PER : 1];   // row offsets
  uint32_t ko[LAYOUT == 0 ? 1 : PER];   // summation offsets of the next step (LAYOUT 1: scalar)
  int row, k;                           // LAYOUT 0: first row, the thread's index; LAYOUT 1: the row, first index

  // rows: the row table at the tile's first row
  __device__ __forceinline__ void init(int tid, const uint32_t *rows) {
    if constexpr (LAYOUT == 0) {
      row = tid / BK;
      k = tid % BK;
#pragma unroll
      for (int p = 0; p < PER; ++p) ro[p] = to_glb(rows)[row + p * (NT / BK)];
    } else {
      row = tid % R;
      k = (UNIFORM ? __builtin_amdgcn_readfirstlane(tid / R) : tid / R) * PER;
      ro[0] = to_glb(rows)[row];
    }
  }
  // the summation offsets of the step at k0 (the table is padded past its end)
  __device__ __forceinline__ void fetch_k(const uint32_t *tab, int k0) {
    if constexpr (LAYOUT == 0) {
      ko[0] = to_glb(tab)[k0 + k];
    } else if constexpr (UNIFORM) {
      const scalar_table st = (scalar_table)(tab + k0 + k);
#pragma unroll
      for (int p = 0; p < PER; ++p) ko[p] = st[p];
    } else {
#pragma unroll
      for (int p = 0; p < PER; ++p) ko[p] = to_glb(tab)[k0 + k + p];
    }
  }
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r) {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      if constexpr (LAYOUT == 0)
        buffer_element(&v[p], r, ro[p] + ko[0], 0);
      else
        buffer_element(&v[p], r, ro[0] + ko[p], 0);
    }
  }
  // LDS writes a thread does per step
  static constexpr int WRITES = LAYOUT == 0 ? PER : PER / VL;
  // into the LDS tile
  __device__ __forceinline__ void store(lds_t<T> *s) const {
    if constexpr (LAYOUT == 0) {
#pragma unroll
      for (int p = 0; p < PER; ++p) s[(row + p * (NT / BK)) * LDK + k] = v[p];
    } else {
#pragma unroll
      for (int p = 0; p < PER; p += VL) {
        vec_t w;
#pragma unroll
        for (int i = 0; i < VL; ++i) w[i] = v[p + i];
        *reinterpret_cast<lds_t<vec_t> *>(s + row * LDK + k + p) = w;
      }
    }
  }
};

// A workgroup of WGM x WGN waves on a BM x BN output tile in summation steps
// of BK.  How long a chain of rounded additions gets: with SETS = 2 * VL each
// of a step's products into an output fragment has an accumulator of its own
// (one in 2 * VL summation indices), the sets added at the end; with FOLD > 0
// the accumulators are added into a second set and cleared every FOLD steps.
template <typename T, int BM_, int BN_, int BK_, int WGM_, int WGN_, int LA, int LB, int SETS = 1, int FOLD = 0>
struct PackedCore {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WGM = WGM_, WGN = WGN_;
  static constexpr int NT = 64 * WGM * WGN;
  typedef WaveTile<T, BM, BN, WGM, WGN> WT;
  typedef PackedLoader<T, BM, BK, LA, NT> LoadA;
  typedef PackedLoader<T, BN, BK, LB, NT> LoadB;
  static constexpr int VL = LoadA::VL, LDK = LoadA::LDK, CHUNK = 4 * VL;
  static constexpr int LDS = 2 * (LoadA::ELEMS + LoadB::ELEMS);

  // The tile's C offsets, asked for ahead of its operands (a short summation
  // would otherwise end in waiting for them) and kept in LDS for the epilogue.
  static_assert(BM + BN <= NT, "one C offset a thread");
  struct COffsets {
    int64_t v;
    __device__ __forceinline__ void load(int tid, const GettTables &c, int m0, int n0, int M, int N) {
      const bool row = tid < BM;
      const int x = row ? m0 + tid : n0 + (tid - BM), last = row ? M - 1 : N - 1;
      v = to_glb(row ? c.offCm : c.offCn)[x < last ? x : last];
    }
    __device__ __forceinline__ void store(int tid, lds_t<int64_t> *tab) const {
      if (tid < BM + BN) tab[tid] = v;
    }
  };

  static_assert(SETS == 1 || (SETS == 2 * VL && FOLD == 0), "one set, or one for each product of a step");
  typedef typename WT::acc_t Acc[WT::FM][WT::FN];

  // the products of chunk c of a step; with SETS > 1 product
  // (c, x) into set c * VL + x, set 0 being w's and the others `more`
  static __device__ __forceinline__ void mma(WT &w, Acc *more, const lds_t<T> *a, const lds_t<T> *b, int c) {
    typedef typename LoadA::vec_t vec_t;
    vec_t af[WT::FM], bf[WT::FN];
#pragma unroll
    for (int i = 0; i < WT::FM; ++i) af[i] = *reinterpret_cast<const lds_t<vec_t> *>(a + i * 16 * LDK + c * CHUNK);
#pragma unroll
    for (int j = 0; j < WT::FN; ++j) bf[j] = *reinterpret_cast<const lds_t<vec_t> *>(b + j * 16 * LDK + c * CHUNK);
#pragma unroll
    for (int x = 0; x < VL; ++x)
#pragma unroll
      for (int i = 0; i < WT::FM; ++i)
#pragma unroll
        for (int j = 0; j < WT::FN; ++j) {
          typename WT::acc_t &acc = SETS == 1 || c * VL + x == 0 ? w.acc[i][j] : more[c * VL + x - 1][i][j];
          acc = mfma16(af[i][x], bf[j][x], acc);
        }
  }
  static constexpr int READS = WT::FM + WT::FN, MMAS = WT::FM * WT::FN * VL;

  // schedule of one chunk: its LDS reads, then its products with one
  // instruction of `kind` every few products
  template <int KIND, int COUNT>
  static __device__ __forceinline__ void schedule() {
    __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
    constexpr int EVERY = COUNT < MMAS ? MMAS / COUNT : 1, GROUP = (COUNT + MMAS - 1) / MMAS;
#pragma unroll
    for (int i = 0; i < (COUNT + GROUP - 1) / GROUP; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x8, EVERY, 0);
      __builtin_amdgcn_sched_group_barrier(KIND, GROUP, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x8, MMAS, 0);
  }

  // the tile's product over the summation steps [s0, s1), s1 > s0; K
  // indices in all
  static __device__ __forceinline__ void accumulate(WT &w, __amdgpu_buffer_rsrc_t ra, __amdgpu_buffer_rsrc_t rb,
                                                    const uint32_t *am, const uint32_t *ak, const uint32_t *bk,
                                                    const uint32_t *bn, int s0, int s1, lds_t<T> *smem,
                                                    const COffsets &co, lds_t<int64_t> *ctab, int tid = int(threadIdx.x)) {
    const int lane = tid & 63, wave = tid >> 6;
    lds_t<T> *const sB = smem + 2 * LoadA::ELEMS;
    const int fa = ((wave / WGN) * WT::WM + (lane & 15)) * LDK + (lane >> 4) * VL;
    const int fb = ((wave % WGN) * WT::WN + (lane & 15)) * LDK + (lane >> 4) * VL;
#pragma unroll
    for (int i = 0; i < WT::FM; ++i)
#pragma unroll
      for (int j = 0; j < WT::FN; ++j) w.acc[i][j] = typename WT::acc_t{0, 0, 0, 0};
    LoadA la;
    LoadB lb;
    la.init(tid, am);
    lb.init(tid, bn);
    // Ahead of the products: LDS holds the next step, registers the one after.
    // (Steps past the summation's end load zeros, past the share's end data
    // that are not used; a loop that leaves them out was 3% faster on FP64's
    // 64 x 64 tile and 10% slower on FP32's 128 x 128.)
    static_assert(BK == 2 * CHUNK, "a step is two chunks");
    la.fetch_k(ak, s0 * BK);
    lb.fetch_k(bk, s0 * BK);
    la.load(ra);
    lb.load(rb);
    la.fetch_k(ak, (s0 + 1) * BK);
    lb.fetch_k(bk, (s0 + 1) * BK);
    la.store(smem);
    lb.store(sB);
    co.store(tid, ctab);
    la.load(ra);
    lb.load(rb);
    la.fetch_k(ak, (s0 + 2) * BK);
    lb.fetch_k(bk, (s0 + 2) * BK);
    __syncthreads();
    constexpr int MORE = SETS > 1 ? SETS - 1 : FOLD > 0 ? 1 : 0;
    Acc more[MORE > 0 ? MORE : 1];
#pragma unroll
    for (int q = 0; q < MORE; ++q)
#pragma unroll
      for (int i = 0; i < WT::FM; ++i)
#pragma unroll
        for (int j = 0; j < WT::FN; ++j) more[q][i][j] = typename WT::acc_t{0, 0, 0, 0};
    int buf = 0;
    auto step = [&](int s) {
      const lds_t<T> *a = smem + buf * LoadA::ELEMS + fa, *b = sB + buf * LoadB::ELEMS + fb;
      mma(w, more, a, b, 0);
      la.store(smem + (buf ^ 1) * LoadA::ELEMS);
      lb.store(sB + (buf ^ 1) * LoadB::ELEMS);
      schedule<0x200, LoadA::WRITES + LoadB::WRITES>();
      __builtin_amdgcn_sched_barrier(0);
      mma(w, more, a, b, 1);
      la.load(ra);
      lb.load(rb);
      schedule<0x20, LoadA::PER + LoadB::PER>();
      __builtin_amdgcn_sched_barrier(0);
      la.fetch_k(ak, (s + 3) * BK);
      lb.fetch_k(bk, (s + 3) * BK);
      __syncthreads();
      buf ^= 1;
    };
    if constexpr (FOLD == 0) {
      for (int s = s0; s < s1; ++s) step(s);
    } else {
      for (int s = s0; s < s1;) {
        const int e = s1 - s < FOLD ? s1 : s + FOLD;
        for (; s < e; ++s) step(s);
#pragma unroll
        for (int i = 0; i < WT::FM; ++i)
#pragma unroll
          for (int j = 0; j < WT::FN; ++j) {
            more[0][i][j] += w.acc[i][j];
            w.acc[i][j] = typename WT::acc_t{0, 0, 0, 0};
          }
      }
    }
    // (pairs of sets, then pairs of those)
#pragma unroll
    for (int d = 1; d < SETS; d *= 2)
#pragma unroll
      for (int q = 0; q < SETS; q += 2 * d)
#pragma unroll
        for (int i = 0; i < WT::FM; ++i)
#pragma unroll
          for (int j = 0; j < WT::FN; ++j) (q ? more[q - 1][i][j] : w.acc[i][j]) += more[q + d - 1][i][j];
    if constexpr (FOLD > 0) {
#pragma unroll
      for (int i = 0; i < WT::FM; ++i)
#pragma unroll
        for (int j = 0; j < WT::FN; ++j) w.acc[i][j] = more[0][i][j];
    }
  }
};

}  // namespace packed
}  // namespace comet
