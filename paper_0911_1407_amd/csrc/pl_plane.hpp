// Plane passes: everything of an operator that stays inside one x plane --
// the y transforms, the z transforms with their pointwise work, and the y
// transforms back -- in one launch, the plane held in LDS throughout.
//
// The passes of pl_kernels.hpp move the half spectrum through memory once per
// axis; on grids whose plane [ny][nz/2 + 1] fits a CU's LDS (128 x 128 in
// FP64, 192 x 192 in FP32) the three passes y, z, y need that only once.
// Small grids gain launches too: what bounds a 32^3 pass is its launch
// (4.4 us), not its 0.3 MB.
//
// Work split: a wave owns 64 / P whole transforms (P threads each, P divides
// 64 for every length), so the exchanges between radix stages stay inside one
// wave and need no workgroup barrier: LDS operations of a wave complete in
// order.  They go through the transform's own storage in the plane (a column's
// ny elements, a row pair's two rows), so a plane needs no LDS beyond itself.
// Waves take transforms in turn; the workgroup meets only between the axes.
// Lanes left over in the last wave's share repeat its last transform step by
// step beside the lanes that own it (the same values to the same places), so
// the code has no branches on them; only their partial sums are dropped.
#pragma once
#include "pl_kernels.hpp"

namespace pl {

// Orders a wave's LDS writes before its later reads by other lanes (the
// hardware keeps the order; this stops the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

// A thread's place in its transform, recomputed for every transform it takes
// part in: left visible as loop-invariant, the twiddles and addresses that
// follow from it would be kept in registers across the loop (spilling).
__device__ __forceinline__ int per_round(int t) {
  asm volatile("" : "+v"(t));
  return t;
}

constexpr int log2_of(int r) { return r <= 1 ? 0 : 1 + log2_of(r / 2); }

// Move a transform's elements from stage SA's output slots to the input
// slots of stage SB through its LDS storage (off: element -> slot).
template <class PL, int SA, int SB, class OFF, typename T>
__device__ __forceinline__ void wave_exchange(cx<T>* v, int t, cx<T>* lds, const OFF& off) {
  constexpr int RA = StageInfo<PL, SA>::R, RB = StageInfo<PL, SB>::R;
  wave_sync();
#pragma unroll
  for (int q = 0; q < PL::W / RA; ++q)
#pragma unroll
    for (int m = 0; m < RA; ++m) lds[off(out_pos<PL, SA>(t, q, m))] = v[q * RA + m];
  wave_sync();
#pragma unroll
  for (int q = 0; q < PL::W / RB; ++q)
#pragma unroll
    for (int r = 0; r < RB; ++r) v[q * RB + r] = lds[off(in_pos<PL, SB>(t, q, r))];
  wave_sync();
}

// Whole transform by the P lanes of one wave that share it (stage-0 input
// slots to last-stage output slots); lengths with P == 1 stay in registers.
template <class PL, bool INV, class OFF, typename T>
__device__ __forceinline__ void wave_fft(cx<T>* v, int t, cx<T>* lds, const cx<T>* __restrict__ tw, const OFF& off) {
  if constexpr (PL::P == 1) {
    fft_thread<PL, INV, LdsMap<1, false>>(v, t, lds, tw);
  } else {
    stage_compute<PL, 0, INV>(v, t, tw);
    if constexpr (PL::NS > 1) {
      wave_exchange<PL, 0, 1>(v, t, lds, off);
      stage_compute<PL, 1, INV>(v, t, tw);
    }
    if constexpr (PL::NS > 2) {
      wave_exchange<PL, 1, 2>(v, t, lds, off);
      stage_compute<PL, 2, INV>(v, t, tw);
    }
  }
}

// A row pair's exchange slots: its two stored rows are one run of N + 2
// complex slots.  The stage-0 writes of neighbouring lanes lie R0 slots
// apart, which would fall on the same LDS banks; exchanging the low three
// bits with the bits above log2(R0) spreads them (a permutation of every
// aligned group of 8, so it stays inside the row).
template <int R0>
struct RowSlot {
  __device__ __forceinline__ int operator()(int e) const { return e ^ ((e >> log2_of(R0)) & 7); }
};

template <typename T, int N>
struct WaveRowFft {
  using PL = Plan<N>;
  // two diagonal values per held element: beyond 8 FP64 elements they would
  // not leave registers for the twiddles
  static constexpr bool PRELOAD_D = sizeof(T) == 4 || PL::W <= 8, STREAM = false;
  // the Gaussian model keeps the row passes: its log1p beside the exp left
  // the plane's gradient kernels 172-468 spilled registers
  static constexpr bool GAUSS = false;
  int t;
  cx<T>* lds;
  const cx<T>* tw;
  // Called after each element of the loops that read two operands per
  // element: all their loads in flight at once would need twice the
  // registers of the transform, for LDS reads that are short.
  __device__ __forceinline__ void chunk(int i) const {
    if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
  }
  // The sums are up to date here (see row_core).
  __device__ __forceinline__ void pin(double (&acc)[2]) const { asm volatile("" : "+v"(acc[0]), "+v"(acc[1])); }
  template <bool INV>
  __device__ __forceinline__ void fft(cx<T>* v) const {
    wave_fft<PL, INV>(v, per_round(t), lds, tw, RowSlot<PL::R0>{});
  }
  __device__ __forceinline__ void turn(cx<T>* v) const {
    constexpr int RL = LastStage<PL>::R;
    if constexpr (RL == PL::R0) {
    } else if constexpr (PL::P == 1) {
      last_to_first<PL, LdsMap<1, false>>(v, t, lds);
    } else {
      wave_exchange<PL, PL::NS - 1, 0>(v, t, lds, RowSlot<PL::R0>{});
    }
  }
};

// y transforms of a plane, wave `wave` of `nwaves`.  INV: from the half
// spectrum in memory into the plane in LDS; else from LDS to memory.
template <typename T, int N, bool INV>
__device__ __forceinline__ void plane_cols(const cx<T>* __restrict__ src, cx<T>* __restrict__ dst, cx<T>* plane, int h,
                                           const cx<T>* __restrict__ tw, int wave, int nwaves) {
  using PL = Plan<N>;
  constexpr int P = PL::P, W = PL::W, C = 64 / P, R0 = PL::R0, RL = LastStage<PL>::R;
  const int lane = threadIdx.x & 63, cl = lane % C;
  const auto off = [h](int e) { return e * h; };
  for (int g = wave; g * C < h; g += nwaves) {
    const int t = per_round(lane / C);
    const int c = min(g * C + cl, h - 1);
    cx<T>* col = plane + c;
    cx<T> v[W];
#pragma unroll
    for (int q = 0; q < W / R0; ++q)
#pragma unroll
      for (int r = 0; r < R0; ++r) {
        const int e = in_pos<PL, 0>(t, q, r);
        if constexpr (INV)
          v[q * R0 + r] = src[e * h + c];
        else
          v[q * R0 + r] = col[e * h];
      }
    wave_fft<PL, INV>(v, t, col, tw, off);
#pragma unroll
    for (int q = 0; q < W / RL; ++q)
#pragma unroll
      for (int m = 0; m < RL; ++m) {
        const int e = out_pos<PL, PL::NS - 1>(t, q, m);
        if constexpr (INV)
          col[e * h] = v[q * RL + m];
        else
          dst[e * h + c] = v[q * RL + m];
      }
  }
}

// z transforms and pointwise work of a plane's row pairs.
template <typename T, int N, int OP>
__device__ __forceinline__ void plane_rows(const RowArgs<T>& a, cx<T>* plane, long row0, int wave, int nwaves,
                                           double (&acc)[2]) {
  using PL = Plan<N>;
  constexpr int P = PL::P, U = 64 / P, H = N / 2 + 1;
  const int lane = threadIdx.x & 63, ul = lane / P;
  const int pairs = a.ny >> 1;
  for (int g = wave; g * U < pairs; g += nwaves) {
    const int t = per_round(lane % P);
    const int u = min(g * U + ul, pairs - 1);
    cx<T>* rows = plane + 2 * u * H;
    const WaveRowFft<T, N> fx{t, rows, a.tw};
    const long rowA = row0 + 2 * u;
    double part[2] = {0.0, 0.0};
    row_core<T, N, OP>(a, fx, t, true, true, rowA, rowA + 1, rows, rows, part);
    if (g * U + ul < pairs) {
      acc[0] += part[0];
      acc[1] += part[1];
    }
  }
}

// Lengths of the plane passes (y and z independently), in two classes, each a
// kernel of its own: a kernel's registers are those of its largest body, and
// the bodies of 16 and more values per thread (FP64: 156 registers) would hold
// the planes of the shorter lengths (128) to their occupancy.
#define PL_PLANE_LENGTHS_C0(X) X(32) X(48) X(64) X(96)
#define PL_PLANE_LENGTHS(X) X(8) X(12) X(16) X(32) X(48) X(64) X(96) X(128) X(256)
constexpr bool plane_length(int n) {
  switch (n) {
#define PL_C(NN) case NN: return true;
    PL_PLANE_LENGTHS(PL_C)
#undef PL_C
    default: return false;
  }
}
// Planes a workgroup can hold: the lengths above, within a CU's 160 KB of LDS
// less the block sums.
constexpr size_t PLANE_LDS_MAX = 163840 - 512;
constexpr size_t plane_lds_bytes(int ny, int nz, int elem) { return (size_t)ny * (nz / 2 + 1) * elem; }
constexpr bool plane_fits(int ny, int nz, int elem) {
  return plane_length(ny) && plane_length(nz) && plane_lds_bytes(ny, nz, elem) <= PLANE_LDS_MAX;
}
int plane_waves(int ny, int nz);

inline bool plane_len_c0(int n) { return n == 32 || n == 48 || n == 64 || n == 96; }
inline int plane_class(int ny, int nz) { return plane_len_c0(ny) && plane_len_c0(nz) ? 0 : 1; }

// y transforms of a plane for the lengths of class CLS.
template <typename T, bool INV, int CLS>
__device__ __forceinline__ void plane_cols_any(int ny, const cx<T>* src, cx<T>* dst, cx<T>* plane, int h,
                                               const cx<T>* tw, int wave, int nwaves) {
#define PL_C(NN) \
  case NN: plane_cols<T, NN, INV>(src, dst, plane, h, tw, wave, nwaves); break;
  if constexpr (CLS == 0) {
    switch (ny) {
      PL_PLANE_LENGTHS_C0(PL_C)
      default: break;
    }
  } else {
    switch (ny) {
      PL_PLANE_LENGTHS(PL_C)
      default: break;
    }
  }
#undef PL_C
}

// One plane: y inverse (for operations that start from half rows), z, y
// forward (for those that end in them).  All waves of the workgroup call this
// together (it holds barriers); `on` is false where a slot has no plane.
template <typename T, int OP, int CLS>
__device__ __forceinline__ void plane_body(const RowArgs<T>& a, int plane_id, bool on, cx<T>* plane, int wave,
                                           int nwaves, double (&acc)[2]) {
  const int h = a.n / 2 + 1;
  const long at = (long)plane_id * a.ny * h;
  if constexpr (row_from_half(OP)) {
    if (on) plane_cols_any<T, true, CLS>(a.ny, a.in_c + at, nullptr, plane, h, a.tw_y, wave, nwaves);
    __syncthreads();
  }
  if (on) {
#define PL_C(NN) \
  case NN: plane_rows<T, NN, OP>(a, plane, (long)plane_id * a.ny, wave, nwaves, acc); break;
    if constexpr (CLS == 0) {
      switch (a.n) {
        PL_PLANE_LENGTHS_C0(PL_C)
        default: break;
      }
    } else {
      switch (a.n) {
        PL_PLANE_LENGTHS(PL_C)
        default: break;
      }
    }
#undef PL_C
  }
  if constexpr (row_to_half(OP)) {
    __syncthreads();
    if (on) plane_cols_any<T, false, CLS>(a.ny, nullptr, a.out_c + at, plane, h, a.tw_y, wave, nwaves);
  }
}

// Waves of a single-grid plane pass: as many as there are wave-sized groups
// of columns or row pairs, at most 10 (an FP64 128 x 128 plane: 9 groups of
// columns, 8 of pairs; three waves per SIMD leave 168 registers each).
constexpr int PLANE_MAX_WAVES = 10;

extern __shared__ __align__(16) char plane_lds[];

template <typename T, int OP, int CLS>
__global__ void __launch_bounds__(PLANE_MAX_WAVES * 64) plane_kernel(RowArgs<T> a) {
  if (a.skip && *a.skip != 0.0) return;  // Krylov iteration after convergence
  double acc[2] = {0.0, 0.0};
  plane_body<T, OP, CLS>(a, blockIdx.x, true, reinterpret_cast<cx<T>*>(plane_lds), threadIdx.x >> 6, blockDim.x >> 6, acc);
  if constexpr (row_has_sums(OP)) block_reduce_store<2>(acc, a.partials, blockIdx.x);
}

}  // namespace pl
