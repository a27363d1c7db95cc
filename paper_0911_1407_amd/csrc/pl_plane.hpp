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
// What bounds it: a plane runs on one CU, so a grid of fewer planes than CUs by
// that CU's LDS and VALU in turn (96 x 96 FP64: 17500 LDS and 11000 VALU cycles
// of 40000), a batch by how many planes a CU holds.  Measured, us per Hessian
// product before (five passes) and now: 24^3 28.1 / 16.8, 32^3 22.6 / 14.9, 64^3
// 25.9 / 18.3, 96^3 45.6 / 35, 128^3 59.5 / 43.8, 128^3 FP32 47.8 / 33.5,
// 192^3 FP32 109 / 68, 64 x 192 x 96 51.5 / 48.4.  Where few of the largest
// planes leave most CUs idle the separate passes are faster (plane_min_planes).
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
#include <type_traits>

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

// Storage of a row pair: two plane rows of `pitch` complex slots hold the N
// elements of its exchanges, one slot left free after every 2^SHIFT so that
// lanes a radix apart meet different LDS banks.
template <int N>
struct RowPad {
  static constexpr int SHIFT = Plan<N>::R0 >= 16 || N == 192 ? 4 : 3;  // (192: so that 96 x 192 FP64 fits)
  static constexpr int LEN = Plan<N>::P == 1 ? N : N + (N >> SHIFT);
  static constexpr int off(int e) { return e + (e >> SHIFT); }
};
// Complex slots between plane rows of nz cells: the half row (and half a row
// pair's exchange storage), then up to a pitch whose rows fall on different
// banks for the lanes that read a column together.
constexpr int plane_pitch(int nz) {
  switch (nz) {
    case 24: return 14;
    case 32: return 18;
    case 48: return 27;
    case 64: return 36;
    case 96: return 54;
    case 128: return 68;
    case 192: return 102;
    case 256: return 136;
    default: return nz / 2 + 1;
  }
}

// Element positions as compile-time functions (see in_pos / out_pos).
template <class PL, int S>
constexpr int pos_in(int t, int q, int r) {
  return t + PL::P * q + r * (PL::N / StageInfo<PL, S>::R);
}
template <class PL, int S>
constexpr int pos_out(int t, int q, int m) {
  constexpr int R = StageInfo<PL, S>::R, Ns = StageInfo<PL, S>::NS;
  const int j = t + PL::P * q, k = j % Ns;
  return (j - k) * R + k + m * Ns;
}
// Whether OFF(position of slot (q, m)) is a part of the thread's plus a part of
// the slot's, for every thread: then an exchange costs one address per thread
// and the slots are instruction offsets.  (Not so where a radix of 3 or 6 meets
// the padding: the first exchange of the reversed 24, 48, 96 and 192 plans.)
template <class OFF, class PL, int S, bool OUT>
constexpr bool splits() {
  constexpr int R = StageInfo<PL, S>::R;
  for (int t = 0; t < PL::P; ++t)
    for (int q = 0; q < PL::W / R; ++q)
      for (int m = 0; m < R; ++m) {
        const int e = OUT ? pos_out<PL, S>(t, q, m) : pos_in<PL, S>(t, q, m);
        const int et = OUT ? pos_out<PL, S>(t, 0, 0) : pos_in<PL, S>(t, 0, 0);
        const int es = OUT ? pos_out<PL, S>(0, q, m) : pos_in<PL, S>(0, q, m);
        if (OFF::at(e) != OFF::at(et) + OFF::at(es)) return false;
      }
  return true;
}
template <int N>
struct RowOff {
  static constexpr int at(int e) { return RowPad<N>::off(e); }
  __device__ __forceinline__ int operator()(int e) const { return at(e); }
};
// (a column's elements lie `pitch` apart; H: the pitch, or 0 where it is only
// known at run time)
template <int H>
struct ColOff {
  int pitch;
  static constexpr int at(int e) { return e * (H ? H : 1); }
  __device__ __forceinline__ int operator()(int e) const { return e * (H ? H : pitch); }
};

// Move a transform's elements from stage SA's output slots to the input
// slots of stage SB through its LDS storage (off: element -> slot).
template <class PL, int SA, int SB, class OFF, typename T>
__device__ __forceinline__ void wave_exchange(cx<T>* v, int t, cx<T>* lds, const OFF& off) {
  constexpr int RA = StageInfo<PL, SA>::R, RB = StageInfo<PL, SB>::R;
  wave_sync();
  if constexpr (splits<OFF, PL, SA, true>()) {
    cx<T>* to = lds + off(out_pos<PL, SA>(t, 0, 0));
#pragma unroll
    for (int q = 0; q < PL::W / RA; ++q)
#pragma unroll
      for (int m = 0; m < RA; ++m) to[off(out_pos<PL, SA>(0, q, m))] = v[q * RA + m];
  } else {
#pragma unroll
    for (int q = 0; q < PL::W / RA; ++q)
#pragma unroll
      for (int m = 0; m < RA; ++m) lds[off(out_pos<PL, SA>(t, q, m))] = v[q * RA + m];
  }
  wave_sync();
  static_assert(splits<OFF, PL, SB, false>(), "exchange addresses");
  const cx<T>* from = lds + off(in_pos<PL, SB>(t, 0, 0));
#pragma unroll
  for (int q = 0; q < PL::W / RB; ++q)
#pragma unroll
    for (int r = 0; r < RB; ++r) v[q * RB + r] = from[off(in_pos<PL, SB>(0, q, r))];
  wave_sync();
}

// Whole transform by the P lanes of one wave that share it (stage-0 input
// slots to last-stage output slots); lengths with P == 1 stay in registers.
template <class PL, bool INV, class OFF, typename T>
__device__ __forceinline__ void wave_fft(cx<T>* v, int t, cx<T>* lds, const cx<T>* __restrict__ tw, const OFF& off) {
  if constexpr (PL::P == 1) {
    fft_thread<PL, INV, LdsMap<1, false>>(v, t, lds, tw);
  } else {
    // each stage's twiddles are asked for a stage ahead, so that the loads'
    // latency overlaps the exchange (its scheduling fences would put them
    // behind it)
    constexpr int S2 = PL::NS > 2 ? 2 : 1;
    cx<T> w1[StageTw<PL, 1>::LOADS * (PL::W / StageInfo<PL, 1>::R)];
    cx<T> w2[StageTw<PL, S2>::LOADS * (PL::W / StageInfo<PL, S2>::R)];
    stage_twiddles<PL, 1>(w1, t, tw);
    stage_compute<PL, 0, INV>(v, t, tw);
    wave_exchange<PL, 0, 1>(v, t, lds, off);
    if constexpr (PL::NS > 2) stage_twiddles<PL, 2>(w2, t, tw);
    stage_butterflies<PL, 1, INV>(v, w1);
    if constexpr (PL::NS > 2) {
      wave_exchange<PL, 1, 2>(v, t, lds, off);
      stage_butterflies<PL, 2, INV>(v, w2);
    }
  }
}

template <typename T, int N, bool PRE>
struct WaveRowFft {
  using PL = Plan<N>;
  using Fwd = RevPlan<PL>;  // takes over the inverse transform's slots
  // elements whose diagonal is loaded ahead (two values each): none in FP64
  // beside the longer bodies of class 1, which would spill (3 registers too many
  // took the 128 x 128 plane from 22 to 31 us)
  static constexpr int PRELOAD_D = PRE ? PL::W : 0;
  static constexpr bool STREAM = false;
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
    using PX = std::conditional_t<INV, PL, Fwd>;
    wave_fft<PX, INV>(v, per_round(t) & (PL::P - 1), lds, tw, RowOff<N>{});
  }
  __device__ __forceinline__ void turn(cx<T>*) const {}
};

// y transforms of a plane, wave `wave` of `nwaves`.  INV: from the half
// spectrum in memory into the plane in LDS; else from LDS to memory.  HC: the
// half row's length where it is known at compile time (square planes of 32 to 128
// points, the cubes of common use), so that every LDS access is one address and an
// instruction offset; else 0 (a body for every pair of lengths would be too many).
template <typename T, int N, bool INV, int HC>
__device__ __forceinline__ void plane_cols(const cx<T>* __restrict__ src, cx<T>* __restrict__ dst, cx<T>* plane,
                                           int h_, int pitch_, const cx<T>* __restrict__ tw, int wave, int nwaves) {
  using PL = Plan<N>;
  constexpr int P = PL::P, W = PL::W, C = 64 / P, R0 = PL::R0, RL = LastStage<PL>::R;
  constexpr int PC = HC ? plane_pitch(2 * (HC - 1)) : 0;
  const int h = HC ? HC : h_;
  const ColOff<PC> off{pitch_};
  const int lane = threadIdx.x & 63, cl = lane % C;
  for (int g = wave; g * C < h; g += nwaves) {
    const int t = per_round(lane / C) & (P - 1);
    const int c = min(g * C + cl, h - 1);
    cx<T>* col = plane + c;
    const cx<T>* first = col + off(t);
    cx<T> v[W];
#pragma unroll
    for (int q = 0; q < W / R0; ++q)
#pragma unroll
      for (int r = 0; r < R0; ++r) {
        const int e = in_pos<PL, 0>(0, q, r);
        if constexpr (INV)
          v[q * R0 + r] = src[(t + e) * h + c];
        else
          v[q * R0 + r] = first[off(e)];
      }
    wave_fft<PL, INV>(v, t, col, tw, off);
    cx<T>* last = col + off(t);
#pragma unroll
    for (int q = 0; q < W / RL; ++q)
#pragma unroll
      for (int m = 0; m < RL; ++m) {
        const int e = out_pos<PL, PL::NS - 1>(0, q, m);
        if constexpr (INV)
          last[off(e)] = v[q * RL + m];
        else
          dst[(t + e) * h + c] = v[q * RL + m];
      }
  }
}

// z transforms and pointwise work of a plane's row pairs.
template <typename T, int N, int OP, bool PRE>
__device__ __forceinline__ void plane_rows(const RowArgs<T>& a, cx<T>* plane, long row0, int wave, int nwaves,
                                           double (&acc)[2]) {
  using PL = Plan<N>;
  constexpr int P = PL::P, U = 64 / P, H = plane_pitch(N);
  static_assert(2 * H >= RowPad<N>::LEN && H >= N / 2 + 1, "row pair storage");
  const int lane = threadIdx.x & 63, ul = lane / P;
  const int pairs = a.ny >> 1;
  for (int g = wave; g * U < pairs; g += nwaves) {
    const int t = per_round(lane % P) & (P - 1);
    const int u = min(g * U + ul, pairs - 1);
    cx<T>* rows = plane + 2 * u * H;
    const WaveRowFft<T, N, PRE> fx{t, rows, a.tw};
    const long rowA = row0 + 2 * u;
    double part[2] = {0.0, 0.0};
    row_core<T, N, OP>(a, fx, t, true, true, rowA, rowA + 1, rows, rows + H, rows, rows + H, part);
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
#define PL_PLANE_LENGTHS(X) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(192) X(256)
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
constexpr size_t plane_lds_bytes(int ny, int nz, int elem) { return (size_t)ny * plane_pitch(nz) * elem; }
constexpr bool plane_fits(int ny, int nz, int elem) {
  return plane_length(ny) && plane_length(nz) && plane_lds_bytes(ny, nz, elem) <= PLANE_LDS_MAX;
}
void plane_groups(int ny, int nz, int* cols, int* rows);
int plane_waves(int ny, int nz);
int plane_rounds(int ny, int nz);

inline bool plane_len_c0(int n) { return n == 32 || n == 48 || n == 64 || n == 96; }
inline int plane_class(int ny, int nz) { return plane_len_c0(ny) && plane_len_c0(nz) ? 0 : 1; }

// y transforms of a plane for the lengths of class CLS.
template <typename T, bool INV, int CLS>
__device__ __forceinline__ void plane_cols_any(int ny, int nz, const cx<T>* src, cx<T>* dst, cx<T>* plane,
                                               const cx<T>* tw, int wave, int nwaves) {
  const int h = nz / 2 + 1, pitch = plane_pitch(nz);
#define PL_C(NN)                                                                            \
  case NN:                                                                                  \
    if (nz == NN && CLS == (NN == 128))                                                     \
      plane_cols<T, NN, INV, NN / 2 + 1>(src, dst, plane, h, pitch, tw, wave, nwaves);      \
    else                                                                                    \
      plane_cols<T, NN, INV, 0>(src, dst, plane, h, pitch, tw, wave, nwaves);               \
    break;
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
  constexpr bool PRE = sizeof(T) == 4 || CLS == 0;
  const int h = a.n / 2 + 1;
  const long at = (long)plane_id * a.ny * h;
  if constexpr (row_from_half(OP)) {
    if (on) plane_cols_any<T, true, CLS>(a.ny, a.n, a.in_c + at, nullptr, plane, a.tw_y, wave, nwaves);
    __syncthreads();
  }
  if (on) {
#define PL_C(NN) \
  case NN: plane_rows<T, NN, OP, PRE>(a, plane, (long)plane_id * a.ny, wave, nwaves, acc); break;
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
    if (on) plane_cols_any<T, false, CLS>(a.ny, a.n, nullptr, a.out_c + at, plane, a.tw_y, wave, nwaves);
  }
}

// Waves of a single-grid plane pass: as many as there are wave-sized groups
// of columns or row pairs, at most 10 (an FP64 128 x 128 plane: 9 groups of
// columns, 8 of pairs; three waves per SIMD leave 168 registers each).  Planes
// of class 0 have at most 7 groups of either.
constexpr int PLANE_MAX_WAVES = 10;

extern __shared__ __align__(16) char plane_lds[];

template <typename T, int OP, int CLS>
__global__ void __launch_bounds__((CLS == 0 ? 8 : PLANE_MAX_WAVES) * 64) plane_kernel(RowArgs<T> a) {
  if (a.skip && *a.skip != 0.0) return;  // Krylov iteration after convergence
  double acc[2] = {0.0, 0.0};
  plane_body<T, OP, CLS>(a, blockIdx.x, true, reinterpret_cast<cx<T>*>(plane_lds), threadIdx.x >> 6, blockDim.x >> 6, acc);
  if constexpr (row_has_sums(OP)) block_reduce_store<2>(acc, a.partials, blockIdx.x);
}

// Batched plane pass (named by its operation, one of the row pass's, like the
// other batched kernels): a block takes up to `per` planes of one instance, w
// waves each (planes of short rows would leave most of a block idle); work
// item: (instance, first plane, w | per << 8, -).  The sums have a record per
// plane, however the planes are split: a block's go to its first plane's, zeros
// to the others'.
constexpr int PLANE_BATCH_WAVES = 8;

template <typename T, int OP, int CLS>
__global__ void __launch_bounds__(PLANE_BATCH_WAVES * 64) row_batch_kernel(const RowArgs<T>* __restrict__ args,
                                                                            const int4* __restrict__ work) {
  const int4 w = work[blockIdx.x];
  const RowArgs<T> a = args[w.x];
  if (a.skip && *a.skip != 0.0) return;
  const int waves = w.z & 255, wave = threadIdx.x >> 6, slot = wave / waves;
  const int id = w.y + slot;
  const bool on = slot < (w.z >> 8) && id < a.nplanes;
  cx<T>* plane = reinterpret_cast<cx<T>*>(plane_lds) + (on ? slot : 0) * a.ny * plane_pitch(a.n);
  double acc[2] = {0.0, 0.0};
  plane_body<T, OP, CLS>(a, id, on, plane, wave - slot * waves, waves, acc);
  if constexpr (row_has_sums(OP)) {
    block_reduce_store<2>(acc, a.partials, w.y);
    const int others = min(w.z >> 8, a.nplanes - w.y) - 1;
    if ((int)threadIdx.x < 2 * others) a.partials[2 * (w.y + 1) + threadIdx.x] = 0.0;
  }
}

}  // namespace pl
