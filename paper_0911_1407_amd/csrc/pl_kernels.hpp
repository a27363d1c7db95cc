// Kernel templates of the Poisson-lognormal MAP hot path.
//
// Layouts (row-major, z fastest, as numpy):
//   real field      [nx][ny][nz]            N = nx ny nz values
//   half spectrum   [nx][ny][nz/2 + 1]      Nh complex values (interleaved)
// Forward transforms are unnormalised (X_k = sum_x x_x e^{-2 pi i m.x/n});
// inverse transforms are unnormalised too and callers pass 1/N as `scale`.
//
// Passes:
//   col_kernel  -- FFT along x or y of the half spectrum, one workgroup per
//                  tile of B adjacent columns (coalesced B*16 byte segments
//                  per row in FP64), optional fused spectral operations on
//                  the x pass (prior multiply, prior add + dots).
//   row_kernel  -- the z axis: real <-> half-complex transforms of two rows
//                  at once (row a in the real part, row b in the imaginary
//                  part of one complex length-nz transform), with fused
//                  pointwise likelihood / Hessian-diagonal work.
#pragma once
#include "pl_fft.hpp"

namespace pl {

constexpr int RED_THREADS = 256;

// Streaming loads: operands read once per pass and not again until the next
// Krylov step can be loaded non-temporally, so that they do not displace
// the pass-to-pass intermediate (each pass's input and output, default
// policy) from the memory-side cache.  The nt field of the pass arguments
// holds one bit per array, covering its loads and stores in the Krylov and
// operator passes: NT_R (residual r), NT_P (direction p, and the operator's
// input), NT_X (iterate x), NT_TAB (per-mode 1/lambda table), NT_DIAG
// (Hessian diagonal).  Which arrays are worth keeping cached beside the
// intermediate depends on their size against the cache (all streamed at
// 256^3 in FP64; r, read twice and written once per step, kept in FP32), so
// the bits are a per-plan schedule choice.  The intermediate keeps the
// default policy.
enum { NT_R = 1, NT_P = 2, NT_X = 4, NT_TAB = 8, NT_DIAG = 16, NT_ALL = 31 };

// Posterior model of a solve: the lognormal prior on s = ln(1 + delta) with
// the power-law bias (section 2.3, 2.4), or the Gaussian prior on delta with
// unit bias (section 2.2.2, eq. MAPG).
enum { MODEL_LOGNORMAL = 0, MODEL_GAUSSIAN = 1 };
template <typename T>
__device__ __forceinline__ T ld_stream(const T* p, int nt) {
  return nt ? __builtin_nontemporal_load(p) : *p;
}
template <typename T>
__device__ __forceinline__ void st_stream(cx<T>* p, cx<T> v, int nt) {
  if (nt) {
    typedef T v2 __attribute__((ext_vector_type(2)));
    v2 x;
    x.x = v.x;
    x.y = v.y;
    __builtin_nontemporal_store(x, reinterpret_cast<v2*>(p));
  } else {
    *p = v;
  }
}
template <typename T>
__device__ __forceinline__ cx<T> ld_stream(const cx<T>* p, int nt) {
  if (nt) {
    typedef T v2 __attribute__((ext_vector_type(2)));
    const v2 x = __builtin_nontemporal_load(reinterpret_cast<const v2*>(p));
    return {x.x, x.y};
  }
  return *p;
}

// ---------------------------------------------------------------------------
// Reductions: per-block partial sums in FP64, summed in a fixed order by a
// separate finalize kernel (deterministic).
// ---------------------------------------------------------------------------

template <int K>
__device__ __forceinline__ void block_reduce_store(double (&v)[K], double* __restrict__ partials,
                                                   int block_linear) {
  __shared__ double sh[K][16];
#pragma unroll
  for (int k = 0; k < K; ++k) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_down(v[k], off, 64);
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int nw = (blockDim.x + 63) >> 6;
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) sh[k][wid] = v[k];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      double acc = 0.0;
      for (int i = 0; i < nw; ++i) acc += sh[k][i];
      partials[(size_t)block_linear * K + k] = acc;
    }
  }
}

// Whether a queued Krylov iteration is to be left out (*skip set), as one
// lane reads it for its whole workgroup: workgroup 0 of the launch, or one
// riding on it, may be storing the flag meanwhile, and waves that read it for
// themselves could part, some leaving and the others going on with sums that
// the leavers never stored.  Either reading is right for a whole workgroup
// (one that goes on finds the same end from the same sums).
__device__ __forceinline__ bool block_skips(const double* skip) {
  if (!skip) return false;
  __shared__ int off;
  if (threadIdx.x == 0) off = *skip != 0.0;
  __syncthreads();
  return off != 0;
}

// Spectral bookkeeping for the half spectrum [nx][ny][h], h = nz/2 + 1.
struct Grid {
  int nx, ny, nz, h;
  long nyh;  // ny * h
};

__device__ __forceinline__ int fold(int m, int n) { return m >= (n >> 1) ? m - n : m; }

// Ways to look up 1/lambda_k (inv_lam_at).
enum TabKind {
  TAB_MODE = 0,    // per-mode table [nx][ny][h], entry `mode`
  TAB_SHELL = 1,   // radial shell table indexed by mx^2 + my^2 + mz^2 (cubic box)
  TAB_MIRROR = 2,  // per-mode table read at (min(kx, nx - kx), ky, kz): for a
                   // spectrum even in kx (a radial one), whose entries at kx
                   // and nx - kx agree; an x pass then reads each table entry
                   // for two modes of one column, and the upper half never
};

// 1/lambda_k (section 2.3: S_L^-1 is diagonal in Fourier space).
template <typename TT>
__device__ __forceinline__ TT inv_lam_at(const TT* __restrict__ tab, int kind, const Grid& g,
                                         int kx, int ky, int kz, long mode, int nt = 0) {
  if (kind == TAB_SHELL) {
    int fx = fold(kx, g.nx), fy = fold(ky, g.ny);
    return tab[fx * fx + fy * fy + kz * kz];
  }
  if (kind == TAB_MIRROR) {
    const int mx = 2 * kx > g.nx ? g.nx - kx : kx;
    return ld_stream(tab + ((long)mx * g.nyh + mode - (long)kx * g.nyh), nt);
  }
  return ld_stream(tab + mode, nt);
}

__device__ __forceinline__ double herm_w(int kz, const Grid& g) {
  return (kz == 0 || 2 * kz == g.nz) ? 1.0 : 2.0;
}

// Device scalar slots
enum Scal {
  SC_RZ = 0,      // r^H M^-1 r
  SC_PQ = 1,      // p^H H p
  SC_ALPHA = 2,   // CG step
  SC_BETA = 3,    // CG direction update
  SC_RR = 4,      // r^H r
  SC_TOL2 = 5,    // stop when r^H r <= TOL2
  SC_DONE = 6,    // 0 running, 1 converged / capped, 2 breakdown
  SC_ITS = 7,     // CG iterations that changed the iterate
  SC_DBAR = 8,    // mean of the Hessian diagonal (preconditioner)
  SC_RR0 = 9,     // r^H r of the initial residual
  SC_JUNK = 10,   // sink for an unused partial
  SC_GG = 11, SC_PRIOR = 12, SC_LIK = 13, SC_DSUM = 14,
  SC_INACTIVE = 15,  // batched solves: instance finished, every pass skips it
  SC_LS_B = 16, SC_LS_C = 17, SC_LS_SLOPE = 18,
  SC_RZ_ODD = 19,  // r^H M^-1 r after an odd number of CG iterations (cg_rz_slot)
  SC_DF = 20,     // 4 slots
  SC_LS_ALPHA = 24,  // step the device-side Armijo test accepted (-1: none)
  SC_ALPHA_ODD = 25,  // CG step length taken after an odd number of iterations (cg_alpha_slot)
  SC_ADJ = 26,    // adjoint sums (4 slots)
  SC_LB_DQ = 30,  // linear-bias Krylov step: sum of phi'' B u q^2 (the diagonal part of p^H H p)
  SC_TOL_REL2 = 31,  // square of a CG tolerance relative to the first residual (0: SC_TOL2 is given)
  SC_GAMMA = 32,    // r^H M^-1 r of the running iteration (two-pass CG)
  SC_COUNT = 40
};

// The single-plan CG keeps r^H M^-1 r after k completed iterations in
// slot cg_rz_slot(k): the first pass of iteration k reads slot k - 1 to form
// beta while one of its workgroups stores slot k.
__host__ __device__ constexpr int cg_rz_slot(int k) { return (k & 1) ? SC_RZ_ODD : SC_RZ; }
// Likewise the step length of the iteration after k completed ones: the next
// iteration reads it while it stores its own.
__host__ __device__ constexpr int cg_alpha_slot(int k) { return (k & 1) ? SC_ALPHA_ODD : SC_ALPHA; }

// The scalars of one CG iteration in the single-reduction form (Chronopoulos
// and Gear 1989): with u = M^-1 r, gamma = r^H u and delta = u^H H u,
//   beta = gamma / gamma_old,  alpha = gamma / (delta - beta gamma / alpha_old)
// (the denominator is p^H H p of p = u + beta p_old).  Both sums are known
// before the pass that needs them, so one x pass per iteration does all vector
// updates.  k: iterations completed; rr = r^H r.  STORE: also the bookkeeping
// for the next iteration and the host.  Returns whether the solve is over.
template <bool STORE>
__device__ __forceinline__ bool cg_scalars(double* scal, double delta, double gamma, double rr, int k, double k_max,
                                           double tol_rel2, double* alpha, double* beta) {
  // a tolerance relative to the first residual is known from the first pass on
  const double tol2 = k == 0 && tol_rel2 > 0.0 ? tol_rel2 * rr : scal[SC_TOL2];
  double b = 0.0, pq = delta;
  if (k > 0) {
    const double g_old = scal[cg_rz_slot(k - 1)], a_old = scal[cg_alpha_slot(k - 1)];
    b = g_old > 0.0 ? gamma / g_old : 0.0;
    pq = a_old != 0.0 ? delta - b * gamma / a_old : delta;
  }
  const bool end = rr <= tol2 || (double)k >= k_max;
  const bool bad = !end && !(pq > 0.0);  // breakdown
  *alpha = end || bad ? 0.0 : gamma / pq;
  *beta = b;
  if (STORE) {
    if (k == 0) {
      scal[SC_RR0] = rr;
      // (a given tolerance stays untouched: other workgroups read it)
      if (tol_rel2 > 0.0) scal[SC_TOL2] = tol2;
    }
    scal[SC_ITS] = (double)k;
    scal[SC_RR] = rr;
    scal[SC_PQ] = pq;
    scal[SC_BETA] = b;
    scal[cg_rz_slot(k)] = gamma;
    scal[cg_alpha_slot(k)] = *alpha;
    if (end || bad) scal[SC_DONE] = end ? 1.0 : 2.0;
  }
  return end || bad;
}

// Inverse of the preconditioner M_k = 1/lambda_k + dbar (dbar a constant
// taken from the Hessian diagonal d), in the Krylov vectors' precision:
// FP64 vectors take the IEEE quotient, FP32 vectors the hardware
// reciprocal.  Every pass that applies M^-1 calls this one function, so M
// is the same operator throughout a solve.
template <typename T>
__device__ __forceinline__ T precond_inv(T il, double dbar) {
  const T m = il + (T)dbar;
  if constexpr (sizeof(T) == 4) {
    return m > 0.0f ? __builtin_amdgcn_rcpf(m) : 0.0f;
  } else {
    return m > 0.0 ? 1.0 / m : 0.0;
  }
}

// u = M^-1 r at one mode and its shares of (u^H Lambda^-1 u, r^H u, r^H r):
// vector arithmetic in the Krylov vectors' precision, sums in FP64, and the
// squares of r too: a right-hand side has the caller's scale, whose squares
// FP32 need not hold (1e-24 squares to zero, 1e20 to infinity).
template <typename T>
__device__ __forceinline__ void cg_precondition(cx<T> r, T il, double dbar, double hw, cx<T>& u, double (&acc)[3]) {
  const T mi = precond_inv<T>(il, dbar);
  u = {mi * r.x, mi * r.y};
  const double rr = (double)r.x * r.x + (double)r.y * r.y;
  acc[0] += hw * (double)(il * (u.x * u.x + u.y * u.y));
  acc[1] += hw * ((double)mi * rr);
  acc[2] += hw * rr;
}

// The step length of one iteration in the textbook order (two x passes per
// iteration): alpha = gamma / p^H H p with p^H H p = pi + dv (the prior part
// from the first x pass, the diagonal part from the z or plane pass).  first:
// the iteration whose first pass was COL_CG_INIT, with gamma and rr from its
// sums; otherwise gamma is SC_GAMMA.  Returns whether the solve is over.
template <bool STORE>
__device__ __forceinline__ bool cg_alpha(double* scal, bool first, double pi, double dv, double gamma, double rr,
                                         double tol_rel2, double* alpha) {
  bool end = false;
  if (first) {
    const double tol2 = tol_rel2 > 0.0 ? tol_rel2 * rr : scal[SC_TOL2];
    end = rr <= tol2;  // converged at the start: x stays 0
    if (STORE) {
      if (tol_rel2 > 0.0) scal[SC_TOL2] = tol2;
      scal[SC_RR0] = scal[SC_RR] = rr;
      scal[cg_rz_slot(0)] = gamma;
      scal[SC_ITS] = 0.0;
    }
  } else {
    gamma = scal[SC_GAMMA];
  }
  const double pq = pi + dv;
  const bool bad = !end && !(pq > 0.0);  // breakdown
  *alpha = end || bad ? 0.0 : gamma / pq;
  if (STORE) {
    scal[SC_PQ] = pq;
    scal[SC_ALPHA] = *alpha;
    if (end || bad) scal[SC_DONE] = end ? 1.0 : 2.0;
  }
  return end || bad;
}

// ---------------------------------------------------------------------------
// Column pass (x or y axis)
// ---------------------------------------------------------------------------

enum ColOp {
  COL_PLAIN = 0,     // transform only
  COL_PRIOR = 1,     // forward, times 1/lambda, inverse (partials K = 1)
  COL_ADDPRIOR = 2,  // forward; out = X + (1/lambda) base (partials K = 3)
  COL_CG_FIRST = 3,  // CG prologue on the input, then inverse transform (partials K = 1)
  COL_CG_LAST = 4,   // forward; q = X + p/lambda; r -= alpha q (partials K = 2)
  COL_CG_INIT = 5,   // r = sign * rhs; u = M^-1 r, then its inverse transform
                     // (partials K = 3: u^H Lambda^-1 u, r^H u, r^H r)
  COL_CG_STEP = 6    // one CG iteration's x pass (forward transform, all vector
                     // updates, inverse transform of the next u; partials as COL_CG_INIT)
};

// Arguments of one finalize (finalize_body): sums of per-block partials and
// the scalar bookkeeping of kind FIN_*.
struct FinArgs {
  const double* partials;
  int nb, K, kind, dst;
  double scale;
  double* scal;
  double aux;
  const double* partials2;
  int nb2;
  double scale2;
};

template <int NT, bool DEVCOUNT = false>
__device__ __forceinline__ void finalize_body(const double* __restrict__ partials, int nb, int K, int kind, int dst,
                                              double scale, double* __restrict__ scal, double aux,
                                              const double* __restrict__ partials2, int nb2, double scale2);
template <int NT, int K>
__device__ __forceinline__ void fin_sums(const double* __restrict__ src, int n, double* out);

template <typename T>
struct ColArgs {
  int n;             // transform length
  const cx<T>* in;
  cx<T>* out;
  int ncols;         // columns per slab
  long row_stride;   // distance (complex elements) between consecutive transform entries
  long slab_stride;  // distance between slabs (blockIdx.y)
  const cx<T>* tw;   // twiddles of this length
  // fused x-pass operations (columns are flattened (ky, kz) pairs)
  Grid g;
  const T* inv_lam;  // 1/lambda table (see inv_lam_at)
  int radial;        // its TabKind
  const cx<T>* base;  // COL_ADDPRIOR: vector added through the prior
  double k0_shift;    // subtracted from mode 0 before the prior multiply
  T out_scale;        // COL_ADDPRIOR: scale of the transformed input
  double* partials;   // per-block partial sums
  // Krylov operands (COL_CG_FIRST / COL_CG_LAST), same layout as the input
  cx<T>* cg_r;
  cx<T>* cg_x;
  const double* scal;  // device scalars (SC_*)
  const double* skip;  // if non-null and *skip != 0 the launch does nothing
  int nt;              // NT_* bits: operands loaded / stored non-temporally
  // COL_CG_INIT: the right-hand side, r = cg_rhs_sign * cg_rhs
  const cx<double>* cg_rhs;
  double cg_rhs_sign;
  int variant;  // batched launches: this instance's tile variant (0 or 2)
  // COL_CG_FIRST with beta_part set: the pass itself closes iteration
  // cg_k - 1 from that iteration's last-pass partials (beta_nb blocks of
  // (r^H r, r^H M^-1 r), times beta_scale): every workgroup sums them in the
  // same order, so all take the same beta and the same convergence
  // decision, and workgroup 0 stores the bookkeeping (SC_ITS = cg_k, SC_RR,
  // cg_rz_slot(cg_k), SC_BETA, SC_DONE when r^H r <= SC_TOL2 or cg_k >=
  // cg_max), in place of a finalize launch of its own
  const double* beta_part;
  int beta_nb;
  double beta_scale;
  int cg_k;
  double cg_max;
  // COL_CG_STEP: cg_p = u + beta cg_p and cg_y = F[d v] + beta cg_y
  // (its share of H p through the diagonal; both unread in the first iteration), cg_r, and on every second iteration
  // cg_x.  With z_part set (sums of d v^2 left by z_nb blocks of the z or
  // plane pass; beta_part then holds the previous x pass's sums of three)
  // every workgroup forms the iteration's scalars itself and workgroup 0
  // stores them; else they are in scal.
  cx<T>* cg_p;
  cx<T>* cg_y;
  const double* z_part;
  int z_nb;
  double tol_rel2;
  // COL_PLAIN launches with fin_on = 1 carry one extra workgroup that runs
  // the finalize `fin` (saving a launch of its own); the host adds it to the
  // grid
  int fin_on;
  FinArgs fin;
};

// Column tile width B: 256 threads per block where possible, at most 64 KB
// of LDS for the stage exchanges, at least 8 columns (128-byte segments).
// Tile variants: V = 0 aims at 256 threads and at most 64 KB of LDS; V = 1
// ("wide") at 512 threads and at most 128 KB, i.e. longer contiguous row
// segments per tile at lower occupancy.  Which wins depends on the length
// and precision; the plan picks one per pass (see pl_plan_autotune).
constexpr int col_tile(int P, int N, int elem_bytes, int threads, int lds_cap) {
  int b = threads / P;
  if (b > 64) b = 64;
  if (b < 8) b = 8;
  while (b > 8 && P > 1 && b * N * elem_bytes > lds_cap) b /= 2;
  return b;
}

// V = 2 ("narrow"): 128 threads and at most 32 KB, for batches of small grids
// and for x passes of few columns (see x_tile).
// V = 3 ("split"): the default tile, with the stage exchanges passing real
// and imaginary parts through LDS one after the other (half the LDS, so
// twice the blocks per CU when registers allow) and the second operand of
// the fused x passes loaded after the transform (fewer registers).
// V = 4 ("extra wide"): 1024 threads and at most 160 KB, one block per CU
// with the longest row segments (256 bytes of FP32 columns at 512 points).
// V = 5 ("wide split"): 512 threads, split exchanges in at most 64 KB:
// the wide tile's row segments (512 bytes of FP64 columns at 256 points)
// at two blocks per CU.  V = 6 ("extra wide split"): 1024 threads, split
// exchanges in at most 128 KB (1 KB segments of FP64 at 256 points).
constexpr int col_threads(int V) {
  return V == 1 || V == 5 ? 512 : (V == 2 ? 128 : (V == 4 || V == 6 ? 1024 : (V == 7 ? 64 : 256)));
}
constexpr int col_lds_cap(int V) {
  return V == 1 || V == 6 ? 131072 : (V == 2 || V == 7 ? 32768 : (V == 4 ? 163840 : 65536));
}
// V = 7 ("one wave"): 64 threads, for the x passes of small grids (see x_tile).
constexpr bool col_split(int V) { return V == 3 || V == 5 || V == 6; }

template <typename T, int N, int V = 0>
struct ColShape {
  static constexpr int P = Plan<N>::P;
  static constexpr bool SPLIT = col_split(V);
  // a split exchange holds one real part per element at a time
  static constexpr int B = col_tile(P, N, (int)sizeof(cx<T>) / (SPLIT ? 2 : 1), col_threads(V), col_lds_cap(V));
  static constexpr int THREADS = B * P;
  static constexpr int LDS = P > 1 ? (SPLIT ? (N * B + 1) / 2 : N * B) : 1;  // complex elements
};

// lengths with a wide variant
constexpr bool has_wide_variant(int n) { return n == 128 || n == 192 || n == 256 || n == 512; }

// Sums of K interleaved per-block partials by a column pass's workgroup.  (A
// batched launch may give a tile a larger block than its own.)
template <typename T, int N, int V, bool BATCHED, int K>
__device__ __forceinline__ void col_sums(const double* __restrict__ src, int n, double* out) {
  if constexpr (BATCHED) {
    if (blockDim.x == 256)
      fin_sums<256, K>(src, n, out);
    else
      fin_sums<128, K>(src, n, out);
  } else {
    fin_sums<ColShape<T, N, V>::THREADS, K>(src, n, out);
  }
}

// One workgroup's share of a column pass: tile `tile` of slab `slab`.
// Threads beyond ColShape::THREADS (when a batched launch uses a larger
// block) only take part in the barriers.
template <typename T, int N, bool INV, int OP, int V = 0, bool BATCHED = false>
__device__ __forceinline__ void col_body(const ColArgs<T>& a, int tile, int slab,
                                         cx<T>* lds_all, int block_linear) {
  using PL = Plan<N>;
  constexpr int B = ColShape<T, N, V>::B;
  constexpr int P = PL::P;
  constexpr int W = PL::W;
  constexpr int R0 = PL::R0;
  constexpr int RL = LastStage<PL>::R;
  using MAP = LdsMap<B, false>;
  // The x passes that add (1/lambda) times a second operand load it and the
  // table before the transform, so that their latency overlaps it, unless
  // the extra registers would cost occupancy (FP32 at 512 points: 146
  // instead of about 90 VGPRs, 3 instead of 4 waves per SIMD; the split
  // tile; 1024-thread blocks, held to 128 VGPRs); the other FP64 passes are
  // held to 2 waves per SIMD by their LDS either way.  Batched launches
  // (BATCHED) never preload: one kernel serves every length of the batch,
  // so its registers are those of the largest body, and the 96-point body
  // (24 values per thread) with preloading needs 173 (FP32) to 256 (FP64)
  // VGPRs, which would hold the blocks of every length to 1-2 waves per SIMD.
  constexpr bool SPLIT = ColShape<T, N, V>::SPLIT;
  constexpr bool PRELOAD = !BATCHED && !(sizeof(T) == 4 && N >= 512) && !SPLIT && ColShape<T, N, V>::THREADS <= 512;

  const bool active = (int)threadIdx.x < ColShape<T, N, V>::THREADS;
  const int cl = threadIdx.x % B;
  const int t = active ? (int)threadIdx.x / B : 0;
  const int c = tile * B + cl;
  const bool valid = active && c < a.ncols;
  const long base_off = (long)slab * a.slab_stride + (valid ? c : 0);
  // the fused operations run on x passes: the column fixes (ky, kz), the
  // transform position is kx, and an element's mode index is its offset
  const int col_ky = c / a.g.h, col_kz = c % a.g.h;
  // column cl's slots: complex elements, or with SPLIT real ones
  cx<T>* lds = SPLIT ? reinterpret_cast<cx<T>*>(reinterpret_cast<T*>(lds_all) + cl) : lds_all + cl;

  cx<T> v[W];
  if constexpr (OP == COL_CG_INIT) {
    const double dbar = a.scal[SC_DBAR];
    const double hw = herm_w(col_kz, a.g);
    double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < W / R0; ++q)
#pragma unroll
      for (int r = 0; r < R0; ++r) {
        const int kx = in_pos<PL, 0>(t, q, r);
        const long mode = base_off + (long)kx * a.row_stride;
        cx<T> u = {T(0), T(0)};
        if (valid) {
          const T il = inv_lam_at(a.inv_lam, a.radial, a.g, kx, col_ky, col_kz, mode, a.nt & NT_TAB);
          const cx<double> b = a.cg_rhs[mode];
          const cx<T> rv = {(T)(a.cg_rhs_sign * b.x), (T)(a.cg_rhs_sign * b.y)};
          st_stream(a.cg_r + mode, rv, a.nt & NT_R);
          cg_precondition<T>(rv, il, dbar, hw, u, acc);
          if (a.cg_p) {  // two-pass CG: p = u, x = 0
            st_stream(a.cg_p + mode, u, a.nt & NT_P);
            st_stream(a.cg_x + mode, cx<T>{T(0), T(0)}, a.nt & NT_X);
          }
        }
        v[q * R0 + r] = u;
      }
    fft_thread<PL, true, MAP, SPLIT>(v, t, lds, a.tw, active);
    block_reduce_store<3>(acc, a.partials, block_linear);
  } else if constexpr (OP == COL_CG_FIRST) {
    // Krylov prologue on the x pass of a half spectrum (columns = (ky, kz)):
    //   p = M^-1 r + beta p_old (in place), partial sum of p^H Lambda^-1 p;
    // then the inverse transform of p.
    const double dbar = a.scal[SC_DBAR];
    const int kz = col_kz;
    const double hw = herm_w(kz, a.g);
    double acc[1] = {0.0};
    cx<T>* pio = const_cast<cx<T>*>(a.in);
    {
      double beta_k = 0.0;
      int cg_k = a.cg_k;
      const double* beta_part = a.beta_part;
      if constexpr (BATCHED) {
        // instances at different iteration counts under one launch: the
        // count is the instance's SC_ITS, which the last pass advances
        // after each iteration (so this launch only reads it); at 0 there
        // is no previous iteration to close (beta = 0)
        cg_k = (int)a.scal[SC_ITS];
        if (cg_k == 0) beta_part = nullptr;
      }
      if (beta_part) {
        double v2[2];
        col_sums<T, N, V, BATCHED, 2>(beta_part, a.beta_nb, v2);
        const double rr = v2[0] * a.beta_scale, rz = v2[1] * a.beta_scale;
        const double rzo = a.scal[cg_rz_slot(cg_k - 1)];
        beta_k = rzo > 0.0 ? rz / rzo : 0.0;
        const bool done = rr <= a.scal[SC_TOL2] || (double)cg_k >= a.cg_max;
        if (block_linear == 0 && threadIdx.x == 0) {
          double* sc = const_cast<double*>(a.scal);
          if constexpr (!BATCHED) sc[SC_ITS] = (double)cg_k;
          sc[SC_RR] = rr;
          sc[cg_rz_slot(cg_k)] = rz;
          sc[SC_GAMMA] = rz;
          sc[SC_BETA] = beta_k;
          if (done) sc[SC_DONE] = 1.0;
        }
        if (done) return;  // the whole workgroup (every one decides alike)
      } else {
        beta_k = a.scal[SC_BETA];
      }
#pragma unroll
      for (int q = 0; q < W / R0; ++q)
#pragma unroll
        for (int r = 0; r < R0; ++r) {
          const int e = in_pos<PL, 0>(t, q, r), kx = e, ky = col_ky;
          long idx = base_off + (long)e * a.row_stride;
          cx<T> pn = {T(0), T(0)};
          if (valid) {
            cx<T> po = ld_stream(pio + idx, a.nt & NT_P), rv = ld_stream(a.cg_r + idx, a.nt & NT_R);
            long mode = base_off + (long)e * a.row_stride;
            const T il = inv_lam_at(a.inv_lam, a.radial, a.g, kx, ky, kz, mode, a.nt & NT_TAB);
            const T mi = precond_inv<T>(il, dbar), bt = (T)beta_k;
            pn = {mi * rv.x + bt * po.x, mi * rv.y + bt * po.y};
            st_stream(pio + idx, pn, a.nt & NT_P);
            acc[0] += hw * (double)(il * (pn.x * pn.x + pn.y * pn.y));
          }
          v[q * R0 + r] = pn;
        }
    }
    fft_thread<PL, true, MAP, SPLIT>(v, t, lds, a.tw, active);
    block_reduce_store<1>(acc, a.partials, block_linear);
  } else {
#pragma unroll
  for (int q = 0; q < W / R0; ++q)
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      int e = in_pos<PL, 0>(t, q, r);
      v[q * R0 + r] = valid ? a.in[base_off + (long)e * a.row_stride] : cx<T>{T(0), T(0)};
    }
  }

  if constexpr (OP == COL_CG_FIRST || OP == COL_CG_INIT) {
    // done above
  } else if constexpr (OP == COL_PLAIN) {
    fft_thread<PL, INV, MAP, SPLIT>(v, t, lds, a.tw, active);
  } else if constexpr (OP == COL_PRIOR) {
    // forward transform, multiply by 1/lambda (after removing the prior mean
    // from mode 0), inverse transform: S_L^-1 applied along the last axis of
    // a field already transformed along y and z.
    fft_thread<PL, false, MAP, SPLIT>(v, t, lds, a.tw, active);
    const int kz = col_kz;
    double acc[1] = {0.0};
#pragma unroll
    for (int q = 0; q < W / RL; ++q)
#pragma unroll
      for (int m = 0; m < RL; ++m) {
        const int e = out_pos<PL, PL::NS - 1>(t, q, m), kx = e, ky = col_ky;
        long mode = base_off + (long)e * a.row_stride;
        cx<T> x = v[q * RL + m];
        if (mode == 0) x.x -= (T)a.k0_shift;
        T il = valid ? inv_lam_at(a.inv_lam, a.radial, a.g, kx, ky, kz, mode, a.nt & NT_TAB) : T(0);
        if (valid) acc[0] += herm_w(kz, a.g) * (double)il * ((double)x.x * x.x + (double)x.y * x.y);
        v[q * RL + m] = {x.x * il, x.y * il};
      }
    last_to_first<PL, MAP, SPLIT>(v, t, lds, active);
    fft_thread<PL, true, MAP, SPLIT>(v, t, lds, a.tw, active);
    block_reduce_store<1>(acc, a.partials, block_linear);
  } else if constexpr (OP == COL_CG_STEP) {
    // forward transform (X = F d v with v = F^-1 u); u = M^-1 r formed again
    // from r; p = u + beta p, y = X + beta y, so that H p = y + p/lambda (the
    // prior part is formed from p itself: carried along in the recurrence its
    // 17 decades cost iterations, 622 instead of 603 at 256^3); r -= alpha H p.
    // x takes two iterations' steps at once, on every second one, when the
    // last two directions are both at hand (p_old is read, p is formed), which
    // saves its read and write on the others.  Then u = M^-1 r of the new
    // residual, its sums and its inverse transform.
    static_assert(!BATCHED, "batches run the two-pass CG");
    const int k = a.cg_k;
    double alpha, beta;
    if (a.z_part) {
      double dv[2], uv[3];
      col_sums<T, N, V, false, 2>(a.z_part, a.z_nb, dv);
      col_sums<T, N, V, false, 3>(a.beta_part, a.beta_nb, uv);
      const double delta = uv[0] * a.beta_scale + dv[0], gamma = uv[1] * a.beta_scale, rr = uv[2] * a.beta_scale;
      double* sc = const_cast<double*>(a.scal);
      const bool over = block_linear == 0 && threadIdx.x == 0
                            ? cg_scalars<true>(sc, delta, gamma, rr, k, a.cg_max, a.tol_rel2, &alpha, &beta)
                            : cg_scalars<false>(sc, delta, gamma, rr, k, a.cg_max, a.tol_rel2, &alpha, &beta);
      if (over) return;  // the whole workgroup (every one decides alike)
    } else {
      alpha = a.scal[cg_alpha_slot(k)];
      beta = a.scal[SC_BETA];
    }
    const double dbar = a.scal[SC_DBAR], hw = herm_w(col_kz, a.g);
    const T al = (T)alpha, bt = (T)beta, al_old = k > 0 ? (T)a.scal[cg_alpha_slot(k - 1)] : T(0);
    fft_thread<PL, false, MAP, SPLIT>(v, t, lds, a.tw, active);
    double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < W / RL; ++q)
#pragma unroll
      for (int m = 0; m < RL; ++m) {
        const int kx = out_pos<PL, PL::NS - 1>(t, q, m);
        const long mode = base_off + (long)kx * a.row_stride;
        cx<T> un = {T(0), T(0)};
        if (valid) {
          const T il = inv_lam_at(a.inv_lam, a.radial, a.g, kx, col_ky, col_kz, mode, a.nt & NT_TAB);
          const cx<T> rv = ld_stream(a.cg_r + mode, a.nt & NT_R);
          const T mi = precond_inv<T>(il, dbar);
          cx<T> pn = {mi * rv.x, mi * rv.y}, po = {T(0), T(0)}, yn = v[q * RL + m];
          if (k > 0) {
            po = ld_stream(a.cg_p + mode, a.nt & NT_P);
            const cx<T> yo = ld_stream(a.cg_y + mode, a.nt & NT_P);
            pn = {pn.x + bt * po.x, pn.y + bt * po.y};
            yn = {yn.x + bt * yo.x, yn.y + bt * yo.y};
          }
          const cx<T> rn = {rv.x - al * (yn.x + il * pn.x), rv.y - al * (yn.y + il * pn.y)};
          st_stream(a.cg_p + mode, pn, a.nt & NT_P);
          st_stream(a.cg_y + mode, yn, a.nt & NT_P);
          st_stream(a.cg_r + mode, rn, a.nt & NT_R);
          if (k & 1) {
            cx<T> xn = {al_old * po.x + al * pn.x, al_old * po.y + al * pn.y};
            if (k > 1) xn = xn + ld_stream(a.cg_x + mode, a.nt & NT_X);
            st_stream(a.cg_x + mode, xn, a.nt & NT_X);
          }
          cg_precondition<T>(rn, il, dbar, hw, un, acc);
        }
        v[q * RL + m] = un;
      }
    last_to_first<PL, MAP, SPLIT>(v, t, lds, active);
    fft_thread<PL, true, MAP, SPLIT>(v, t, lds, a.tw, active);
    block_reduce_store<3>(acc, a.partials, block_linear);
  } else if constexpr (OP == COL_CG_LAST) {
    // forward transform; q = X + p/lambda (= H p); r -= alpha q and
    // x += alpha p in place; partials (r^H r, r^H M^-1 r).  q is not stored.
    // p and 1/lambda at the output positions are loaded before the
    // transform so that their latency overlaps it.  With z_part set every
    // workgroup forms alpha itself and workgroup 0 stores it.
    double alpha = 0.0;
    if (a.z_part) {
      const bool first = !BATCHED && a.cg_k == 0;
      double dv[2], e[3] = {0.0, 0.0, 0.0};
      col_sums<T, N, V, BATCHED, 2>(a.z_part, a.z_nb, dv);
      if (first)
        col_sums<T, N, V, BATCHED, 3>(a.beta_part, a.beta_nb, e);
      else
        col_sums<T, N, V, BATCHED, 1>(a.beta_part, a.beta_nb, e);
      double* sc = const_cast<double*>(a.scal);
      const double pi = e[0] * a.beta_scale, gamma = e[1] * a.beta_scale, rr = e[2] * a.beta_scale;
      const bool over = block_linear == 0 && threadIdx.x == 0
                            ? cg_alpha<true>(sc, first, pi, dv[0], gamma, rr, a.tol_rel2, &alpha)
                            : cg_alpha<false>(sc, first, pi, dv[0], gamma, rr, a.tol_rel2, &alpha);
      if (over) return;  // the whole workgroup (every one decides alike)
    } else {
      alpha = a.scal[SC_ALPHA];
    }
    const int kz = col_kz;
    cx<T> pre_p[PRELOAD ? W : 1];
    T pre_il[PRELOAD ? W : 1];
    if constexpr (PRELOAD) {
#pragma unroll
      for (int q = 0; q < W / RL; ++q)
#pragma unroll
        for (int m = 0; m < RL; ++m) {
          const int e = out_pos<PL, PL::NS - 1>(t, q, m), kx = e, ky = col_ky;
          long mode = base_off + (long)e * a.row_stride;
          pre_p[q * RL + m] = valid ? ld_stream(a.base + mode, a.nt & NT_P) : cx<T>{T(0), T(0)};
          pre_il[q * RL + m] = valid ? inv_lam_at(a.inv_lam, a.radial, a.g, kx, ky, kz, mode, a.nt & NT_TAB) : T(0);
        }
    }
    fft_thread<PL, false, MAP, SPLIT>(v, t, lds, a.tw, active);
    const double hw = herm_w(kz, a.g);
    const double dbar = a.scal[SC_DBAR];
    double acc[2] = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < W / RL; ++q)
#pragma unroll
      for (int m = 0; m < RL; ++m) {
        const int e = out_pos<PL, PL::NS - 1>(t, q, m), kx = e, ky = col_ky;
        long mode = base_off + (long)e * a.row_stride;
        if (valid) {
          // vector arithmetic in the Krylov vectors' precision, sums in FP64
          cx<T> pv;
          T il;
          if constexpr (PRELOAD) {
            pv = pre_p[q * RL + m];
            il = pre_il[q * RL + m];
          } else {
            pv = ld_stream(a.base + mode, a.nt & NT_P);
            il = inv_lam_at(a.inv_lam, a.radial, a.g, kx, ky, kz, mode, a.nt & NT_TAB);
          }
          cx<T> x = v[q * RL + m];
          const T qx = x.x + il * pv.x, qy = x.y + il * pv.y, al = (T)alpha;
          cx<T> rv = ld_stream(a.cg_r + mode, a.nt & NT_R), xv = ld_stream(a.cg_x + mode, a.nt & NT_X);
          cx<T> rn = {rv.x - al * qx, rv.y - al * qy};
          st_stream(a.cg_r + mode, rn, a.nt & NT_R);
          st_stream(a.cg_x + mode, cx<T>{xv.x + al * pv.x, xv.y + al * pv.y}, a.nt & NT_X);
          const T rr = rn.x * rn.x + rn.y * rn.y;
          acc[0] += hw * (double)rr;
          acc[1] += hw * (double)(precond_inv<T>(il, dbar) * rr);
        }
      }
    block_reduce_store<2>(acc, a.partials, block_linear);
    // batched CG: this iteration is complete (no other workgroup of this
    // launch reads the count)
    if constexpr (BATCHED)
      if (block_linear == 0 && threadIdx.x == 0) const_cast<double*>(a.scal)[SC_ITS] += 1.0;
    return;
  } else {
    // forward transform; out = scale * X + (1/lambda) (base - shift at mode 0);
    // base and 1/lambda are loaded before the transform (latency overlap)
    const int kz = col_kz;
    cx<T> pre_b[PRELOAD ? W : 1];
    T pre_il[PRELOAD ? W : 1];
    if constexpr (PRELOAD) {
#pragma unroll
      for (int q = 0; q < W / RL; ++q)
#pragma unroll
        for (int m = 0; m < RL; ++m) {
          const int e = out_pos<PL, PL::NS - 1>(t, q, m), kx = e, ky = col_ky;
          long mode = base_off + (long)e * a.row_stride;
          pre_b[q * RL + m] = valid ? ld_stream(a.base + mode, a.nt & NT_P) : cx<T>{T(0), T(0)};
          pre_il[q * RL + m] = valid ? inv_lam_at(a.inv_lam, a.radial, a.g, kx, ky, kz, mode, a.nt & NT_TAB) : T(0);
        }
    }
    fft_thread<PL, false, MAP, SPLIT>(v, t, lds, a.tw, active);
    double acc[3] = {0.0, 0.0, 0.0};
    const double hw = herm_w(kz, a.g);
#pragma unroll
    for (int q = 0; q < W / RL; ++q)
#pragma unroll
      for (int m = 0; m < RL; ++m) {
        const int e = out_pos<PL, PL::NS - 1>(t, q, m), kx = e, ky = col_ky;
        long mode = base_off + (long)e * a.row_stride;
        if (valid) {
          cx<T> b;
          T il;
          if constexpr (PRELOAD) {
            b = pre_b[q * RL + m];
            il = pre_il[q * RL + m];
          } else {
            b = ld_stream(a.base + mode, a.nt & NT_P);
            il = inv_lam_at(a.inv_lam, a.radial, a.g, kx, ky, kz, mode, a.nt & NT_TAB);
          }
          cx<T> bs = b;
          if (mode == 0) bs.x -= (T)a.k0_shift;
          cx<T> x = v[q * RL + m];
          cx<T> o = {x.x * a.out_scale + il * bs.x, x.y * a.out_scale + il * bs.y};
          v[q * RL + m] = o;
          acc[0] += hw * ((double)b.x * o.x + (double)b.y * o.y);
          acc[1] += hw * ((double)o.x * o.x + (double)o.y * o.y);
          acc[2] += hw * (double)il * ((double)bs.x * bs.x + (double)bs.y * bs.y);
        }
      }
    block_reduce_store<3>(acc, a.partials, block_linear);
  }

  if (valid) {
#pragma unroll
    for (int q = 0; q < W / RL; ++q)
#pragma unroll
      for (int m = 0; m < RL; ++m) {
        int e = out_pos<PL, PL::NS - 1>(t, q, m);
        a.out[base_off + (long)e * a.row_stride] = v[q * RL + m];
      }
  }
}


template <typename T, int N, bool INV, int OP, int V>
__global__ void __launch_bounds__((ColShape<T, N, V>::THREADS)) col_kernel(ColArgs<T> a) {
  __shared__ cx<T> lds_all[ColShape<T, N, V>::LDS];
  if (block_skips(a.skip)) return;  // Krylov iteration after convergence
  int gx = gridDim.x, gy = gridDim.y;
  const int hw = blockIdx.x + gridDim.x * blockIdx.y;
  if constexpr (OP == COL_PLAIN) {
    if (a.fin_on) {
      // the workgroups past the tiles (one more column of the grid, or one
      // more row when there are several slabs) hold the finalize riding on
      // this launch (it only reads partials of earlier launches); its first
      // one runs it.  The tiles keep their hardware ids, so the XCD mapping
      // below holds.
      bool rider, lead;
      if (gy > 1) {
        --gy;
        rider = (int)blockIdx.y == gy;
        lead = blockIdx.x == 0;
      } else {
        --gx;
        rider = hw == gx;
        lead = true;
      }
      if (rider) {
        if (lead) {
          const FinArgs& f = a.fin;
          finalize_body<ColShape<T, N, V>::THREADS>(f.partials, f.nb, f.K, f.kind, f.dst, f.scale, f.scal, f.aux,
                                                    f.partials2, f.nb2, f.scale2);
        }
        return;
      }
    }
  }
  const int total = gx * gy;
  // Workgroups are dispatched round-robin over the 8 XCDs (each with its own
  // L2).  Give every XCD a contiguous range of (tile, slab) work items so
  // that neighbouring column tiles, whose row segments share cache lines
  // when the row pitch is not a multiple of 128 bytes, meet in one L2, and
  // so that the 1/lambda table entries gathered by neighbouring x-pass tiles
  // (similar ky) are reused from that L2.
  int tile = blockIdx.x, slab = blockIdx.y;
  {
    const int xcd = hw & 7, k = hw >> 3;
    const int per = total >> 3, rem = total & 7;
    const int logical = xcd * per + (xcd < rem ? xcd : rem) + k;
    tile = logical % gx;
    slab = logical / gx;
  }
  col_body<T, N, INV, OP, V>(a, tile, slab, lds_all, hw);
}

// ---------------------------------------------------------------------------
// Row pass (z axis): two real rows per complex transform
// ---------------------------------------------------------------------------

enum RowOp {
  ROW_R2C = 0,         // real rows -> half rows
  ROW_C2R = 1,         // half rows -> real rows (times scale)
  ROW_HVP = 2,         // half -> real v, times d, -> half; partials (sum d v^2)
  ROW_GRAD = 3,        // half (s_hat) -> s -> likelihood gradient l -> half;
                       // writes s, e, d; partials sum(e - beta N s), sum(d)
  ROW_C2R_DIAG = 4,    // half -> real: scale * x + d * v
  ROW_C2R_GRADLIK = 5,  // half -> real: scale * x + beta (nbar w e^{beta s} - N);
                        // writes d; partials sum(e - beta N s)
  ROW_LB_IN = 6,        // half -> real q (stored to out_r), times d, -> half
  ROW_LB_OUT = 7,       // half -> real g, d g + lb_d1 lb_q, -> half (double only)
  ROW_GRAD_STEP = 8     // ROW_GRAD after a step: s = s_in + alpha v in real space
                        // (alpha = scal[SC_LS_ALPHA], none if <= 0) instead of
                        // the inverse transform of s_hat (double only)
};

template <typename T>
struct RowArgs {
  int n;  // transform length (z)
  const cx<T>* in_c;
  cx<T>* out_c;
  const T* in_r;
  T* out_r;
  int nunits;  // row pairs
  const cx<T>* tw;
  T scale;
  const double* d;  // Hessian diagonal beta^2 nbar w e^{beta s} (unscaled)
  const float* d32;  // same in FP32 (mixed-precision HVP)
  const T* v;
  const double* w;
  const double* counts;
  double nbar, beta;
  const double* s_in;
  double* s_out;
  double* e_out;
  double* d_out;
  double* partials;
  const double* skip;  // if non-null and *skip != 0 the launch does nothing
  int nt;              // NT_* bits: operands loaded / stored non-temporally
  int model;           // ROW_GRAD likelihood: MODEL_LOGNORMAL or MODEL_GAUSSIAN
  const double* lb_d1;  // ROW_LB_OUT: the curvature diagonal and the kept field q
  const double* lb_q;
  const double* scal;  // ROW_GRAD_STEP: device scalars (the step length)
  // plane passes (plane_body): rows per x plane, x planes, y twiddles
  int ny, nplanes;
  const cx<T>* tw_y;
};

// The likelihood terms of the gradient at one cell (sections 2.1 and 2.4,
// the power-law bias; the Gaussian-prior model of section 2.2.2): writes s,
// e and the Hessian diagonal d, adds to the partial sums (the likelihood
// part of f, sum d) and returns the likelihood gradient l.  GAUSS: whether
// the Gaussian model may be asked for.
template <typename T, bool GAUSS>
__device__ __forceinline__ double grad_cell(const RowArgs<T>& a, long i, double s, double* acc) {
  const double cnt = a.counts[i];
  a.s_out[i] = s;
  if (GAUSS && a.model == MODEL_GAUSSIAN) {
    // Gaussian prior on delta = s, unity bias:
    // -ln L = sum nbar w (1 + delta) - N ln(1 + delta) + const
    const double nw = a.nbar * a.w[i], op = 1.0 + s;
    const double inv = cnt > 0.0 ? 1.0 / op : 0.0;
    const double dd = cnt * inv * inv;
    a.e_out[i] = op;
    a.d_out[i] = dd;
    acc[0] += nw * s - (cnt > 0.0 ? cnt * log1p(s) : 0.0);
    acc[1] += dd;
    return nw - cnt * inv;
  }
  const double ex = a.nbar * a.w[i] * exp(a.beta * s);
  a.e_out[i] = ex;
  const double dd = a.beta * a.beta * ex;
  a.d_out[i] = dd;
  acc[0] += ex - a.beta * cnt * s;
  acc[1] += dd;
  return a.beta * (ex - cnt);
}

template <int N, int V = 0>
struct RowShape {
  static constexpr int P = Plan<N>::P;
  static constexpr int TH = V == 1 ? 512 : 256;
  static constexpr int G = (TH / P) > 32 ? 32 : (TH / P < 1 ? 1 : TH / P);  // row pairs per block
  static constexpr int THREADS = G * P;
  static constexpr int LEN = PaddedLen<N + 2, true>::value;  // LDS slots per pair
};

// which row operations leave partial sums, start from half rows, end in them
constexpr bool row_has_sums(int op) {
  return op == ROW_GRAD || op == ROW_GRAD_STEP || op == ROW_HVP || op == ROW_LB_IN || op == ROW_C2R_GRADLIK;
}
constexpr bool row_from_half(int op) { return op != ROW_R2C && op != ROW_GRAD_STEP; }
constexpr bool row_to_half(int op) { return op != ROW_C2R && op != ROW_C2R_DIAG && op != ROW_C2R_GRADLIK; }

// The Hessian diagonal at real cell i, in the transforms' precision.
template <typename T>
__device__ __forceinline__ T diag_at(const RowArgs<T>& a, long i, int nt) {
  if constexpr (sizeof(T) == 8)
    return ld_stream(a.d + i, nt);
  else
    return ld_stream(a.d32 + i, nt);
}

// How the threads of a row pair transform: exchanges through the padded LDS
// rows of a row pass, the whole workgroup meeting at barriers.
template <typename T, int N>
struct BlockRowFft {
  using PL = Plan<N>;
  using Fwd = PL;
  using MAP = LdsMap<1, true>;
  static constexpr int PRELOAD_D = PL::W;
  static constexpr bool STREAM = true, GAUSS = true;
  int t;
  cx<T>* lds;
  const cx<T>* tw;
  bool active;
  template <bool INV>
  __device__ __forceinline__ void fft(cx<T>* v) const { fft_thread<PL, INV, MAP>(v, t, lds, tw, active); }
  __device__ __forceinline__ void turn(cx<T>* v) const { last_to_first<PL, MAP>(v, t, lds, active); }
  __device__ __forceinline__ void chunk(int) const {}
  __device__ __forceinline__ void pin(double (&)[2]) const {}
};

// One row pair's z transforms and pointwise work: thread t of the Plan<N>::P
// sharing the pair; rowA, rowB: the two real rows; src / dst: their half rows.  acc: the thread's partial sums.
template <typename T, int N, int OP, class FX>
__device__ __forceinline__ void row_core(const RowArgs<T>& a, const FX& fx, const int t, const bool active,
                                         const bool valid, const long rowA, const long rowB, const cx<T>* srcA,
                                         const cx<T>* srcB, cx<T>* dstA, cx<T>* dstB, double (&acc)[2]) {
  using PL = Plan<N>;              // inverse transforms
  using PLF = typename FX::Fwd;    // forward ones
  constexpr int P = PL::P;
  constexpr int W = PL::W;
  constexpr int R0 = row_from_half(OP) ? PL::R0 : PLF::R0;  // of the first transform
  constexpr int RL = LastStage<PL>::R;
  constexpr int H = N / 2 + 1;

  // Pairs that are not valid stand at a valid pair's addresses: their loads
  // are unconditional (a branch around each would end the basic block the
  // loads are scheduled in) and what they load is not used.
  cx<T> v[W];
  // (no runtime choice where FX::STREAM is off: its branch would group the
  // loads of all elements on one side of it)
  const int nt_d = FX::STREAM ? a.nt & NT_DIAG : 0;
  // ---- gather the complex length-N input Z = A + i B (stage-0 slots) ----
  if constexpr (OP == ROW_GRAD_STEP) {
    // real rows of the stepped iterate: the likelihood gradient l at each
    // cell is this transform's input
    const double al = a.scal[SC_LS_ALPHA] > 0.0 ? a.scal[SC_LS_ALPHA] : 0.0;
#pragma unroll
    for (int q = 0; q < W / R0; ++q)
#pragma unroll
      for (int r = 0; r < R0; ++r) {
        const int e = in_pos<PLF, 0>(t, q, r);
        double l[2] = {0.0, 0.0};
        if (valid) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const long i = (h ? rowB : rowA) * N + e;
            l[h] = grad_cell<T, FX::GAUSS>(a, i, a.s_in[i] + al * (double)a.v[i], acc);
          }
        }
        v[q * R0 + r] = {(T)l[0], (T)l[1]};
        fx.chunk(3);
        fx.pin(acc);
      }
  } else if constexpr (OP == ROW_R2C) {
#pragma unroll
    for (int q = 0; q < W / R0; ++q)
#pragma unroll
      for (int r = 0; r < R0; ++r) {
        const int e = in_pos<PLF, 0>(t, q, r);
        const T ra = a.in_r[rowA * N + e], rb = a.in_r[rowB * N + e];
        v[q * R0 + r] = {valid ? ra : T(0), valid ? rb : T(0)};
      }
  } else {
    // the two half rows A and B give
    // Z[e] = A[e] + i B[e], with A[e] = conj A[N - e] above N/2: each lane
    // loads its elements straight from memory (the lanes of a row pair read
    // consecutive, or mirrored consecutive, values)
#pragma unroll
    for (int q = 0; q < W / R0; ++q)
#pragma unroll
      for (int r = 0; r < R0; ++r) {
        const int e = active ? in_pos<PL, 0>(t, q, r) : 0;
        const bool lo = e <= N / 2;
        const int ie = lo ? e : N - e;
        cx<T> A = srcA[ie], Bv = srcB[ie];
        if (!lo) {
          A.y = -A.y;
          Bv.y = -Bv.y;
        } else if (e == 0 || e == N / 2) {
          A.y = T(0);
          Bv.y = T(0);
        }
        v[q * R0 + r] = {valid ? A.x - Bv.y : T(0), valid ? A.y + Bv.x : T(0)};
        fx.chunk(q * R0 + r);
      }
  }

  // ROW_HVP / ROW_LB_IN: the diagonal at the positions this thread
  // multiplies, loaded before the transforms so that its latency overlaps them
  // (FX::PRELOAD_D of them)
  constexpr int PRE_D = OP == ROW_HVP || OP == ROW_LB_IN ? FX::PRELOAD_D : 0;
  T pre_dA[PRE_D ? PRE_D : 1], pre_dB[PRE_D ? PRE_D : 1];
#pragma unroll
  for (int i = 0; i < PRE_D; ++i) {
    const int e = active ? out_pos<PL, PL::NS - 1>(t, i / RL, i % RL) : 0;
    pre_dA[i] = diag_at<T>(a, rowA * N + e, nt_d);
    pre_dB[i] = diag_at<T>(a, rowB * N + e, nt_d);
  }

  if constexpr (OP == ROW_R2C || OP == ROW_GRAD_STEP) {
    fx.template fft<false>(v);
  } else {
    fx.template fft<true>(v);
    // v now holds z[e] = a[e] + i b[e] at last-stage slots (unscaled)
    if constexpr (OP == ROW_C2R) {
      if (valid) {
#pragma unroll
        for (int q = 0; q < W / RL; ++q)
#pragma unroll
          for (int m = 0; m < RL; ++m) {
            int e = out_pos<PL, PL::NS - 1>(t, q, m);
            a.out_r[rowA * N + e] = v[q * RL + m].x * a.scale;
            a.out_r[rowB * N + e] = v[q * RL + m].y * a.scale;
          }
      }
      return;
    } else if constexpr (OP == ROW_C2R_DIAG) {
      if (valid) {
#pragma unroll
        for (int q = 0; q < W / RL; ++q)
#pragma unroll
          for (int m = 0; m < RL; ++m) {
            int e = out_pos<PL, PL::NS - 1>(t, q, m);
            long iA = rowA * N + e, iB = rowB * N + e;
            if constexpr (sizeof(T) == 8) {
              a.out_r[iA] = v[q * RL + m].x * a.scale + (T)a.d[iA] * a.v[iA];
              a.out_r[iB] = v[q * RL + m].y * a.scale + (T)a.d[iB] * a.v[iB];
            } else {
              a.out_r[iA] = v[q * RL + m].x * a.scale + a.d32[iA] * a.v[iA];
              a.out_r[iB] = v[q * RL + m].y * a.scale + a.d32[iB] * a.v[iB];
            }
          }
      }
      return;
    } else if constexpr (OP == ROW_C2R_GRADLIK) {
      if (valid) {
#pragma unroll
        for (int q = 0; q < W / RL; ++q)
#pragma unroll
          for (int m = 0; m < RL; ++m) {
            int e = out_pos<PL, PL::NS - 1>(t, q, m);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              long i = (h ? rowB : rowA) * N + e;
              double prior = (double)(h ? v[q * RL + m].y : v[q * RL + m].x) * (double)a.scale;
              double s = a.s_in[i];
              double ex = a.nbar * a.w[i] * exp(a.beta * s);
              double cnt = a.counts[i];
              a.out_r[i] = (T)(prior + a.beta * (ex - cnt));
              a.d_out[i] = a.beta * a.beta * ex;
              acc[0] += ex - a.beta * cnt * s;
            }
            fx.chunk(3);
            fx.pin(acc);
          }
      }
      return;
    } else {
      // pointwise work on the real values, then back to half spectra
      if constexpr (OP == ROW_HVP) {
#pragma unroll
        for (int q = 0; q < W / RL; ++q)
#pragma unroll
          for (int m = 0; m < RL; ++m) {
            T dA, dB;
            if (q * RL + m < PRE_D) {
              dA = pre_dA[q * RL + m];
              dB = pre_dB[q * RL + m];
            } else {
              const int e = out_pos<PL, PL::NS - 1>(t, q, m);
              dA = diag_at<T>(a, rowA * N + e, nt_d);
              dB = diag_at<T>(a, rowB * N + e, nt_d);
            }
            dA = valid ? dA : T(0);
            dB = valid ? dB : T(0);
            cx<T> z = v[q * RL + m];
            T va = z.x * a.scale, vb = z.y * a.scale;
            acc[0] += (double)dA * va * va + (double)dB * vb * vb;
            v[q * RL + m] = {va * dA, vb * dB};
            fx.chunk(q * RL + m);
          }
      } else if constexpr (OP == ROW_LB_IN) {
        // keep q = F^-1 p (real) for the output pass, go on with d q;
        // partial sums of lb_d1 q^2
#pragma unroll
        for (int q = 0; q < W / RL; ++q)
#pragma unroll
          for (int m = 0; m < RL; ++m) {
            const int e = out_pos<PL, PL::NS - 1>(t, q, m);
            cx<T> z = v[q * RL + m];
            const T va = z.x * a.scale, vb = z.y * a.scale;
            // (loads outside the branch: one per element would wait for its own)
            const T d1A = a.lb_d1[rowA * N + e], d1B = a.lb_d1[rowB * N + e];
            if (valid) {
              a.out_r[rowA * N + e] = va;
              a.out_r[rowB * N + e] = vb;
            }
            const double sum = (double)d1A * va * va + (double)d1B * vb * vb;
            acc[0] += valid ? sum : 0.0;
            T dA, dB;
            if (q * RL + m < PRE_D) {
              dA = pre_dA[q * RL + m];
              dB = pre_dB[q * RL + m];
            } else {
              dA = diag_at<T>(a, rowA * N + e, nt_d);
              dB = diag_at<T>(a, rowB * N + e, nt_d);
            }
            v[q * RL + m] = {va * dA, vb * dB};
          }
      } else if constexpr (OP == ROW_LB_OUT) {
        // d g + d1 q at each real position
#pragma unroll
        for (int q = 0; q < W / RL; ++q)
#pragma unroll
          for (int m = 0; m < RL; ++m) {
            const int e = out_pos<PL, PL::NS - 1>(t, q, m);
            cx<T> z = v[q * RL + m];
            const long iA = rowA * N + e, iB = rowB * N + e;
            const T oA = a.d[iA] * (z.x * a.scale) + a.lb_d1[iA] * a.lb_q[iA];
            const T oB = a.d[iB] * (z.y * a.scale) + a.lb_d1[iB] * a.lb_q[iB];
            v[q * RL + m] = {valid ? oA : T(0), valid ? oB : T(0)};
            fx.chunk(q * RL + m);
          }
      } else {  // ROW_GRAD (double only)
#pragma unroll
        for (int q = 0; q < W / RL; ++q)
#pragma unroll
          for (int m = 0; m < RL; ++m) {
            int e = out_pos<PL, PL::NS - 1>(t, q, m);
            cx<T> z = v[q * RL + m];
            double l[2] = {0.0, 0.0};
            if (valid) {
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                long i = (h ? rowB : rowA) * N + e;
                l[h] = grad_cell<T, FX::GAUSS>(a, i, (double)(h ? z.y : z.x) * (double)a.scale, acc);
              }
            }
            v[q * RL + m] = {(T)l[0], (T)l[1]};
            fx.chunk(3);
            fx.pin(acc);
          }
      }
      // the sums so far, now: they are used last, and left to the end they
      // would keep every operand in registers through the second transform
      asm volatile("" : "+v"(acc[0]), "+v"(acc[1]));
      fx.turn(v);
      fx.template fft<false>(v);
    }
  }

  // ---- split Z' into the two half rows: A'[k] = (Z[k] + conj Z[N-k])/2,
  //      B'[k] = (Z[k] - conj Z[N-k])/(2i) ----
  // The last stage leaves element k = t + P j (j = q + (W/RL) m) in slot
  // (q, m) of lane t.  Its mirror N - k = (P - t) + P (W - 1 - j) sits in
  // lane (P - t) mod P of the same row pair, slot W - 1 - j (lane 0: its
  // own slot (W - j) mod W); it is fetched with a cross-lane shuffle, so the
  // split needs neither LDS nor a barrier.  All lanes take part in the
  // shuffles (uniform control flow); only valid ones store.
  {
    constexpr int RF = LastStage<PLF>::R, QL = W / RF;
    const int lane = (int)(threadIdx.x & 63);
    const int src_lane = (lane & ~(P - 1)) | ((P - t) & (P - 1));
#pragma unroll
    for (int j = 0; j <= W / 2; ++j) {
      const int jo = W - 1 - j;                   // partner slot (t > 0)
      const int jz = (W - j) % W;                 // own slot (t = 0)
      const cx<T> send = v[(jo % QL) * RF + jo / QL];
      cx<T> zc;
      if constexpr (P > 1) {
        zc.x = __shfl(send.x, src_lane, 64);
        zc.y = __shfl(send.y, src_lane, 64);
        if (t == 0) zc = v[(jz % QL) * RF + jz / QL];
      } else {
        zc = v[(jz % QL) * RF + jz / QL];
      }
      const cx<T> zk = v[(j % QL) * RF + j / QL];
      const int k = t + P * j;
      if (valid && k < H) {
        dstA[k] = {T(0.5) * (zk.x + zc.x), T(0.5) * (zk.y - zc.y)};
        dstB[k] = {T(0.5) * (zk.y + zc.y), T(0.5) * (zc.x - zk.x)};
      }
      fx.chunk(j);
    }
  }
}

template <typename T, int N, int OP, int V = 0>
__device__ __forceinline__ void row_body(const RowArgs<T>& a, int ublock, cx<T>* lds_all, int block_linear) {
  constexpr int P = Plan<N>::P;
  constexpr int G = RowShape<N, V>::G;
  constexpr int LEN = RowShape<N, V>::LEN;
  constexpr int H = N / 2 + 1;
  const bool active = (int)threadIdx.x < RowShape<N, V>::THREADS;
  const int t = threadIdx.x % P;
  const int ul = active ? (int)threadIdx.x / P : 0;
  const int u = ublock * G + ul;
  const bool valid = active && u < a.nunits;
  const int uc = valid ? u : 0;
  const long rowA = 2L * uc, rowB = 2L * uc + 1;
  const BlockRowFft<T, N> fx{t, lds_all + ul * LEN, a.tw, active};
  double acc[2] = {0.0, 0.0};
  const cx<T>* src = a.in_c + rowA * H;
  cx<T>* dst = a.out_c + rowA * H;
  row_core<T, N, OP>(a, fx, t, active, valid, rowA, rowB, src, src + H, dst, dst + H, acc);
  if constexpr (row_has_sums(OP)) block_reduce_store<2>(acc, a.partials, block_linear);
}

template <typename T, int N, int OP, int V>
__global__ void __launch_bounds__((RowShape<N, V>::THREADS)) row_kernel(RowArgs<T> a) {
  __shared__ cx<T> lds_all[RowShape<N, V>::G * RowShape<N, V>::LEN];
  if (a.skip && *a.skip != 0.0) return;  // Krylov iteration after convergence
  row_body<T, N, OP, V>(a, blockIdx.x, lds_all, blockIdx.x);
}

// ---------------------------------------------------------------------------
// Elementwise / Krylov kernels on half spectra (grid-stride loops)
// ---------------------------------------------------------------------------



struct ModeIter {
  Grid g;
  // 32-bit unsigned divisions: half spectra hold at most 512 x 512 x 257
  // modes, far below 2^32 (64-bit division is a long software sequence)
  __device__ __forceinline__ void decompose(long i, int& kx, int& ky, int& kz) const {
    const unsigned ui = (unsigned)i, nyh = (unsigned)g.nyh, h = (unsigned)g.h;
    const unsigned x = ui / nyh, r = ui - x * nyh, y = r / h;
    kx = (int)x;
    ky = (int)y;
    kz = (int)(r - y * h);
  }
};


// CG start on H x = rhs: x = 0, r = rhs_sign * rhs, p = 0 (the first
// fused first pass then forms p = M^-1 r); partials (r^H M^-1 r, r^H r)
template <typename T>
__device__ __forceinline__ void cg_init_body(const cx<double>* __restrict__ rhs, double rhs_sign, cx<T>* __restrict__ x,
                                             cx<T>* __restrict__ r, cx<T>* __restrict__ p, const T* __restrict__ tab,
                                             int radial, const Grid& g, long nh, const double* __restrict__ scal,
                                             double* __restrict__ partials, int bx, int nbx) {
  ModeIter mi{g};
  const double dbar = scal[SC_DBAR];
  double acc[2] = {0.0, 0.0};
  for (long i = bx * (long)blockDim.x + threadIdx.x; i < nh; i += (long)nbx * blockDim.x) {
    int kx, ky, kz;
    mi.decompose(i, kx, ky, kz);
    cx<double> b = rhs[i];
    cx<T> rv = {(T)(rhs_sign * b.x), (T)(rhs_sign * b.y)};
    const double minv = (double)precond_inv<T>(inv_lam_at(tab, radial, g, kx, ky, kz, i), dbar);
    x[i] = {T(0), T(0)};
    r[i] = rv;
    p[i] = {T(0), T(0)};
    double hw = herm_w(kz, g);
    acc[0] += hw * minv * ((double)rv.x * rv.x + (double)rv.y * rv.y);
    acc[1] += hw * ((double)rv.x * rv.x + (double)rv.y * rv.y);
  }
  block_reduce_store<2>(acc, partials, bx);
}

template <typename T>
__global__ void __launch_bounds__(RED_THREADS) cg_init_kernel(const cx<double>* __restrict__ rhs, double rhs_sign,
                                                              cx<T>* __restrict__ x, cx<T>* __restrict__ r,
                                                              cx<T>* __restrict__ p, const T* __restrict__ tab,
                                                              int radial, Grid g, long nh,
                                                              const double* __restrict__ scal,
                                                              double* __restrict__ partials) {
  cg_init_body<T>(rhs, rhs_sign, x, r, p, tab, radial, g, nh, scal, partials, blockIdx.x, gridDim.x);
}

enum FinKind { FIN_STORE = 0, FIN_CG_INIT = 1, FIN_CG_BETA = 3, FIN_DBAR = 4, FIN_CG_ALPHA_ADD = 5,
               FIN_CG_STEP = 6, FIN_CG_CHECK = 7, FIN_CG_BETA_DEV = 8, FIN_CG_ALPHA_FIRST = 9,
               FIN_CG_ALPHA_K = 10, FIN_CG_BETA_K = 11 };

// Sum partials[nb][K] in a fixed order; then scalar bookkeeping.
// kind FIN_CG_ALPHA_ADD: p^H H p = scale2 * sum(partials2[nb2]) (prior part from
// the first pass) + scale * sum(partials[nb][K], k = 0) (diagonal part).
// Sum K interleaved per-block partials (src[i * K + k], i < n) over the
// block: every thread keeps 4 K loads in flight per round over a fixed
// partition, then a fixed-order wave and cross-wave reduction, so the result
// is the same on every run.  Returns the sums in out[] (every thread).
template <int NT, int K>
__device__ __forceinline__ void fin_sums(const double* __restrict__ src, int n, double* out) {
  __shared__ double sh[K][NT / 64];
  double acc[K];
#pragma unroll
  for (int k = 0; k < K; ++k) acc[k] = 0.0;
  for (int base = 0; base < n; base += 4 * NT) {
    double x[4][K];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = base + u * NT + (int)threadIdx.x;
#pragma unroll
      for (int k = 0; k < K; ++k) x[u][k] = i < n ? src[(size_t)i * K + k] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] += (x[0][k] + x[1][k]) + (x[2][k] + x[3][k]);
  }
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc[k] += __shfl_down(acc[k], off, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < K; ++k) sh[k][threadIdx.x >> 6] = acc[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double t = 0.0;
    for (int w = 0; w < NT / 64; ++w) t += sh[k][w];
    out[k] = t;
  }
}

// Device-side reduction of per-block partials and the scalar bookkeeping
// of the Krylov / Newton loops (kind: FinKind).  One block of NT threads.
// DEVCOUNT: the batched CG's form, with the iteration count in SC_ITS
// (FIN_CG_BETA_DEV); the single-grid callers compile without it.
template <int NT, bool DEVCOUNT>
__device__ __forceinline__ void finalize_body(const double* __restrict__ partials, int nb, int K, int kind, int dst,
                                              double scale, double* __restrict__ scal, double aux,
                                              const double* __restrict__ partials2, int nb2, double scale2) {
  double v[8];
  switch (K) {
    case 1: fin_sums<NT, 1>(partials, nb, v); break;
    case 2: fin_sums<NT, 2>(partials, nb, v); break;
    case 3: fin_sums<NT, 3>(partials, nb, v); break;
    default: fin_sums<NT, 4>(partials, nb, v); break;
  }
  double extra = 0.0;
  double e3[3] = {0.0, 0.0, 0.0};
  if (partials2) {
    if (kind == FIN_CG_STEP || kind == FIN_CG_ALPHA_FIRST) {
      fin_sums<NT, 3>(partials2, nb2, e3);
    } else {
      fin_sums<NT, 1>(partials2, nb2, e3);
    }
    extra = e3[0] * scale2;
  }
  if (threadIdx.x != 0) return;
  for (int k = 0; k < K; ++k) v[k] *= scale;
  if constexpr (DEVCOUNT) {
    if (kind == FIN_CG_BETA_DEV) {
      // the same bookkeeping as FIN_CG_BETA_K with the iterations completed
      // taken from SC_ITS, which the batched CG's last pass advances
      if (scal[SC_DONE] != 0.0) return;  // iteration skipped
      const int k = (int)scal[SC_ITS];
      scal[SC_RR] = v[0];
      const double rzo = scal[cg_rz_slot(k - 1)];
      scal[cg_rz_slot(k)] = v[1];
      scal[SC_GAMMA] = v[1];
      scal[SC_BETA] = rzo > 0.0 ? v[1] / rzo : 0.0;
      if (v[0] <= scal[SC_TOL2] || (double)k >= aux) scal[SC_DONE] = 1.0;
      return;
    }
  }
  switch (kind) {
    case FIN_STORE:
      for (int k = 0; k < K; ++k) scal[dst + k] = v[k];
      break;
    case FIN_CG_INIT:
      scal[SC_RZ] = v[0];
      scal[SC_GAMMA] = v[0];
      scal[SC_RR] = v[1];
      scal[SC_RR0] = v[1];
      scal[SC_DONE] = (v[1] <= scal[SC_TOL2]) ? 1.0 : 0.0;
      scal[SC_ITS] = 0.0;
      scal[SC_ALPHA] = 0.0;
      scal[SC_BETA] = 0.0;
      break;
    case FIN_CG_ALPHA_ADD: {  // p^H H p also holds scal[dst]
      if (scal[SC_DONE] != 0.0) break;  // iteration skipped
      const double pq = v[0] + extra + scal[dst];
      scal[SC_PQ] = pq;
      double al = 0.0;
      if (scal[SC_DONE] == 0.0 && pq > 0.0) al = scal[SC_RZ] / pq;
      if (scal[SC_DONE] == 0.0 && !(pq > 0.0)) scal[SC_DONE] = 2.0;  // breakdown
      scal[SC_ALPHA] = al;
      break;
    }
    case FIN_CG_STEP: {
      // the scalars of iteration dst + 1, from the z pass's sum of d v^2 and
      // the last x pass's (u^H Lambda^-1 u, r^H u, r^H r); aux: the iteration
      // cap, scal[SC_TOL_REL2] the relative tolerance
      if (scal[SC_DONE] != 0.0) break;  // iteration skipped
      double alpha, beta;
      cg_scalars<true>(scal, e3[0] * scale2 + v[0], e3[1] * scale2, e3[2] * scale2, dst, aux, scal[SC_TOL_REL2], &alpha,
                       &beta);
      break;
    }
    case FIN_CG_ALPHA_FIRST:
    case FIN_CG_ALPHA_K: {
      // the step length of the two-pass CG (cg_alpha), of its first iteration
      // and of the later ones
      if (scal[SC_DONE] != 0.0) break;  // iteration skipped
      double alpha;
      cg_alpha<true>(scal, kind == FIN_CG_ALPHA_FIRST, e3[0] * scale2, v[0], e3[1] * scale2, e3[2] * scale2,
                     scal[SC_TOL_REL2], &alpha);
      break;
    }
    case FIN_CG_BETA_K: {
      // the bookkeeping a COL_CG_FIRST pass with beta_part does, for the
      // host's check after a chunk: dst = iterations completed
      if (scal[SC_DONE] != 0.0) break;  // iteration skipped
      scal[SC_ITS] = (double)dst;
      scal[SC_RR] = v[0];
      if (v[0] <= scal[SC_TOL2] || (double)dst >= aux) scal[SC_DONE] = 1.0;
      break;
    }
    case FIN_CG_BETA: {
      if (scal[SC_DONE] != 0.0) break;  // iteration skipped
      scal[SC_ITS] += 1.0;
      scal[SC_RR] = v[0];
      const double b = scal[SC_RZ] > 0.0 ? v[1] / scal[SC_RZ] : 0.0;
      scal[SC_RZ] = v[1];
      scal[SC_BETA] = b;
      if (v[0] <= scal[SC_TOL2] || scal[SC_ITS] >= aux) scal[SC_DONE] = 1.0;
      break;
    }
    case FIN_CG_CHECK: {
      // the convergence test a COL_CG_STEP pass starts with, for the host's
      // check after a chunk: dst = iterations completed
      if (scal[SC_DONE] != 0.0) break;  // iteration skipped
      scal[SC_ITS] = (double)dst;
      scal[SC_RR] = v[2];
      if (v[2] <= scal[SC_TOL2] || (double)dst >= aux) scal[SC_DONE] = 1.0;
      break;
    }
    case FIN_DBAR:
      scal[SC_DBAR] = v[0];
      break;
  }
}

#ifdef PL_OPS_KERNELS
constexpr int FIN_THREADS = 1024;
__global__ void __launch_bounds__(FIN_THREADS) finalize_kernel(const double* __restrict__ partials, int nb, int K,
                                                               int kind, int dst, double scale,
                                                               double* __restrict__ scal, double aux,
                                                               const double* __restrict__ partials2, int nb2,
                                                               double scale2) {
  finalize_body<FIN_THREADS>(partials, nb, K, kind, dst, scale, scal, aux, partials2, nb2, scale2);
}

// r = b - q on the half spectrum, with per-block partial sums of the
// Hermitian-weighted |r|^2 (N times the squared norm, by Parseval).
__global__ void __launch_bounds__(RED_THREADS) resid_hat_kernel(const cx<double>* __restrict__ b,
                                                                const cx<double>* __restrict__ q,
                                                                cx<double>* __restrict__ r, Grid g, long nh,
                                                                double* __restrict__ partials) {
  ModeIter mi{g};
  double acc[1] = {0.0};
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x) {
    int kx, ky, kz;
    mi.decompose(i, kx, ky, kz);
    const cx<double> bv = b[i], qv = q[i];
    const cx<double> v = {bv.x - qv.x, bv.y - qv.y};
    r[i] = v;
    acc[0] += herm_w(kz, g) * (v.x * v.x + v.y * v.y);
  }
  block_reduce_store<1>(acc, partials, blockIdx.x);
}

// LSQ-Wiener set-up: the constant Hessian diagonal d = nbar w and the
// right-hand side N - nbar w (real space).
__global__ void __launch_bounds__(RED_THREADS) lsq_setup_kernel(const double* __restrict__ w,
                                                                const double* __restrict__ counts, double nbar,
                                                                double* __restrict__ d, double* __restrict__ rhs,
                                                                long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const double nw = nbar * w[i];
    d[i] = nw;
    rhs[i] = counts[i] - nw;
  }
}

// Inverse-weighted overdensity N / (w nbar) - 1 (the paper's IW estimator,
// section 4.1.1); cells without data (w = 0) are set to the mean, 0.
__global__ void __launch_bounds__(RED_THREADS) inverse_weight_kernel(const double* __restrict__ w,
                                                                     const double* __restrict__ counts, double nbar,
                                                                     double* __restrict__ out, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const double wv = w[i];
    out[i] = wv > 0.0 ? counts[i] / (wv * nbar) - 1.0 : 0.0;
  }
}

// Sums for the correlation coefficient and the Euclidean distance between a
// reconstruction and a reference field (section 4.1.2): per block
// (sum ref rec, sum ref^2, sum rec^2, sum (rec - ref)^2).
__global__ void __launch_bounds__(RED_THREADS) compare_fields_kernel(const double* __restrict__ rec,
                                                                     const double* __restrict__ ref, long n,
                                                                     double* __restrict__ partials) {
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const double x = ref[i], y = rec[i], dd = y - x;
    acc[0] += x * y;
    acc[1] += x * x;
    acc[2] += y * y;
    acc[3] += dd * dd;
  }
  block_reduce_store<4>(acc, partials, blockIdx.x);
}

// Nonlinear CG (the Krylov step with a nonlinear-CG search vector): per
// block, sum_k c_k m_k |g_k|^2 and sum_k c_k m_k Re(conj(g_k) g_old_k) with
// m_k = 1 / (1/lambda_k + dbar) (the preconditioner) and c_k the Hermitian
// weights -- N times the real-space dots g^T M^-1 g and g^T M^-1 g_old.
__global__ void __launch_bounds__(RED_THREADS) nlcg_dots_kernel(const cx<double>* __restrict__ g,
                                                                const cx<double>* __restrict__ g_old,
                                                                const double* __restrict__ tab, int radial, Grid gr,
                                                                long nh, const double* __restrict__ scal,
                                                                double* __restrict__ partials) {
  ModeIter mi{gr};
  const double dbar = scal[SC_DBAR];
  double acc[2] = {0.0, 0.0};
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x) {
    int kx, ky, kz;
    mi.decompose(i, kx, ky, kz);
    const double m = precond_inv<double>(inv_lam_at(tab, radial, gr, kx, ky, kz, i), dbar) * herm_w(kz, gr);
    const cx<double> gv = g[i], go = g_old[i];
    acc[0] += m * (gv.x * gv.x + gv.y * gv.y);
    acc[1] += m * (gv.x * go.x + gv.y * go.y);
  }
  block_reduce_store<2>(acc, partials, blockIdx.x);
}

// xi = -M^-1 g + beta xi (beta = 0: steepest descent), g_old = g; per block
// sum_k c_k Re(conj(xi_k) g_k) (N times the slope xi^T g).
__global__ void __launch_bounds__(RED_THREADS) nlcg_update_kernel(const cx<double>* __restrict__ g,
                                                                  cx<double>* __restrict__ g_old,
                                                                  cx<double>* __restrict__ xi, double beta,
                                                                  const double* __restrict__ tab, int radial, Grid gr,
                                                                  long nh, const double* __restrict__ scal,
                                                                  double* __restrict__ partials) {
  ModeIter mi{gr};
  const double dbar = scal[SC_DBAR];
  double acc[1] = {0.0};
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x) {
    int kx, ky, kz;
    mi.decompose(i, kx, ky, kz);
    const double m = precond_inv<double>(inv_lam_at(tab, radial, gr, kx, ky, kz, i), dbar);
    const cx<double> gv = g[i], xv = xi[i];
    const cx<double> xn = {beta == 0.0 ? -m * gv.x : -m * gv.x + beta * xv.x,
                           beta == 0.0 ? -m * gv.y : -m * gv.y + beta * xv.y};
    xi[i] = xn;
    g_old[i] = gv;
    acc[0] += herm_w(kz, gr) * (xn.x * gv.x + xn.y * gv.y);
  }
  block_reduce_store<1>(acc, partials, blockIdx.x);
}

// Lognormal prior from a matter spectrum (section 2.3): the eigenvalues of
// S, lambda_k = coef pk_k (coef = amp N / V), as a real half spectrum.
__global__ void __launch_bounds__(RED_THREADS) spectrum_to_half_kernel(const double* __restrict__ pk, double coef,
                                                                       cx<double>* __restrict__ out, long nh) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x)
    out[i] = {coef * pk[i], 0.0};
}

// S_L(r) = ln(1 + S(r)) in place; flags[0] |= 1 where S(r) <= -1 (no
// logarithm).
__global__ void __launch_bounds__(RED_THREADS) log1p_field_kernel(double* __restrict__ x, long n,
                                                                  int* __restrict__ flags) {
  int bad = 0;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const double v = x[i];
    if (!(v > -1.0)) bad = 1;
    x[i] = log1p(v);
  }
  if (bad) atomicOr(flags, 1);
}

// P_L = lambda^L_k / coef (the real part of F S_L), raised to floor where
// it is not above it; flags[1] counts the raised k != 0 modes.
__global__ void __launch_bounds__(RED_THREADS) half_to_spectrum_kernel(const cx<double>* __restrict__ in,
                                                                       double inv_coef, double floor_val,
                                                                       double* __restrict__ pk_out, long nh,
                                                                       int* __restrict__ flags) {
  int clipped = 0;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x) {
    const double lam = in[i].x;
    const bool low = !(lam > floor_val);
    if (low && i != 0) ++clipped;
    pk_out[i] = (low ? floor_val : lam) * inv_coef;
  }
  if (clipped) atomicAdd(flags + 1, clipped);
}

// flags[0] = 1 where a cell with counts has 1 + delta <= 0 (the Gaussian
// model's likelihood is undefined there); flags[0] must start at 0.
__global__ void __launch_bounds__(RED_THREADS) gauss_domain_kernel(const double* __restrict__ delta,
                                                                   const double* __restrict__ counts, long n,
                                                                   int* __restrict__ flags) {
  int bad = 0;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    if (counts[i] > 0.0 && !(1.0 + delta[i] > 0.0)) bad = 1;
  if (bad) atomicOr(flags, 1);
}

__global__ void set_scalar_kernel(double* scal, int idx, double value) {
  if (threadIdx.x == 0 && blockIdx.x == 0) scal[idx] = value;
}

// Start of a CG solve: stopping threshold (absolute, or relative to the first
// residual), iteration count and state.
__global__ void cg_start_kernel(double* scal, double tol2, double tol_rel2) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    scal[SC_TOL2] = tol2;
    scal[SC_TOL_REL2] = tol_rel2;
    scal[SC_DONE] = 0.0;
    scal[SC_ITS] = 0.0;
    scal[SC_BETA] = 0.0;
    scal[SC_ALPHA] = 0.0;
  }
}

#endif  // PL_OPS_KERNELS

// s_hat += alpha x  (alpha from the host)
template <typename T>
__global__ void __launch_bounds__(RED_THREADS) axpy_hat_kernel(cx<double>* __restrict__ y, const cx<T>* __restrict__ x,
                                                               double alpha, long nh) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x) {
    cx<T> xv = x[i];
    cx<double> yv = y[i];
    y[i] = {yv.x + alpha * (double)xv.x, yv.y + alpha * (double)xv.y};
  }
}

// s_hat += alpha x with alpha read from the device (a step the line search
// accepted on the device); nothing when alpha <= 0 (no step accepted)
template <typename T>
__global__ void __launch_bounds__(RED_THREADS) axpy_hat_dev_kernel(cx<double>* __restrict__ y,
                                                                   const cx<T>* __restrict__ x,
                                                                   const double* __restrict__ alpha_p, long nh) {
  const double alpha = *alpha_p;
  if (!(alpha > 0.0)) return;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x) {
    cx<T> xv = x[i];
    cx<double> yv = y[i];
    y[i] = {yv.x + alpha * (double)xv.x, yv.y + alpha * (double)xv.y};
  }
}

#ifdef PL_OPS_KERNELS
// The part of the CG's x that COL_CG_STEP has not added yet: after an odd
// number of iterations the last direction's step, after none x = 0.
__global__ void __launch_bounds__(RED_THREADS) cg_flush_kernel(cx<double>* __restrict__ x,
                                                               const cx<double>* __restrict__ p,
                                                               const double* __restrict__ scal, long nh) {
  const int its = (int)scal[SC_ITS];
  if (its > 0 && !(its & 1)) return;
  const double al = its > 0 ? scal[cg_alpha_slot(its - 1)] : 0.0;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x) {
    cx<double> xn = {0.0, 0.0};
    if (its > 0) {
      const cx<double> pv = p[i];
      xn = {al * pv.x, al * pv.y};
      if (its > 1) xn = xn + x[i];
    }
    x[i] = xn;
  }
}

// Armijo test of the first batch of trial steps a0, a0/2, a0/4, a0/8 on the
// device: decrease a b + a^2 c / 2 + sum_i [...] (slots SC_LS_B, SC_LS_C,
// SC_DF + j) against c1 a slope; the first accepted step goes to
// SC_LS_ALPHA, -1 if none (or if the direction does not descend).  Written
// with rounded (unfused) operations, the arithmetic the host test uses.
__device__ __forceinline__ void ls_select_scal(double* scal, double a0, double c1) {
  const double b = scal[SC_LS_B], c = scal[SC_LS_C], slope = scal[SC_LS_SLOPE];
  double alpha = -1.0;
  if (slope < 0.0) {
    double a = a0;
    for (int j = 0; j < 4; ++j, a *= 0.5) {
      const double df = __dadd_rn(__dadd_rn(__dmul_rn(a, b), __dmul_rn(__dmul_rn(__dmul_rn(0.5, a), a), c)),
                                  scal[SC_DF + j]);
      if (df <= __dmul_rn(__dmul_rn(c1, a), slope)) {
        alpha = a;
        break;
      }
    }
  }
  scal[SC_LS_ALPHA] = alpha;
}

__global__ void ls_select_kernel(double* scal, double a0, double c1) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  ls_select_scal(scal, a0, c1);
}
#endif

// Line-search dots on half spectra: b = <p, S^-1 (s - mu)>, c = <p, S^-1 p>,
// slope = <g, p> (times N; the finalize applies 1/N).
template <typename T>
__device__ __forceinline__ void ls_dots_body(const cx<T>* __restrict__ p, const cx<double>* __restrict__ s_hat,
                                             const cx<double>* __restrict__ g_hat, const double* __restrict__ tab,
                                             int radial, const Grid& g, long nh, double k0_shift,
                                             double* __restrict__ partials, int bx, int nbx) {
  ModeIter mi{g};
  double acc[3] = {0.0, 0.0, 0.0};
  for (long i = bx * (long)blockDim.x + threadIdx.x; i < nh; i += (long)nbx * blockDim.x) {
    int kx, ky, kz;
    mi.decompose(i, kx, ky, kz);
    double il = inv_lam_at(tab, radial, g, kx, ky, kz, i);
    cx<T> pv = p[i];
    cx<double> sv = s_hat[i], gv = g_hat[i];
    if (i == 0) sv.x -= k0_shift;
    double hw = herm_w(kz, g);
    acc[0] += hw * il * ((double)pv.x * sv.x + (double)pv.y * sv.y);
    acc[1] += hw * il * ((double)pv.x * pv.x + (double)pv.y * pv.y);
    acc[2] += hw * ((double)pv.x * gv.x + (double)pv.y * gv.y);
  }
  block_reduce_store<3>(acc, partials, bx);
}

template <typename T>
__global__ void __launch_bounds__(RED_THREADS) ls_dots_kernel(const cx<T>* __restrict__ p, const cx<double>* __restrict__ s_hat,
                                                              const cx<double>* __restrict__ g_hat,
                                                              const double* __restrict__ tab, int radial, Grid g,
                                                              long nh, double k0_shift,
                                                              double* __restrict__ partials) {
  ls_dots_body<T>(p, s_hat, g_hat, tab, radial, g, nh, k0_shift, partials, blockIdx.x, gridDim.x);
}

// Likelihood part of f(s + a p) - f(s) for four trial steps a_j:
// sum_i [e_i expm1(a_j beta p_i) - a_j beta N_i p_i]
template <typename T>
__device__ __forceinline__ void ls_eval_body(const T* __restrict__ p, const double* __restrict__ e,
                                             const double* __restrict__ counts, double beta, double a0, long n,
                                             double* __restrict__ partials, int bx, int nbx) {
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (long i = bx * (long)blockDim.x + threadIdx.x; i < n; i += (long)nbx * blockDim.x) {
    double bp = beta * (double)p[i];
    double ei = e[i], ci = counts[i];
    double a = a0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[j] += ei * expm1(a * bp) - a * ci * bp;
      a *= 0.5;
    }
  }
  block_reduce_store<4>(acc, partials, bx);
}

template <typename T>
__global__ void __launch_bounds__(RED_THREADS) ls_eval_kernel(const T* __restrict__ p, const double* __restrict__ e,
                                                              const double* __restrict__ counts, double beta,
                                                              double a0, long n, double* __restrict__ partials) {
  ls_eval_body<T>(p, e, counts, beta, a0, n, partials, blockIdx.x, gridDim.x);
}

// Line search of the Gaussian-prior model: for a = a0, a0/2, a0/4, a0/8 the
// likelihood part of f(delta + a p) - f(delta),
//   sum_i [nbar w_i a p_i - N_i log1p(a p_i / (1 + delta_i))]  (op = 1 + delta),
// which is +inf or NaN (rejected) where a step leaves 1 + delta > 0 in a
// cell with counts.
template <typename T>
__global__ void __launch_bounds__(RED_THREADS) ls_eval_gauss_kernel(const T* __restrict__ p,
                                                                    const double* __restrict__ op,
                                                                    const double* __restrict__ w,
                                                                    const double* __restrict__ counts, double nbar,
                                                                    double a0, long n, double* __restrict__ partials) {
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const double pi = (double)p[i], nw = nbar * w[i], ci = counts[i];
    const double ratio = ci > 0.0 ? pi / op[i] : 0.0;
    double a = a0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[j] += nw * a * pi - (ci > 0.0 ? ci * log1p(a * ratio) : 0.0);
      a *= 0.5;
    }
  }
  block_reduce_store<4>(acc, partials, blockIdx.x);
}

#ifdef PL_OPS_KERNELS
// Non-template kernels are defined in one translation unit only.
// Preconditioner constant.  M_k = 1/lambda_k + c is the Fourier-diagonal
// preconditioner of H = S_L^-1 + diag(d); it is exact when d is uniform.
// When d spans many decades (masked holes, selection falling to zero,
// peaks of 1 + delta ~ 1e4), the slow CG modes are the many large-scale
// modes living where d is small, while the few peaks only add isolated
// large eigenvalues; c is therefore taken at the low end of the bulk of d:
// its 25th percentile over all cells, floored at 1e-3 mean(d).  The
// percentile is read from a histogram of log2(d / mean(d)).
constexpr int DQ_BINS = 2048;
constexpr float DQ_LO = -24.0f, DQ_HI = 24.0f;

// One sub-histogram per wave (fewer same-address LDS atomics), four loads in
// flight per thread before their bins are counted, d scaled by 1/mean.
__device__ __forceinline__ int dquant_bin(double dv, double inv_mean) {
  const double r = dv * inv_mean;
  if (!(r > 0.0)) return 0;
  const float x = (log2f((float)r) - DQ_LO) * ((float)DQ_BINS / (DQ_HI - DQ_LO));
  return x < 0.0f ? 0 : (x >= (float)(DQ_BINS - 1) ? DQ_BINS - 1 : (int)x);
}

__device__ __forceinline__ void dquant_hist_body(const double* __restrict__ d, long n, const double* __restrict__ scal,
                                                 int* __restrict__ hist, int bx, int nbx) {
  constexpr int NW = RED_THREADS / 64;
  __shared__ int h[NW * DQ_BINS];
  for (int i = threadIdx.x; i < NW * DQ_BINS; i += blockDim.x) h[i] = 0;
  __syncthreads();
  int* hw = h + (threadIdx.x >> 6) * DQ_BINS;
  const double mean = scal[SC_DSUM] / (double)n;
  const double inv_mean = mean > 0.0 ? 1.0 / mean : 0.0;
  const long stride = (long)nbx * blockDim.x;
  long i = bx * (long)blockDim.x + threadIdx.x;
  for (; i + 3 * stride < n; i += 4 * stride) {
    const double v0 = d[i], v1 = d[i + stride], v2 = d[i + 2 * stride], v3 = d[i + 3 * stride];
    atomicAdd(&hw[dquant_bin(v0, inv_mean)], 1);
    atomicAdd(&hw[dquant_bin(v1, inv_mean)], 1);
    atomicAdd(&hw[dquant_bin(v2, inv_mean)], 1);
    atomicAdd(&hw[dquant_bin(v3, inv_mean)], 1);
  }
  for (; i < n; i += stride) atomicAdd(&hw[dquant_bin(d[i], inv_mean)], 1);
  __syncthreads();
  for (int b = threadIdx.x; b < DQ_BINS; b += blockDim.x) {
    int c = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) c += h[w * DQ_BINS + b];
    if (c) atomicAdd(&hist[b], c);
  }
}

// Block of DQ_SELECT_THREADS: each thread owns DQ_BINS / DQ_SELECT_THREADS
// consecutive bins; a block prefix sum finds the first bin whose cumulative
// count exceeds n/4, and the histogram is cleared for its next use.
constexpr int DQ_SELECT_THREADS = 256;
__device__ __forceinline__ void dquant_select_body(int* __restrict__ hist, long n, double* __restrict__ scal) {
  constexpr int PER = DQ_BINS / DQ_SELECT_THREADS;
  static_assert(DQ_BINS % DQ_SELECT_THREADS == 0 && DQ_SELECT_THREADS % 64 == 0, "select block shape");
  __shared__ long wave_tot[DQ_SELECT_THREADS / 64];
  __shared__ int found;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  int v[PER];
  long own = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    v[j] = hist[t * PER + j];
    own += v[j];
  }
  long incl = own;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const long y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wave_tot[wv] = incl;
  if (t == 0) found = DQ_BINS;
  __syncthreads();
  long acc = incl - own;
  for (int w = 0; w < wv; ++w) acc += wave_tot[w];
  const long target = (long)(0.25 * (double)n);
  if (acc <= target && acc + own > target) {  // exactly one thread: cumulative counts are monotone
    int b = t * PER;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      acc += v[j];
      if (acc > target) {
        b = t * PER + j;
        break;
      }
    }
    found = b;
  }
#pragma unroll
  for (int j = 0; j < PER; ++j) hist[t * PER + j] = 0;  // ready for the next use
  __syncthreads();
  if (t == 0) {
    const int b = found;
    const double mean = scal[SC_DSUM] / (double)n;
    double c = 0.0;
    if (b > 0 && b < DQ_BINS) c = mean * exp2((double)DQ_LO + ((double)b + 0.5) * (double)(DQ_HI - DQ_LO) / DQ_BINS);
    if (c < 1e-3 * mean) c = 1e-3 * mean;
    scal[SC_DBAR] = c;
  }
}

// d = beta^2 nbar w e^{beta s}, e = nbar w e^{beta s} (real-space input s)
__global__ void __launch_bounds__(RED_THREADS) linearize_kernel(const double* __restrict__ s, const double* __restrict__ w,
                                                                double nbar, double beta, double* __restrict__ e,
                                                                double* __restrict__ d, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    double ex = nbar * w[i] * exp(beta * s[i]);
    if (e) e[i] = ex;
    d[i] = beta * beta * ex;
  }
}

__global__ void __launch_bounds__(RED_THREADS) d_to_f32_kernel(const double* __restrict__ d, float* __restrict__ d32,
                                                               long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    d32[i] = (float)d[i];
}

__global__ void __launch_bounds__(RED_THREADS) dquant_hist_kernel(const double* __restrict__ d, long n,
                                                                  const double* __restrict__ scal,
                                                                  int* __restrict__ hist) {
  dquant_hist_body(d, n, scal, hist, blockIdx.x, gridDim.x);
}

__global__ void __launch_bounds__(DQ_SELECT_THREADS) dquant_select_kernel(int* __restrict__ hist, long n, double* __restrict__ scal) {
  dquant_select_body(hist, n, scal);
}

// Sum of d
__global__ void __launch_bounds__(RED_THREADS) sum_kernel(const double* __restrict__ x, long n,
                                                          double* __restrict__ partials) {
  double acc[1] = {0.0};
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) acc[0] += x[i];
  block_reduce_store<1>(acc, partials, blockIdx.x);
}

// Adjoint per-cell parameter derivatives (mu held fixed):
// dL/dN_i = beta lambda_i, dL/dw_i = -lambda_i beta nbar e^{beta s_i};
// partial sums of lambda (nbar w e^{bs}(1 + beta s) - N) and lambda beta w e^{bs}
__global__ void __launch_bounds__(RED_THREADS) adjoint_cells_kernel(const double* __restrict__ lam, const double* __restrict__ s,
                                                                    const double* __restrict__ w,
                                                                    const double* __restrict__ counts, double nbar,
                                                                    double beta, double* __restrict__ dN,
                                                                    double* __restrict__ dw, long n,
                                                                    double* __restrict__ partials) {
  double acc[3] = {0.0, 0.0, 0.0};
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    double l = lam[i], sv = s[i];
    double ebs = exp(beta * sv);
    double ex = nbar * w[i] * ebs;
    acc[0] += l * (ex * (1.0 + beta * sv) - counts[i]);
    acc[1] += l * beta * w[i] * ebs;
    acc[2] += l;
    if (dN) dN[i] = beta * l;
    if (dw) dw[i] = -l * beta * nbar * ebs;
  }
  block_reduce_store<3>(acc, partials, blockIdx.x);
}

// <lambda, S'^-1 (s - mu)> over k != 0 modes (times N)
__global__ void __launch_bounds__(RED_THREADS) adjoint_prior_dot_kernel(const cx<double>* __restrict__ lam_hat,
                                                                        const cx<double>* __restrict__ s_hat,
                                                                        const double* __restrict__ tab, int radial,
                                                                        Grid g, long nh, double* __restrict__ partials) {
  ModeIter mi{g};
  double acc[1] = {0.0};
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x) {
    if (i == 0) continue;
    int kx, ky, kz;
    mi.decompose(i, kx, ky, kz);
    double il = inv_lam_at(tab, radial, g, kx, ky, kz, i);
    cx<double> l = lam_hat[i], sv = s_hat[i];
    acc[0] += herm_w(kz, g) * il * (l.x * sv.x + l.y * sv.y);
  }
  block_reduce_store<1>(acc, partials, blockIdx.x);
}

// Build 1/lambda per mode from pk: V / (N amp pk); mode 0 -> inv_p0.  Also
// scatters into the radial table and flags entries that disagree.
__global__ void __launch_bounds__(RED_THREADS) inv_lam_mode_kernel(const double* __restrict__ pk, double coef,
                                                                   double inv_p0, Grid g, long nh,
                                                                   double* __restrict__ per_mode,
                                                                   int* __restrict__ bad) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x) {
    double v;
    if (i == 0) {
      v = inv_p0;
    } else {
      double p = pk[i];
      if (!(p > 0.0) || !isfinite(p)) {
        atomicOr(bad, 1);
        v = 0.0;
      } else {
        v = coef / p;
      }
    }
    per_mode[i] = v;
  }
}

__global__ void __launch_bounds__(RED_THREADS) radial_scatter_kernel(const double* __restrict__ per_mode, Grid g, long nh,
                                                                     double* __restrict__ radial) {
  ModeIter mi{g};
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x) {
    int kx, ky, kz;
    mi.decompose(i, kx, ky, kz);
    int fx = fold(kx, g.nx), fy = fold(ky, g.ny);
    radial[fx * fx + fy * fy + kz * kz] = per_mode[i];
  }
}

// The radial table stands in for the per-mode one when every mode agrees
// with its shell's entry to 8 ulp (spectra given per mode are usually
// radial up to the rounding of |k| computed from permuted components).
__global__ void __launch_bounds__(RED_THREADS) radial_check_kernel(const double* __restrict__ per_mode, Grid g, long nh,
                                                                   const double* __restrict__ radial,
                                                                   int* __restrict__ mismatch) {
  ModeIter mi{g};
  int bad = 0;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nh; i += (long)gridDim.x * blockDim.x) {
    int kx, ky, kz;
    mi.decompose(i, kx, ky, kz);
    int fx = fold(kx, g.nx), fy = fold(ky, g.ny);
    const double r = radial[fx * fx + fy * fy + kz * kz], v = per_mode[i];
    if (!(fabs(r - v) <= 8.0 * 2.220446049250313e-16 * fabs(v))) bad = 1;
  }
  if (bad) atomicOr(mismatch, 1);
}

// Timing operands for the autotuner: x[i] in [lo, lo + span) from an
// integer hash of (i, seed), so timed passes stream realistic, non-zero data.
template <typename T>
__global__ void __launch_bounds__(RED_THREADS) fill_hash_kernel(T* __restrict__ x, long n, unsigned seed, double lo,
                                                                double span) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    unsigned long long h = (unsigned long long)i * 0x9E3779B97F4A7C15ull + seed;
    h ^= h >> 31;
    h *= 0xBF58476D1CE4E5B9ull;
    h ^= h >> 29;
    x[i] = (T)(lo + span * (double)(h >> 11) * (1.0 / 9007199254740992.0));
  }
}

__global__ void __launch_bounds__(RED_THREADS) to_f32_kernel(const double* __restrict__ x, float* __restrict__ y, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) y[i] = (float)x[i];
}

// Input validation: counts >= 0, w >= 0, counts > 0 => w > 0, all finite.
// Counts need not be integral: the s-dependent part of the log-likelihood is
// linear in N, which keeps derivatives with respect to N well defined.
// flags bit 1: bad counts, bit 2: bad w, bit 4: counts where w = 0
__global__ void __launch_bounds__(RED_THREADS) validate_kernel(const double* __restrict__ w, const double* __restrict__ counts,
                                                               long n, int* __restrict__ flags) {
  int f = 0;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    double c = counts[i], wv = w[i];
    if (!(c >= 0.0) || !isfinite(c)) f |= 1;
    if (!(wv >= 0.0) || !isfinite(wv)) f |= 2;
    if (c > 0.0 && !(wv > 0.0)) f |= 4;
  }
  if (f) atomicOr(flags, f);
}

// all finite check on a real field; flags |= 8 if not
__global__ void __launch_bounds__(RED_THREADS) finite_kernel(const double* __restrict__ x, long n, int* __restrict__ flags) {
  int f = 0;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    if (!isfinite(x[i])) f = 8;
  if (f) atomicOr(flags, f);
}

#endif  // PL_OPS_KERNELS

}  // namespace pl
