// CPU runs of the x passes that decide the end of a CG solve themselves
// (COL_CG_STEP, COL_CG_LAST, COL_CG_FIRST): every workgroup forms the
// iteration's scalars and workgroup 0 stores the done flag that the launch's
// workgroups test at entry.  A workgroup whose waves meet that store at
// different times has to decide as one: here the flag is set after the first of
// its waves has read it, in both orders of waves, and the vectors must stay as
// they were.  The iteration before it leaves its sums in workgroup memory, as
// on the GPU.  And the start pass (COL_CG_INIT) forms its sums in 64 bits from
// right-hand sides of any scale that FP32 vectors hold.  Prints one line per
// case; exit status 1 on a failure.
#include "pl_kernels.hpp"

#include <algorithm>
#include <random>

using namespace pl;

constexpr int NX = 32, NY = 8, NZ = 8, H = NZ / 2 + 1, COLS = NY * H, NH = NX * COLS, NREC = 256;

template <typename T>
struct Pass {
  using C = cx<T>;
  std::vector<C> t, r, p, y, x, tw;
  std::vector<cx<double>> rhs;
  std::vector<T> tab;
  std::vector<double> scal, part_in, part_z, part_out;
  ColArgs<T> a{};

  Pass() : t(NH), r(NH), p(NH), y(NH), x(NH), tw(NX), rhs(NH), tab(NH), scal(SC_COUNT, 0.0), part_in(3 * NREC),
           part_z(2 * NREC), part_out(3 * 64) {
    std::mt19937 gen(7);
    std::normal_distribution<double> nd;
    auto fill = [&](auto& v) {
      for (auto& z : v) {
        z.x = nd(gen);
        z.y = nd(gen);
      }
    };
    fill(t), fill(r), fill(p), fill(y), fill(x), fill(rhs);
    for (auto& q : tab) q = (T)(1.0 + std::fabs(nd(gen)));
    for (int e = 0; e < NX; ++e) tw[e] = {(T)std::cos(2 * M_PI * e / NX), (T)-std::sin(2 * M_PI * e / NX)};
    a.n = NX;
    a.in = t.data();
    a.out = t.data();
    a.tw = tw.data();
    a.g = {NX, NY, NZ, H, (long)COLS};
    a.inv_lam = tab.data();
    a.radial = TAB_MODE;
    a.partials = part_out.data();
    a.out_scale = T(1);
    a.ncols = COLS;
    a.row_stride = COLS;
    a.slab_stride = 0;
    a.cg_r = r.data();
    a.cg_x = x.data();
    a.cg_p = p.data();
    a.cg_y = y.data();
    a.cg_rhs = rhs.data();
    a.cg_rhs_sign = 1.0;
    a.base = p.data();
    a.scal = scal.data();
    a.skip = scal.data() + SC_DONE;
    a.cg_max = 1000.0;
    a.beta_scale = 1.0;
  }
  std::vector<C> vectors() const {
    std::vector<C> all;
    for (const auto* v : {&r, &p, &y, &x}) all.insert(all.end(), v->begin(), v->end());
    return all;
  }
};

// the sums of an iteration: delta or pi, gamma and rr spread over all records
template <typename T>
void sums(Pass<T>& s, int k_in, double first, double gamma, double rr, double dv) {
  for (int i = 0; i < NREC; ++i) {
    if (k_in == 3) {
      s.part_in[3 * i] = first / NREC;
      s.part_in[3 * i + 1] = gamma / NREC;
      s.part_in[3 * i + 2] = rr / NREC;
    } else if (k_in == 2) {  // (r^H r, r^H M^-1 r)
      s.part_in[2 * i] = rr / NREC;
      s.part_in[2 * i + 1] = gamma / NREC;
    } else {
      s.part_in[i] = first / NREC;
    }
    s.part_z[2 * i] = dv / NREC;
    s.part_z[2 * i + 1] = 0.0;
  }
}

template <typename T, bool INV, int OP>
void launch(Pass<T>& s, const std::vector<int>& order, int flip_before) {
  constexpr int THREADS = ColShape<T, NX, 0>::THREADS;
  static_assert(THREADS == 256 && ColShape<T, NX, 0>::B >= COLS, "one workgroup of four waves");
  gridDim = {1, 1, 1};
  blockIdx = {0, 0, 0};
  hostgpu::run_block(
      THREADS, order, [&] { col_kernel<T, NX, INV, OP, 0>(s.a); },
      [&](int i) {
        if (i == flip_before) s.scal[SC_DONE] = 1.0;
      });
}

static bool g_ok = true;

template <typename T, bool INV, int OP>
void check(const char* name, const std::vector<int>& order) {
  Pass<T> s;
  const int k_in = OP == COL_CG_STEP ? 3 : (OP == COL_CG_LAST ? 1 : 2);
  s.scal[SC_TOL2] = 1.0;
  s.scal[SC_DBAR] = 0.5;
  s.scal[SC_RZ] = s.scal[SC_RZ_ODD] = s.scal[SC_GAMMA] = 3.0;
  s.scal[SC_ALPHA] = s.scal[SC_ALPHA_ODD] = 2.0;
  if (OP != COL_CG_FIRST) {
    s.a.z_part = s.part_z.data();
    s.a.z_nb = NREC;
  }
  s.a.beta_part = s.part_in.data();
  s.a.beta_nb = NREC;
  if (OP == COL_CG_FIRST) s.a.in = s.p.data();
  // an iteration far from the end
  s.a.cg_k = 2;
  sums(s, k_in, 4.0, 3.0, 50.0, 2.0);
  const auto before = s.vectors();
  launch<T, INV, OP>(s, {0, 1, 2, 3}, -1);
  const auto after = s.vectors();
  const bool moved = std::memcmp(before.data(), after.data(), sizeof(after[0]) * after.size()) != 0;
  // the next one finds the solve over: converged, or (the last pass) broken down
  s.a.cg_k = 3;
  sums(s, k_in, OP == COL_CG_LAST ? -8.0 : 4.0, 3.0, 0.5, 2.0);
  launch<T, INV, OP>(s, order, 1);
  const auto end = s.vectors();
  const bool kept = std::memcmp(end.data(), after.data(), sizeof(after[0]) * after.size()) == 0;
  const bool ok = moved && kept && s.scal[SC_DONE] != 0.0;
  g_ok = g_ok && ok;
  std::printf("end %s waves %d%d%d%d: vectors %s ok=%d\n", name, order[0], order[1], order[2], order[3],
              kept ? "kept" : "changed", (int)ok);
}

// r^H M^-1 r and r^H r of the start pass against sums of the same FP32 vectors
// in 64 bits; M^-1 carries FP32's rounding (a few 2^-24)
void check_start(double scale) {
  Pass<float> s;
  s.scal[SC_DBAR] = 0.5;
  s.a.in = nullptr;
  s.a.cg_rhs_sign = scale;
  s.a.skip = nullptr;
  launch<float, true, COL_CG_INIT>(s, {0, 1, 2, 3}, -1);
  double rz = 0.0, rr = 0.0;
  for (int i = 0; i < NH; ++i) {
    const double hw = (i % H == 0 || i % H == H - 1) ? 1.0 : 2.0, x = s.r[i].x, y = s.r[i].y;
    rr += hw * (x * x + y * y);
    rz += hw * (x * x + y * y) / ((double)s.tab[i] + 0.5);
  }
  const double e1 = std::fabs(s.part_out[1] / rz - 1.0), e2 = std::fabs(s.part_out[2] / rr - 1.0);
  const bool ok = rr > 0.0 && std::isfinite(rr) && e1 < 4e-7 && e2 < 1e-13;
  g_ok = g_ok && ok;
  std::printf("start scale %g: r^H r %g (error %.1e, r^H M^-1 r %.1e) ok=%d\n", scale, s.part_out[2], e2, e1, (int)ok);
}

int main() {
  for (double scale : {1.0, 1e-24, 1e-30, 1e20, 1e30}) check_start(scale);
  for (const std::vector<int>& order : {std::vector<int>{0, 1, 2, 3}, std::vector<int>{3, 2, 1, 0}}) {
    check<double, false, COL_CG_STEP>("one-pass x pass FP64", order);
    check<float, false, COL_CG_LAST>("last x pass FP32", order);
    check<double, false, COL_CG_LAST>("last x pass FP64", order);
    check<float, true, COL_CG_FIRST>("first x pass FP32", order);
  }
  return g_ok ? 0 : 1;
}
