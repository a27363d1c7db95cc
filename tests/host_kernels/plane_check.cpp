// CPU runs of the plane passes (y inverse, z with the Hessian diagonal, y forward of
// one x plane in one workgroup's memory) against the transforms written out as
// sums, at every transform length on either axis: the reversed plans, the
// exchange addresses and paddings, ragged last waves, several planes per block.
// Memory past the plane's own is poisoned, so that a sanitizer build stops at an
// access out of it.  (Lengths of one lane per transform, 8 to 16, take planes
// whose row pairs fill their waves: their left-over lanes repeat a transform in
// step with its owner, which lanes run one after the other do not.)  Prints one
// line per case; exit status 1 on a failure.
#include "pl_plane.hpp"

#include <algorithm>
#include <complex>
#include <random>

#if defined(__SANITIZE_ADDRESS__) || (defined(__has_feature) && __has_feature(address_sanitizer))
#include <sanitizer/asan_interface.h>
#define POISON(p, n) __asan_poison_memory_region(p, n)
#define UNPOISON(p, n) __asan_unpoison_memory_region(p, n)
#else
#define POISON(p, n) ((void)0)
#define UNPOISON(p, n) ((void)0)
#endif

namespace pl {
thread_local __attribute__((aligned(16))) char plane_lds[163840];
}
using namespace pl;
using C = std::complex<double>;

static bool g_ok = true;

template <int N>
constexpr int lanes_of() {
  return Plan<N>::P;
}
static int lanes(int n) {
  switch (n) {
#define PL_C(NN) case NN: return lanes_of<NN>();
    PL_PLANE_LENGTHS(PL_C)
#undef PL_C
    default: return 0;
  }
}

template <typename T>
struct Planes {
  int ny, nz, h, count;
  std::vector<cx<T>> in, out, twy, twz;
  std::vector<double> d, partials;
  std::vector<float> d32;
  RowArgs<T> a{};

  Planes(int ny_, int nz_, int count_) : ny(ny_), nz(nz_), h(nz_ / 2 + 1), count(count_), in(count_ * ny_ * (nz_ / 2 + 1)),
                                         out(in.size()), twy(ny_), twz(nz_), d(count_ * ny_ * nz_), partials(2 * count_, -1.0),
                                         d32(d.size()) {
    std::mt19937 gen(ny * 1000 + nz);
    std::normal_distribution<double> nd;
    for (auto& z : in) z = {(T)nd(gen), (T)nd(gen)};
    for (size_t i = 0; i < d.size(); ++i) {
      d32[i] = (float)std::fabs(nd(gen));
      d[i] = d32[i];
    }
    for (int e = 0; e < ny; ++e) twy[e] = {(T)std::cos(2 * M_PI * e / ny), (T)-std::sin(2 * M_PI * e / ny)};
    for (int e = 0; e < nz; ++e) twz[e] = {(T)std::cos(2 * M_PI * e / nz), (T)-std::sin(2 * M_PI * e / nz)};
    a.n = nz;
    a.nunits = count * ny / 2;
    a.in_c = in.data();
    a.out_c = out.data();
    a.tw = twz.data();
    a.tw_y = twy.data();
    a.ny = ny;
    a.nplanes = count;
    a.d = d.data();
    a.d32 = d32.data();
    a.scale = T(0.5);
    a.partials = partials.data();
  }

  // plane k by sums: returns the largest error over the plane's largest value,
  // and the sum of d v^2 in *dv
  double error(int k, double* dv) const {
    const double s = 0.5;
    std::vector<C> X(ny * h), y(ny * h), Y(ny * h), ey(ny), ez(nz);
    for (int e = 0; e < ny; ++e) ey[e] = std::polar(1.0, 2 * M_PI * e / ny);
    for (int e = 0; e < nz; ++e) ez[e] = std::polar(1.0, 2 * M_PI * e / nz);
    for (int i = 0; i < ny * h; ++i) X[i] = {in[(size_t)k * ny * h + i].x, in[(size_t)k * ny * h + i].y};
    for (int r = 0; r < ny; ++r)
      for (int q = 0; q < ny; ++q)
        for (int c = 0; c < h; ++c) y[r * h + c] += X[q * h + c] * ey[(size_t)r * q % ny];
    *dv = 0.0;
    std::vector<double> v(nz);
    for (int r = 0; r < ny; ++r) {
      for (int z = 0; z < nz; ++z) {
        double t = y[r * h].real() + (z & 1 ? -1.0 : 1.0) * y[r * h + h - 1].real();
        for (int c = 1; c < h - 1; ++c) t += 2.0 * (y[r * h + c] * ez[(size_t)z * c % nz]).real();
        const double dd = d[((size_t)k * ny + r) * nz + z];
        *dv += dd * (t * s) * (t * s);
        v[z] = dd * t * s;
      }
      for (int c = 0; c < h; ++c) {
        C f = 0.0;
        for (int z = 0; z < nz; ++z) f += v[z] * std::conj(ez[(size_t)z * c % nz]);
        y[r * h + c] = f;
      }
    }
    for (int r = 0; r < ny; ++r)
      for (int q = 0; q < ny; ++q)
        for (int c = 0; c < h; ++c) Y[r * h + c] += y[q * h + c] * std::conj(ey[(size_t)r * q % ny]);
    double err = 0.0, top = 0.0;
    for (int i = 0; i < ny * h; ++i) {
      const cx<T> o = out[(size_t)k * ny * h + i];
      err = std::max(err, std::abs(Y[i] - C(o.x, o.y)));
      top = std::max(top, std::abs(Y[i]));
    }
    return err / top;
  }
};

static int group_waves(int ny, int nz, int most) {
  const int cols = (nz / 2 + 64 / lanes(ny)) / (64 / lanes(ny)), rows = (ny / 2 + 64 / lanes(nz) - 1) / (64 / lanes(nz));
  const int groups = std::max(cols, rows), rounds = (groups + most - 1) / most;
  return (groups + rounds - 1) / rounds;
}

template <typename F>
void run(int waves, size_t lds, F f) {
  std::vector<int> order(waves);
  for (int i = 0; i < waves; ++i) order[i] = i;
  UNPOISON(plane_lds, sizeof(plane_lds));
  std::fill(plane_lds, plane_lds + sizeof(plane_lds), (char)0x7f);
  POISON(plane_lds + lds, sizeof(plane_lds) - lds);
  hostgpu::run_block(64 * waves, order, f, [](int) {});
  UNPOISON(plane_lds, sizeof(plane_lds));
}

template <typename T>
void report(const char* what, const Planes<T>& p, int waves, double sum, int records) {
  const double tol = sizeof(T) == 8 ? 1e-14 : 1e-6;  // a few roundings of each of the four transforms
  double err = 0.0, dv = 0.0, got = 0.0;
  for (int k = 0; k < p.count; ++k) {
    double s;
    err = std::max(err, p.error(k, &s));
    dv += s;
  }
  for (int i = 0; i < records; ++i) got += p.partials[2 * i];
  const double es = std::fabs(got - dv) / dv;
  const bool ok = err <= tol && es <= 10 * tol;
  g_ok = g_ok && ok;
  std::printf("%s %d x %d FP%d, %d waves: error %.1e, sum %.1e ok=%d\n", what, p.ny, p.nz, (int)sizeof(T) * 8, waves, err, es,
              (int)ok);
}

template <typename T>
void single(int ny, int nz) {
  Planes<T> p(ny, nz, 1);
  const int waves = group_waves(ny, nz, 10);
  gridDim = {1, 1, 1};
  blockIdx = {0, 0, 0};
  run(waves, plane_lds_bytes(ny, nz, sizeof(cx<T>)), [&] {
    if (plane_class(ny, nz) == 0)
      plane_kernel<T, ROW_HVP, 0>(p.a);
    else
      plane_kernel<T, ROW_HVP, 1>(p.a);
  });
  report("plane", p, waves, 0.0, 1);
}

// three planes of one instance in a block of eight waves, four slots
template <typename T>
void batched(int ny, int nz) {
  Planes<T> p(ny, nz, 3);
  const int waves = group_waves(ny, nz, 8);
  const int4 work = {0, 0, waves | (8 / waves) << 8, 0};
  gridDim = {1, 1, 1};
  blockIdx = {0, 0, 0};
  run(8, (8 / waves) * plane_lds_bytes(ny, nz, sizeof(cx<T>)), [&] { row_batch_kernel<T, ROW_HVP, 0>(&p.a, &work); });
  report("batch", p, waves, 0.0, 3);
}

int main() {
  // each length on both axes; the largest planes; columns and pairs that do
  // not fill a wave
  const int shapes[][2] = {{128, 8}, {128, 12}, {128, 16}, {8, 24},  {12, 32},  {16, 48},  {24, 24},   {24, 192}, {48, 32},
                           {32, 96}, {96, 48},  {64, 64},  {192, 24}, {96, 96},  {128, 64}, {64, 128}, {256, 24}, {24, 256}};
  for (const auto& s : shapes) {
    single<double>(s[0], s[1]);
    single<float>(s[0], s[1]);
  }
  single<double>(128, 128);
  single<double>(256, 64);
  single<double>(96, 192);
  single<float>(192, 192);
  single<float>(256, 128);
  batched<double>(32, 32);
  batched<float>(32, 48);
  return g_ok ? 0 : 1;
}
