// Variance of the long background mode in the survey disk, for the
// super-sample term resolved along the line of sight.
//
// Rizzato et al. (2019), arXiv 1812.07437: sigma_W^2(chi) is defined after
// eq. CovPP22 (Sec. 3.2.3); the disk is the thin-shell limit of the cylinder
// window of eq. Mask (App. B).  In polar coordinates,
//   sigma_W^2(chi) = (2 / pi) int eps^2 [J1(x) / x]^2 P(eps, chi) d ln eps,
//   x = eps chi Theta,
// with Theta the survey's angular radius, Omega = 2 pi (1 - cos Theta) (the
// relation given after eq. PSest, Sec. 3.2.2).  The integral runs over the k table by the trapezoid rule in ln eps
// on WINDOW_NODES uniformly spaced nodes, the two end nodes being the table's
// first and last k; P is read by the table interpolation of every other
// kernel (linear in ln P against ln k).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"

namespace wlc {

constexpr double PI_D = 3.14159265358979323846;

// Bessel function of the first kind of order one, x > 0 (Abramowitz &
// Stegun, ch. 9):
//   x < 2        its power series (9.1.10), terms falling at least 6-fold;
//   2 <= x < 25  Bessel's integral J1(x) = (1/pi) int_0^pi cos(t - x sin t) dt
//                (9.1.21) by the trapezoid rule on 32 intervals; for this
//                periodic analytic integrand the rule is exact up to
//                J_65(x) - J_63(x), below 1e-18 here, the two end terms
//                cancel (cos 0 + cos pi = 0), and those at t and pi - t add to
//                cos(t - x sin t) - cos(t + x sin t) = 2 sin t sin(x sin t);
//   x >= 25      Hankel's expansion (9.2.5, 9.2.9, 9.2.10) with mu = 4:
//                J1 = sqrt(2 / (pi x)) (P cos w - Q sin w), w = x - 3 pi / 4,
//                rewritten through sin x and cos x (exactly reduced by the
//                math library) as (P (sin x - cos x) + Q (sin x + cos x)) /
//                sqrt(pi x); the terms t_k = t_(k-1) (mu - (2k - 1)^2) / (8 k x)
//                fall for every k < 2x and are summed down to 1e-17.
// tab[0 .. 15] = sin(j pi / 32), tab[16 + k] = (4 - (2k - 1)^2) / (8 k) with the
// signs of P and Q, tab[47 + m] = -1 / (4 m (m + 1)).
constexpr int J1_TERMS = 30, J1_SERIES = 14;
constexpr int J1_TAB = 16 + J1_TERMS + 1 + J1_SERIES + 1;

__device__ __forceinline__ double bessel_tab(int i) {
  if (i < 16) return sin(i * (PI_D / 32.0));
  if (i > 16 + J1_TERMS) {
    const int m = i - 17 - J1_TERMS;
    return m == 0 ? 0.0 : -0.25 / (double)(m * (m + 1));
  }
  const int k = i - 16;
  // k = 1, 2, 3, 4, ... contributes +Q, -P, -Q, +P, ...: a sign change at every even k
  return k == 0 ? 0.0 : (double)(4 - (2 * k - 1) * (2 * k - 1)) / (8.0 * k) * ((k & 1) ? 1.0 : -1.0);
}

__device__ __forceinline__ double bessel_j1(double x, const double *tab) {
  if (x < 2.0) {
    const double q = x * x;
    double t = 0.5 * x, s = t;
    for (int m = 1; m <= J1_SERIES; ++m) {
      t *= q * tab[17 + J1_TERMS + m];
      s += t;
    }
    return s;
  }
  if (x < 25.0) {
    double s = 0.0;
    for (int j = 1; j < 16; ++j) s += tab[j] * sin(x * tab[j]);
    return (2.0 * s + sin(x)) * (1.0 / 32.0);
  }
  double P = 1.0, Q = 0.0, t = 1.0;
  const double inv = 1.0 / x;
  for (int k = 1; k < J1_TERMS; k += 2) {
    t *= tab[16 + k] * inv;
    Q += t;
    t *= tab[17 + k] * inv;
    P += t;
    if (fabs(t) < 1e-17) break;
  }
  double sx, cx;
  sincos(x, &sx, &cx);
  return (P * (sx - cx) + Q * (sx + cx)) / sqrt(PI_D * x);
}

// One workgroup per chi node: threads stride over the window nodes, then a
// block reduction of the trapezoid sum.  STAGED: ln k and ln P of the node's
// table row are taken once, into LDS (tables of up to SIG_NK nodes, its 64 KB;
// longer ones are read and their logarithms taken for every window node).  A
// node's eps^2 P is one exponential of its ln eps.
//
// Bound by FP64 arithmetic (two exponentials, a sine and cosine, a square root
// and two divisions for every node): 256 chi nodes 69 us (83 with a bisection for every node), against 284 with the
// interval, four logarithms of the table and twice the sines found for every node.
constexpr int SIG_THREADS = 512;
constexpr int SIG_NK = 4000;
template <bool STAGED>
__global__ __launch_bounds__(SIG_THREADS) void k_sigma_w2(DevTables T, double theta, int base, double *sw) {
  extern __shared__ double lds[];  // ln k, ln P [n_k] each
  __shared__ double tab[J1_TAB];
  __shared__ double part[SIG_THREADS / WAVE];
  const int n = base + blockIdx.x, nk = T.n_k;
  double *lk = lds, *lp = lds + nk;
  for (int i = threadIdx.x; i < J1_TAB; i += SIG_THREADS) tab[i] = bessel_tab(i);
  if constexpr (STAGED)
    for (int i = threadIdx.x; i < nk; i += SIG_THREADS) {
      lk[i] = log(T.k[i]);
      lp[i] = log(T.P[(size_t)n * nk + i]);
    }
  __syncthreads();
  auto ln_k = [&](int i) { return STAGED ? lk[i] : log(T.k[i]); };
  auto ln_p = [&](int i) { return STAGED ? lp[i] : log(T.P[(size_t)n * nk + i]); };
  const double scale = T.chi[n] * theta;
  const double l0 = ln_k(0), l1 = ln_k(nk - 1);
  const double h = (l1 - l0) / (WINDOW_NODES - 1), even = (nk - 1) / (l1 - l0);
  double s = 0.0;
  for (int j = threadIdx.x; j < WINDOW_NODES; j += SIG_THREADS) {
    const double le = j == WINDOW_NODES - 1 ? l1 : l0 + j * h;
    const double eps = exp(le), x = eps * scale;
    // the last lo <= n_k - 2 at or below the node: on a table even in ln k where
    // it should be, else by bisection
    int lo = 0, hi = nk - 1;
    if constexpr (STAGED) {
      const int g = min(max((int)((le - l0) * even), 0), nk - 2);
      if (lk[g] <= le && (g == nk - 2 || le < lk[g + 1])) lo = g, hi = g + 1;
    }
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (STAGED ? lk[mid] <= le : T.k[mid] <= eps) lo = mid; else hi = mid;
    }
    const double k0 = ln_k(lo), t = (le - k0) / (ln_k(lo + 1) - k0);
    const double win = bessel_j1(x, tab) / x;
    const double w = (j == 0 || j == WINDOW_NODES - 1) ? 0.5 * h : h;
    s += w * win * win * exp(2.0 * le + ((1.0 - t) * ln_p(lo) + t * ln_p(lo + 1)));
  }
  s = wave_sum(s);
  if ((threadIdx.x & (WAVE - 1)) == 0) part[threadIdx.x / WAVE] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot = 0.0;
    for (int w = 0; w < SIG_THREADS / WAVE; ++w) tot += part[w];
    sw[n] = 2.0 / PI_D * tot;
  }
}

void launch_sigma_w2(const DevTables &T, double theta, double *sw, hipStream_t s) {
  const int most = (int)(LAUNCH_THREADS / SIG_THREADS);
  for (int base = 0; base < T.n_chi; base += most) {
    const dim3 grid((unsigned)std::min(most, T.n_chi - base));
    if (T.n_k <= SIG_NK)
      hipLaunchKernelGGL(k_sigma_w2<true>, grid, dim3(SIG_THREADS), (size_t)T.n_k * 16, s, T, theta, base, sw);
    else
      hipLaunchKernelGGL(k_sigma_w2<false>, grid, dim3(SIG_THREADS), 0, s, T, theta, base, sw);
  }
}

}  // namespace wlc
