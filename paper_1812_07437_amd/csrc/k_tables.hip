// Table staging, halo-model quadrature, Limber projection and the Gram factor.
//
// Rizzato et al. (2019), arXiv 1812.07437:
//   halo mass integrals I_mu^beta ............ eq. ImunuHalos (Sec. 4.1)
//   P_HM, B_HM ............................... eqs. PspHMtot2, B1halo, B2halos, B3halos (first line)
//   responses to a long mode ................. eqs. PowerHMResp, BispHMResp, RespP, RespB (Sec. 4.3)
//   Limber projection ........................ eq. nProjection (Sec. 3.1)
//   one-halo n-point function ................ eq. General1h (Sec. 4.2)
//   k_max cut of the line-of-sight integrand . Sec. 4.4
// Tables are read by linear interpolation of ln X in ln k between the
// bracketing nodes; d ln P / d ln k uses centred node differences (one-sided
// at the ends) interpolated linearly in ln k.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"

namespace wlc {

// ------------------------------------------------------------- validation
// flags[0]: a bad value; flags[1]: some ell/chi below k_max off the k table;
// flags[2]: theta > 0 and k_0 chi_max theta > 0.1 (the table starts above the
// scale of the survey window at the farthest node).
__global__ void k_validate(DevTables T, const double *centres, int n_ell, double theta, int *flags) {
  const int64_t nP = (int64_t)T.n_chi * T.n_k, nU = (int64_t)T.n_m_pts * T.n_k, nW = (int64_t)T.n_z * T.n_chi;
  const int64_t nM = T.n_m_pts, nC = T.n_chi, nK = T.n_k, nCov = (int64_t)n_ell * T.n_chi;
  const int64_t total = nP + nU + nW + nM + nC + nK + nCov;
  int bad = 0, range = 0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    int64_t q = i;
    if (q < nP) { double v = T.P[q]; bad |= !(isfinite(v) && v > 0.0); continue; }
    q -= nP;
    if (q < nU) { double v = T.u[q]; bad |= !(isfinite(v) && v > 0.0); continue; }
    q -= nU;
    if (q < nW) { double v = T.W[q]; bad |= !(isfinite(v) && v >= 0.0); continue; }
    q -= nW;
    if (q < nM) {
      bad |= !(isfinite(T.n_m[q]) && T.n_m[q] > 0.0);
      bad |= !(isfinite(T.m[q]) && T.m[q] > 0.0);
      bad |= !(isfinite(T.w_m[q]) && T.w_m[q] >= 0.0);
      if (T.b1) bad |= !isfinite(T.b1[q]);
      if (T.b2) bad |= !isfinite(T.b2[q]);
      continue;
    }
    q -= nM;
    if (q < nC) {
      bad |= !(isfinite(T.chi[q]) && T.chi[q] > 0.0 && isfinite(T.w_chi[q]) && T.w_chi[q] >= 0.0);
      if (q > 0) bad |= !(T.chi[q] > T.chi[q - 1]);
      continue;
    }
    q -= nC;
    if (q < nK) {
      bad |= !(isfinite(T.k[q]) && T.k[q] > 0.0);
      if (q > 0) bad |= !(T.k[q] > T.k[q - 1]);
      continue;
    }
    q -= nK;
    {
      const int b = (int)(q / T.n_chi), n = (int)(q % T.n_chi);
      const double kk = centres[b] / T.chi[n];
      if (kk <= T.k_max && !(kk >= T.k[0] && kk <= T.k[T.n_k - 1])) range = 1;
    }
  }
  if (bad) atomicOr(&flags[0], 1);
  if (range) atomicOr(&flags[1], 1);
  if (theta > 0.0 && blockIdx.x == 0 && threadIdx.x == 0 && !(T.k[0] * T.chi[T.n_chi - 1] * theta <= 0.1))
    atomicOr(&flags[2], 1);
}

void launch_validate(const DevTables &T, const double *centres, int n_ell, double theta, int *flags,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_validate, dim3(512), dim3(256), 0, s, T, centres, n_ell, theta, flags);
}

// ------------------------------------------------------------- staging
// One wavefront per (staged ell value l, chi node n): the k interval of
// l / chi_n is found once for the node (two or three rounds of 64 probes), lanes stride
// over the masses of U[l][n][m] = u(m, l / chi_n), and the same pass sums
// I_1^1 over them.  Lanes 0 to 3 hold the four table nodes that P and its
// logarithmic slope take.  Everything is 0 above k_max.
// The wavefronts past the last node fill the chi factors that the rows of
// either kind share, F[4][n_chi]: w chi^-2 and w chi^-4 of the projections
// (p = 2, 3 legs), sqrt(w) chi^-3 and sqrt(w) chi^-5 of the Gram factor.
//
// Bound by the latency of its loads and logarithms: at 30 sub-bins, 256 chi
// nodes and 128 masses 22 us (with an interval search for every mass 26, and
// 9 for P and the slope).

// The last j <= nk - 2 with kg[j] <= kk, for kg[0] <= kk <= kg[nk - 1], by a
// wavefront.
__device__ __forceinline__ int wave_bracket(const double *kg, int nk, double kk, int lane) {
  int lo = 0, hi = nk - 1;
  while (hi - lo > 1) {
    const int step = (hi - lo + WAVE - 1) / WAVE;
    const int q = lo + lane * step;
    const bool below = q < hi && kg[q] <= kk;
    lo += (max(__popcll(__ballot(below)), 1) - 1) * step;
    hi = min(hi, lo + step);
  }
  return min(lo, nk - 2);
}

__global__ __launch_bounds__(256) void k_stage(DevTables T, const double *__restrict__ centres, int n_ls, int base,
                                               double *U, LegTerm *legs, double *F) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int item = __builtin_amdgcn_readfirstlane(base + blockIdx.x * (256 / WAVE) + threadIdx.x / WAVE);
  const int nm = T.n_m_pts;
  if (item >= n_ls * T.n_chi) {
    const int q = (item - n_ls * T.n_chi) * WAVE + lane;
    if (q < 4 * T.n_chi) {
      const int f = q / T.n_chi, n = q % T.n_chi;
      const double w = T.w_chi[n];
      F[q] = f < 2 ? w * pow(T.chi[n], f == 0 ? -2.0 : -4.0) : sqrt(w) * pow(T.chi[n], f == 2 ? -3.0 : -5.0);
    }
    return;
  }
  const int l = item / T.n_chi, n = item % T.n_chi;
  const double kk = centres[l] / T.chi[n];
  double *Uo = U + (size_t)item * nm;
  LegTerm leg = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (kk <= T.k_max && kk >= T.k[0] && kk <= T.k[T.n_k - 1]) {
    const int j = wave_bracket(T.k, T.n_k, kk, lane);
    // nodes j - 1 .. j + 2, the end nodes twice at the ends of the table
    const int jn = min(max(j - 1 + (lane & 3), 0), T.n_k - 1);
    const double lk = log(T.k[jn]), lp = log(T.P[(size_t)n * T.n_k + jn]);
    const double k0 = __shfl(lk, 0), k1 = __shfl(lk, 1), k2 = __shfl(lk, 2), k3 = __shfl(lk, 3);
    const double p0 = __shfl(lp, 0), p1 = __shfl(lp, 1), p2 = __shfl(lp, 2), p3 = __shfl(lp, 3);
    const double t = (log(kk) - k1) / (k2 - k1);
    double i1 = 0.0;
    for (int mi = lane; mi < nm; mi += WAVE) {
      const double *row = T.u + (size_t)mi * T.n_k + j;
      const double u = exp((1.0 - t) * log(row[0]) + t * log(row[1]));
      Uo[mi] = u;
      i1 += T.w_m[mi] * T.n_m[mi] * (T.b1 ? T.b1[mi] : 1.0) * (T.m[mi] / T.rho) * u;
    }
    leg.i1 = wave_sum(i1);
    leg.p = exp((1.0 - t) * p1 + t * p2);
    leg.ne = (1.0 - t) * ((p2 - p0) / (k2 - k0)) + t * ((p3 - p1) / (k3 - k1));
    leg.lin = leg.i1 * leg.p;
    leg.resp = leg.i1 * (47.0 / 21.0 * leg.p - leg.ne * leg.p / 3.0);
  } else {
    for (int mi = lane; mi < nm; mi += WAVE) Uo[mi] = 0.0;
  }
  if (lane == 0) legs[item] = leg;
}

void launch_stage(const DevTables &T, const double *centres, int n_ls, double *U, LegTerm *legs, double *F,
                  hipStream_t s) {
  const int64_t waves = (int64_t)n_ls * T.n_chi + (4 * T.n_chi + WAVE - 1) / WAVE, most = LAUNCH_THREADS / WAVE;
  for (int64_t base = 0; base < waves; base += most)
    hipLaunchKernelGGL(k_stage, dim3((unsigned)((std::min(most, waves - base) + 3) / 4)), dim3(256), 0, s, T, centres,
                       n_ls, (int)base, U, legs, F);
}

// ------------------------------------------------------------- 3-D spectra
// One wavefront per (configuration, chi node) gives the spectrum X, its
// response R and the Gram factor G, all averaged over the configuration's
// list of ell-triples (its bin centres, or its sub-bins, with weights w_e).
//
// The one-halo (p_a + p_b)-point function factorises over the legs of each
// row (eq. General1h), so
//   A[row][(n, m)] = sqrt(w_n) chi_n^-(2p-1) prod_i W_i(chi_n)        (= T[row][n])
//                  * sqrt(w_m n_m) (m/rho)^p prod_legs u(m, l/chi_n)   (= G[cfg][n][m])
// and (1/Omega) A A^T is the one-halo covariance of eqs. CovPPNG, Ins5P, Ins6P.
// With sw, one more column per chi node carries the super-sample term of eq.
// WLSSCflatskyLimber resolved along chi,
//   sum_n w_n sigma_W^2(chi_n) chi_n^(2-2p) prod W R_cfg(chi_n) (same for b),
// as G[cfg][n][n_m] = sqrt(Omega) chi_n sqrt(sigma_W^2(chi_n)) R[cfg][n].
//
// Every mass integral of X and R is linear in products of u over legs, with
// factors (I_1^1 P and I_1^1 P_response of the other leg) that do not depend on the
// mass, so the list is summed first, for each mass, and one reduction over the
// masses serves the whole list:
//   t = sum_e w_e u0 u1 u2,  h = sum_e w_e sum_a (I11 P)_a u_b u_c,  r alike with the
//   response factor;  X = sum_m w_m n_m x^2 (x t + b1 h) + tree terms,
//   R = sum_m w_m n_m x^2 (b2 h + b1 r + b1 x t) + tree terms.
// Entries that share their first two legs are consecutive, and only the third
// one's u is read for each.  The tree terms take one entry per lane.
//
// At 74 configurations of up to 27 sub-bin triples, 256 chi nodes and 128
// masses 74 us, where a reduction over the masses for every integral of every
// entry and a second pass for G took 560 + 119; bound by FP64 arithmetic at the
// four wavefronts a SIMD that the rows in LDS leave.
// the value that lane i (the same for all) holds
__device__ __forceinline__ double lane_value(double x, int i) {
  const int64_t b = __double_as_longlong(x);
  const uint32_t lo = __builtin_amdgcn_readlane((int)b, i), hi = __builtin_amdgcn_readlane((int)(b >> 32), i);
  return __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ double cosine3(double ki, double kj, double kl) {
  return (kl * kl - ki * ki - kj * kj) / (2.0 * ki * kj);
}

// SUB: with S sub-bins to a bin the 3 S rows of u that a configuration's entries
// take again and again lie in LDS, one wavefront's beside the other's, and the
// entries and their legs come from one lane each instead of a chain of loads
// for every entry (at the sizes above 74 us; from memory, a load each, 84).  Bin
// centres have one entry and take each row once: they stay with memory and loads
// (3276 configurations of 64 nodes: 120 us, with lanes 146).  Rows past LDS_U
// bytes, two workgroups to a CU, do too.
constexpr int64_t LDS_U = 64 * 1024;
template <bool SUB>
__global__ __launch_bounds__(256) void k_spectra(DevTables T, const int32_t *__restrict__ cfgT, int n_cfg,
                                                 const int32_t *__restrict__ first,
                                                 const int4 *__restrict__ lists,
                                                 const double *__restrict__ weights, const double *__restrict__ U,
                                                 const LegTerm *__restrict__ legs,
                                                 const double *__restrict__ centres, const double *__restrict__ sw,
                                                 double sq_omega, int n_mg, int S, double *X, double *R, double *G,
                                                 double *Gmax, double *Gsq) {
  extern __shared__ double lds[];
  const int lane = threadIdx.x & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int item = __builtin_amdgcn_readfirstlane(blockIdx.x * (256 / WAVE) + wave);
  if (item >= n_cfg * T.n_chi) return;
  const int c = item / T.n_chi, n = item % T.n_chi, nm = T.n_m_pts;
  const bool tri = cfgT[4 * c] == 3;
  const int e0 = first[c], e1 = first[c + 1];
  const double chi = T.chi[n];
  double xs = 0.0, rs = 0.0, mx = 0.0, sq = 0.0;
  // the terms without a mass integral over more than one leg
  for (int e = e0 + lane; e < e1; e += WAVE) {
    const int4 q = lists[e];
    const double w = weights[e];
    const LegTerm a = legs[(size_t)q.x * T.n_chi + n];
    if (!tri) {
      xs += w * a.i1 * a.i1 * a.p;
      rs += w * a.i1 * a.resp;
      continue;
    }
    const LegTerm b = legs[(size_t)q.y * T.n_chi + n], d = legs[(size_t)q.z * T.n_chi + n];
    const double P[3] = {a.p, b.p, d.p}, ne[3] = {a.ne, b.ne, d.ne};
    const double kv[3] = {centres[q.x] / chi, centres[q.y] / chi, centres[q.z] / chi};
    double Bpt = 0.0, Bg2 = 0.0, dil = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int j = (i + 1) % 3, l = (i + 2) % 3;
      const double mu = cosine3(kv[i], kv[j], kv[l]);
      const double Fk = 5.0 / 7.0 + 0.5 * mu * (kv[i] / kv[j] + kv[j] / kv[i]) + 2.0 / 7.0 * mu * mu;
      Bpt += 2.0 * Fk * P[i] * P[j];
      Bg2 += 2.0 * (mu * mu - 1.0) * P[i] * P[j];
      dil += 2.0 * Fk * P[i] * P[j] * (ne[i] + ne[j]);
    }
    const double I111 = w * a.i1 * b.i1 * d.i1;
    xs += I111 * Bpt;
    rs += I111 * (433.0 / 126.0 * Bpt + 5.0 / 126.0 * Bg2 - dil / 3.0);
  }
  double *Go = G + (size_t)item * n_mg;
  const size_t at = (size_t)n * nm, step = (size_t)T.n_chi * nm;
  const int bin[3] = {cfgT[4 * c + 1], cfgT[4 * c + 2], cfgT[4 * c + 3]};
  double *rows = lds + (size_t)wave * 3 * S * nm;
  if constexpr (SUB) {
    for (int a = 0; a < (tri ? 3 : 1); ++a) {
      const double *Ua = U + (size_t)bin[a] * S * step + at;
      double *dst = rows + a * S * nm;
      int mi = lane % nm, q = lane / nm;
#pragma unroll 6
      for (int e = lane; e < S * nm; e += WAVE) {
        dst[e] = Ua[q * step + mi];
        for (mi += WAVE; mi >= nm; mi -= nm) ++q;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  // u of leg a, staged ell value l, mass mi
  auto u_of = [&](int a, int l, int mi) {
    if constexpr (SUB) return rows[(a * S + l - bin[a] * S) * nm + mi];
    else return U[l * step + at + mi];
  };
  for (int m0 = 0; m0 < nm; m0 += 2 * WAVE) {
    const bool in0 = m0 + lane < nm, in1 = m0 + WAVE + lane < nm;
    const int mi[2] = {in0 ? m0 + lane : nm - 1, in1 ? m0 + WAVE + lane : nm - 1};
    double t[2] = {0.0, 0.0}, h[2] = {0.0, 0.0}, r[2] = {0.0, 0.0};
    if constexpr (SUB) {
      // a run: the entries that share l0, l1; v, lin and resp sum over their third leg
      int l0 = -1, l1 = -1;
      double u0[2] = {0.0, 0.0}, u1[2] = {0.0, 0.0}, v[2] = {0.0, 0.0}, lin = 0.0, resp = 0.0;
      double lin0 = 0.0, lin1 = 0.0, resp0 = 0.0, resp1 = 0.0;
      auto run_ends = [&]() {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const double u01 = u0[j] * u1[j];
          t[j] += u01 * v[j];
          h[j] += (lin0 * u1[j] + lin1 * u0[j]) * v[j] + u01 * lin;
          r[j] += (resp0 * u1[j] + resp1 * u0[j]) * v[j] + u01 * resp;
          v[j] = 0.0;
        }
        lin = resp = 0.0;
      };
      // 64 entries at a time, one in each lane, and from there to all lanes in turn
      for (int eb = e0; eb < e1; eb += WAVE) {
        const int e = min(eb + lane, e1 - 1), cnt = min(WAVE, e1 - eb);
        const int4 q = lists[e];
        const double w = weights[e];
        LegTerm a = {}, b = {}, d = {};
        if (tri) {
          a = legs[(size_t)q.x * T.n_chi + n];
          b = legs[(size_t)q.y * T.n_chi + n];
          d = legs[(size_t)q.z * T.n_chi + n];
        }
        const double wl = w * d.lin, wr = w * d.resp;
        for (int i = 0; i < cnt; ++i) {
          const double wi = lane_value(w, i);
          const int x = __builtin_amdgcn_readlane(q.x, i);
          if (!tri) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              const double u = u_of(0, x, mi[j]);
              t[j] += wi * (u * u);
            }
            continue;
          }
          const int y = __builtin_amdgcn_readlane(q.y, i), z = __builtin_amdgcn_readlane(q.z, i);
          if (x != l0 || y != l1) {
            run_ends();
            l0 = x;
            l1 = y;
            lin0 = lane_value(a.lin, i);
            lin1 = lane_value(b.lin, i);
            resp0 = lane_value(a.resp, i);
            resp1 = lane_value(b.resp, i);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              u0[j] = u_of(0, x, mi[j]);
              u1[j] = u_of(1, y, mi[j]);
            }
          }
          v[0] += wi * u_of(2, z, mi[0]);
          v[1] += wi * u_of(2, z, mi[1]);
          lin += lane_value(wl, i);
          resp += lane_value(wr, i);
        }
      }
      if (tri) run_ends();
    } else {
      int4 q = lists[e0];
      for (int e = e0; e < e1;) {
        const int l0 = q.x, l1 = q.y;
        const double u0[2] = {u_of(0, l0, mi[0]), u_of(0, l0, mi[1])};
        if (!tri) {
          const double w = weights[e];
          t[0] += w * (u0[0] * u0[0]);
          t[1] += w * (u0[1] * u0[1]);
          if (++e < e1) q = lists[e];
          continue;
        }
        const double u1[2] = {u_of(1, l1, mi[0]), u_of(1, l1, mi[1])};
        const LegTerm &a0 = legs[(size_t)l0 * T.n_chi + n], &a1 = legs[(size_t)l1 * T.n_chi + n];
        double v[2] = {0.0, 0.0}, lin = 0.0, resp = 0.0;
        do {
          const double w = weights[e];
          const LegTerm &a2 = legs[(size_t)q.z * T.n_chi + n];
          v[0] += w * u_of(2, q.z, mi[0]);
          v[1] += w * u_of(2, q.z, mi[1]);
          lin += w * a2.lin;
          resp += w * a2.resp;
          if (++e == e1) break;
          q = lists[e];
        } while (q.x == l0 && q.y == l1);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const double u01 = u0[j] * u1[j];
          t[j] += u01 * v[j];
          h[j] += (a0.lin * u1[j] + a1.lin * u0[j]) * v[j] + u01 * lin;
          r[j] += (a0.resp * u1[j] + a1.resp * u0[j]) * v[j] + u01 * resp;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (!(j == 0 ? in0 : in1)) continue;
      const double x = T.m[mi[j]] / T.rho, wn = T.w_m[mi[j]] * T.n_m[mi[j]];
      const double b1 = T.b1 ? T.b1[mi[j]] : 1.0, b2 = T.b2 ? T.b2[mi[j]] : 0.0;
      const double f = tri ? x * t[j] : t[j];
      xs += wn * x * x * (f + b1 * h[j]);
      rs += wn * x * x * (b2 * h[j] + b1 * (r[j] + f));
      const double g = sqrt(wn) * x * x * f;
      Go[mi[j]] = g;
      mx = fmax(mx, fabs(g));
      sq += g * g;
    }
  }
  xs = wave_sum(xs);
  rs = wave_sum(rs);
  if (sw) {
    const double g = sq_omega * chi * sqrt(sw[n]) * rs;
    if (lane == 0) {
      Go[nm] = g;
      sq += g * g;
    }
    mx = fmax(mx, fabs(g));
  }
  mx = wave_max(mx);
  if (Gsq) sq = wave_sum(sq);
  if (lane == 0) {
    X[item] = xs;
    R[item] = rs;
    Gmax[item] = mx;
    if (Gsq) Gsq[item] = sq;
  }
}

void launch_spectra(const DevTables &T, const int32_t *cfgT, int n_cfg, const SubList &sl, const double *U,
                    const LegTerm *legs, const double *centres, const double *sw, double sq_omega, int n_mg, int n_sub,
                    double *X, double *R, double *G, double *Gmax, double *Gsq, hipStream_t s) {
  const int64_t items = (int64_t)n_cfg * T.n_chi, bytes = (int64_t)4 * 3 * n_sub * T.n_m_pts * 8;
  const dim3 grid((unsigned)((items + 3) / 4));
  if (n_sub > 1 && bytes <= LDS_U)
    hipLaunchKernelGGL(k_spectra<true>, grid, dim3(256), (size_t)bytes, s, T, cfgT, n_cfg, sl.off,
                       (const int4 *)sl.leg, sl.w, U, legs, centres, sw, sq_omega, n_mg, n_sub, X, R, G, Gmax, Gsq);
  else
    hipLaunchKernelGGL(k_spectra<false>, grid, dim3(256), 0, s, T, cfgT, n_cfg, sl.off, (const int4 *)sl.leg, sl.w,
                       U, legs, centres, sw, sq_omega,
                       n_mg, n_sub, X, R, G, Gmax, Gsq);
}

// ------------------------------------------------------------- rows
// One wavefront per distinct row, lanes over chi: the projections d and r,
// the row's factor T[n] with the exponent s = -e, max_k |A[row][k]| = f 2^e,
// f in [0.5, 1), Ts[row][n] = 2^s T[n], the last chi node with a nonzero Ts
// (-1: none) and, with Gsq (sum_m G^2), the row's Gram diagonal
// sum_n Ts^2 Gsq.  The power-spectrum rows lead, and also give the shot-noise power
// P^s_ij(l_b) = P_ij(l_b) + delta_ij sigma_eps^2 / n_i (eq. ShotNoise).
// Bound by the write of Ts: 33165 rows of 512 nodes take 113 us (1.3 TB/s), against
// 133 + 285 for projection and factor with powers of chi for every row.
__global__ __launch_bounds__(256) void k_rows(DevTables T, const int32_t *__restrict__ rowR,
                                              const int32_t *__restrict__ cfgT, int64_t n_R,
                                              const double *__restrict__ F, const double *__restrict__ X,
                                              const double *__restrict__ R, const double *__restrict__ Gmax,
                                              const double *__restrict__ Gsq, double noise, double *dR, double *rR,
                                              double *Ps, double *Ts, int32_t *sexp, int32_t *last, double *gd) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t row = (int64_t)blockIdx.x * (256 / WAVE) + threadIdx.x / WAVE;
  if (row >= n_R) return;
  const int4 rc = ((const int4 *)rowR)[row];
  const int c = rc.x, nc = T.n_chi;
  const bool tri = cfgT[4 * c] == 3;
  const double *W0 = T.W + (size_t)rc.y * nc, *W1 = T.W + (size_t)rc.z * nc;
  const double *W2 = tri ? T.W + (size_t)rc.w * nc : nullptr;
  const double *Fp = F + (tri ? nc : 0), *Ft = Fp + 2 * nc;
  const double *Xc = X + (size_t)c * nc, *Rc = R + (size_t)c * nc, *gm = Gmax + (size_t)c * nc;
  double sd = 0.0, sr = 0.0, mx = 0.0;
  for (int n = lane; n < nc; n += WAVE) {
    double w = W0[n] * W1[n];
    if (tri) w *= W2[n];
    const double pw = Fp[n] * w;
    sd += pw * Xc[n];
    sr += pw * Rc[n];
    mx = fmax(mx, fabs(Ft[n] * w) * gm[n]);
  }
  mx = wave_max(mx);
  const int s = -exp2_of(mx);
  double dg = 0.0;
  int top = -1;
  for (int n = lane; n < nc; n += WAVE) {
    double w = W0[n] * W1[n];
    if (tri) w *= W2[n];
    const double t = ldexp(Ft[n] * w, s);
    Ts[(size_t)row * nc + n] = t;
    if (t != 0.0) top = n;
    if (Gsq) dg += t * t * Gsq[(size_t)c * nc + n];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o, WAVE));
  sd = wave_sum(sd);
  sr = wave_sum(sr);
  if (Gsq) dg = wave_sum(dg);
  if (lane == 0) {
    dR[row] = sd;
    rR[row] = sr;
    sexp[row] = s;
    last[row] = top;
    if (Gsq) gd[row] = dg;
    if (!tri) {  // configuration c of kind 2 is ell-bin c
      double *P = Ps + (size_t)c * T.n_z * T.n_z;
      P[rc.y * T.n_z + rc.z] = P[rc.z * T.n_z + rc.y] = sd + (rc.y == rc.z ? noise : 0.0);
    }
  }
}

void launch_rows(const DevTables &T, const int32_t *rowR, const int32_t *cfgT, int64_t n_R, const double *F,
                 const double *X, const double *R, const double *Gmax, const double *Gsq, double noise, double *dR,
                 double *rR, double *Ps, double *Ts, int32_t *sexp, int32_t *last, double *gd, hipStream_t s) {
  hipLaunchKernelGGL(k_rows, dim3((unsigned)((n_R + 3) / 4)), dim3(256), 0, s, T, rowR, cfgT, n_R, F, X, R, Gmax,
                     Gsq, noise, dR, rR, Ps, Ts, sexp, last, gd);
}

// ------------------------------------------------------------- two-leg factors
// The projected one-halo trispectrum that enters the P.T term of eq. CovBB
// at the two remaining legs of each of two triangles factorises like the
// one-halo covariance: for a two-leg configuration (ell-bins p <= q) and
// bins (j at p, k at q),
//   T[(pq, jk)][(p'q', j'k')] = sum_n Ts2[(pq, jk)][n] Ts2[(p'q', j'k')][n]
//                               * sum_m G2[pq][n][m] G2[p'q'][n][m],
//   Ts2 = sqrt(w_n) chi_n^-3 W_j(chi_n) W_k(chi_n),
//   G2  = sqrt(w_m n_m) (m/rho)^2 u(m, l_p/chi_n) u(m, l_q/chi_n)
// (eq. nProjection with n = 4, I_4^0 of eq. ImunuHalos).  Configurations:
// p = q first (index p), then p < q in lexicographic order; rows: pairs
// j <= k for p = q, all n_z^2 ordered pairs (j, k) for p < q.
__global__ void k_g2factor(DevTables T, int n_ell, const double *U, double *G2) {
  const int n2 = n_ell + n_ell * (n_ell - 1) / 2;
  const int64_t total = (int64_t)n2 * T.n_chi * T.n_m_pts;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int mi = (int)(i % T.n_m_pts);
    const int64_t cn = i / T.n_m_pts;
    const int n = (int)(cn % T.n_chi), c = (int)(cn / T.n_chi);
    int p, q;
    if (c < n_ell) {
      p = q = c;
    } else {
      int r = c - n_ell;
      for (p = 0; r >= n_ell - 1 - p; ++p) r -= n_ell - 1 - p;
      q = p + 1 + r;
    }
    const double x = T.m[mi] / T.rho;
    G2[i] = sqrt(T.w_m[mi] * T.n_m[mi]) * x * x * U[((size_t)p * T.n_chi + n) * T.n_m_pts + mi] *
            U[((size_t)q * T.n_chi + n) * T.n_m_pts + mi];
  }
}

__global__ void k_t2factor(DevTables T, int n_ell, int64_t rows, double *Ts2) {
  const int nz = T.n_z, sp = nz * (nz + 1) / 2;
  const int64_t total = rows * T.n_chi;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int n = (int)(i % T.n_chi);
    const int64_t row = i / T.n_chi;
    int j, k;
    if (row < (int64_t)n_ell * sp) {
      int w = (int)(row % sp);
      for (j = 0; w >= nz - j; ++j) w -= nz - j;
      k = j + w;
    } else {
      const int w = (int)((row - (int64_t)n_ell * sp) % (nz * nz));
      j = w / nz;
      k = w % nz;
    }
    const double chi = T.chi[n];
    Ts2[i] = sqrt(T.w_chi[n]) / (chi * chi * chi) * T.W[(size_t)j * T.n_chi + n] * T.W[(size_t)k * T.n_chi + n];
  }
}

void launch_twoleg(const DevTables &T, int n_ell, const double *U, double *G2, double *Ts2, hipStream_t s) {
  const int n2 = n_ell + n_ell * (n_ell - 1) / 2;
  const int nz = T.n_z;
  const int64_t rows = (int64_t)n_ell * (nz * (nz + 1) / 2) + (int64_t)(n2 - n_ell) * nz * nz;
  const int64_t tg = (int64_t)n2 * T.n_chi * T.n_m_pts, tt = rows * T.n_chi;
  hipLaunchKernelGGL(k_g2factor, dim3((unsigned)std::min<int64_t>((tg + 255) / 256, 65536)), dim3(256), 0, s, T,
                     n_ell, U, G2);
  hipLaunchKernelGGL(k_t2factor, dim3((unsigned)std::min<int64_t>((tt + 255) / 256, 65536)), dim3(256), 0, s, T,
                     n_ell, rows, Ts2);
}

// ------------------------------------------------------------- A build
// A[row][k], k = n * n_m + m; rows >= n_R and k >= n_chi * n_m are zero.  A
// row of A is T_row(chi_n) G_cfg(chi_n, M_m).  The write traffic is the
// kernel's whole HBM cost.
//
// Row-major f64 / f32 ([r_pad][lda]): consecutive rows mostly share their
// configuration, so each block holds 8 consecutive k of G_cfg per thread in
// registers and writes them, times T_row, for `rows` consecutive rows,
// reloading G only where the configuration changes.  With arow, row r of A
// is the distinct row arow[r] (zero where it is negative), and with ext a
// 256-row panel is written up to its last k-block (no product reads it there).
// rows is AB_ROWS, or as many fewer as it takes for 1024 workgroups: a row is a
// chain of loads, and a small product is over sooner with more of them side by side (256
// rows of 2048 k in FP64: 8 us, with 16 rows to each of 16 workgroups 26).
constexpr int AB_ROWS = 16;

template <int FMT>
__global__ __launch_bounds__(256) void k_abuild(const int32_t *__restrict__ rowR, const double *__restrict__ Ts,
                                               const double *__restrict__ G, int64_t n_R, int n_chi, int n_m,
                                               int64_t k_pad, int64_t lda, void *A0, void *A1,
                                               const int32_t *__restrict__ arow,
                                               const int32_t *__restrict__ ext, int rows) {
  const int64_t r0 = (int64_t)blockIdx.y * rows;  // rows divides 256: one panel
  if (ext) k_pad = min(k_pad, (int64_t)ext[r0 / 256] * GRAM_KB);
  const int64_t k0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 8;
  if (k0 >= k_pad) return;
  const int64_t k_len = (int64_t)n_chi * n_m;
  int nq[8];
  {
    int n = (int)(k0 / n_m), m = (int)(k0 % n_m);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      nq[q] = k0 + q < k_len ? n : -1;
      if (++m == n_m) { m = 0; ++n; }
    }
  }
  double g[8];
  int cc = -1;
  for (int rr = 0; rr < rows; ++rr) {
    const int64_t row = r0 + rr;
    const int64_t e = arow ? (int64_t)arow[row] : (row < n_R ? row : -1);  // its distinct row
    double v[8];
    if (e >= 0) {
      const int c = rowR[4 * e];
      if (c != cc) {
        cc = c;
        const double *Gc = G + (size_t)c * k_len + k0;
        if (k0 + 8 <= k_len && (k_len & 1) == 0) {  // 16-byte aligned pairs
#pragma unroll
          for (int q = 0; q < 8; q += 2) {
            const double2 t = *(const double2 *)(Gc + q);
            g[q] = t.x;
            g[q + 1] = t.y;
          }
        } else {
#pragma unroll
          for (int q = 0; q < 8; ++q) g[q] = nq[q] >= 0 ? Gc[q] : 0.0;
        }
      }
      const double *Tr = Ts + (size_t)e * n_chi;
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = nq[q] >= 0 ? Tr[nq[q]] * g[q] : 0.0;
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = 0.0;
    }
    const size_t off = (size_t)row * lda + k0;
    if constexpr (FMT == 0) {
      double *o = (double *)A0 + off;
#pragma unroll
      for (int q = 0; q < 8; q += 2) *(double2 *)(o + q) = make_double2(v[q], v[q + 1]);
    } else if constexpr (FMT == 3) {
      float *o = (float *)A0 + off;
      *(float4 *)o = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
      *(float4 *)(o + 4) = make_float4((float)v[4], (float)v[5], (float)v[6], (float)v[7]);
    }
  }
}

// k-blocked bf16 (fmt 1: hi only; fmt 2: hi and lo; see launch_abuild): a 256-thread
// block covers 64 rows and kb_wg consecutive 32-column k-blocks: AB_KB, or as many
// fewer (four, one pass, at least) as it takes for 512 blocks (512 rows of 4608
// k with lo: 12 us, with 32 k-blocks to each of 40 blocks 30).  Each
// wavefront takes every fourth k-block of the block; in one, lane l converts
// 8 consecutive k (chunk l % 4) of the rows l / 4 + 16 j, j < AB_RW, so that
// each of its stores writes 16 whole rows of the k-block, 1 KB contiguous
// (non-temporal: at large10 1.55 -> 1.3 ms with hi, 2.2 -> 1.6 ms with lo).
// Rows of one configuration are consecutive (in the A-row order of the bf16
// products, those of one lowest redshift bin), so a lane's 8 values of G
// serve all its rows of one configuration, and T is taken once per row and
// chi node.  When N_M is a multiple of 8 a chunk lies in one chi
// node, and T of the workgroup's rows and G of its configurations (at most
// AB_GC of them) are staged in LDS with coalesced loads; otherwise the values
// are taken one by one from global memory.
constexpr int AB_KB = 32;
constexpr int AB_RW = 4;
// chi nodes of T a workgroup stages in LDS: its AB_KB k-blocks span
// AB_KB 32 / N_M + 1 nodes at most (33 for N_M >= 32); more go to global memory
constexpr int AB_TN = 40;
// configurations whose G a workgroup stages in LDS, pass by pass (a pass is
// the four k-blocks the wavefronts convert together): in the A-row order at
// n_z = 10, 64 rows of one lowest bin z span at most eight configurations
// for z <= 6 (10 or more rows each); wider spans take the global path
// (measured at large10: 1.58 ms with 6 or 8, 1.63 with 3, 1.82 with 12)
constexpr int AB_GC = 8;

// Two floats to packed bf16, rounded to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16_rne(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}

// With panel_f (the per-tile precision of WLC_BF16_AUTO: per 256-row panel
// the largest one-halo share, then the largest of all), the lo half of a
// panel is written only if some tile of its row or column can take the split
// product, F_P F_max > lim; the product never reads it otherwise.
template <int FMT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FMT == 1 ? 5 : 4))) void k_abuild_blk(const int32_t *__restrict__ rowR, const double *__restrict__ Ts,
                                                   const double *__restrict__ G, int64_t n_R, int n_chi, int n_m,
                                                   int64_t k_pad, int64_t r_pad, uint16_t *__restrict__ A0,
                                                   uint16_t *__restrict__ A1, const double *__restrict__ panel_f,
                                                   double lim, const int32_t *__restrict__ arow,
                                                   const int32_t *__restrict__ ext, int kb_wg) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int chunk = lane & 3;
  const int64_t row0 = (int64_t)blockIdx.y * 64 + (lane >> 2);  // A-rows row0 + 16 j
  // a workgroup's 64 rows lie in one 256-row panel; with ext the panel's rows
  // are zero from k-block ext[panel] on, and no product reads them there
  const int panel = blockIdx.y / 4;
  const int n_kb =
      (int)min((int64_t)kb_wg, (ext ? (int64_t)ext[panel] : k_pad / GRAM_KB) - (int64_t)blockIdx.x * kb_wg);
  if (n_kb <= 0) return;  // workgroup-uniform, before any barrier
  const bool need_lo = FMT == 2 && (panel_f == nullptr || panel_f[panel] * panel_f[r_pad / 256] > lim);
  const int64_t k_len = (int64_t)n_chi * n_m;
  const bool whole = (n_m & 7) == 0;  // a chunk of 8 k lies in one chi node
  // the distinct row of an A-row (-1 for padding)
  auto distinct = [&](int64_t r) -> int { return arow ? arow[r] : (r < n_R ? (int)r : -1); };
  int cfg[AB_RW];
  const double *Tr[AB_RW];
#pragma unroll
  for (int j = 0; j < AB_RW; ++j) {
    const int e = distinct(row0 + 16 * j);
    cfg[j] = e >= 0 ? rowR[4 * e] : -1;
    Tr[j] = Ts + (size_t)(e >= 0 ? e : 0) * n_chi;
  }
  // T of the workgroup's 64 rows at the chi nodes of its k range, staged in
  // LDS with coalesced loads (a lane would otherwise gather T of its rows
  // from 16 rows n_chi apart at every node change)
  __shared__ double Tl[64][AB_TN + 1];
  __shared__ int c_rng[2];  // smallest and largest configuration of the workgroup's rows
  const int64_t kbeg = (int64_t)blockIdx.x * kb_wg * GRAM_KB;
  const int n_lo = kbeg < k_len ? (int)(kbeg / n_m) : 0;
  const int n_hi = kbeg < k_len ? (int)((min(kbeg + (int64_t)n_kb * GRAM_KB, k_len) - 1) / n_m) : 0;
  const int nodes = n_hi - n_lo + 1;
  const bool staged = whole && kbeg < k_len && nodes <= AB_TN;  // workgroup-uniform
  if (staged) {
    if (threadIdx.x == 0) c_rng[0] = 0x7FFFFFFF, c_rng[1] = -1;
    __syncthreads();
    if (threadIdx.x < 64) {
      const int e = distinct((int64_t)blockIdx.y * 64 + threadIdx.x);
      if (e >= 0) {
        atomicMin(&c_rng[0], rowR[4 * e]);
        atomicMax(&c_rng[1], rowR[4 * e]);
      }
    }
    for (int idx = threadIdx.x; idx < 64 * nodes; idx += 256) {
      const int r = idx / nodes, q = idx % nodes;
      const int e = distinct((int64_t)blockIdx.y * 64 + r);
      Tl[r][q] = e >= 0 ? Ts[(int64_t)e * n_chi + n_lo + q] : 0.0;
    }
    __syncthreads();
  }
  // G of the workgroup's configurations for the four k-blocks of a pass, in
  // two alternating buffers: the barrier after filling one for pass p also
  // ends every wavefront's reads of pass p - 1, whose buffer pass p + 1 fills
  __shared__ double Gl[2][AB_GC][4 * GRAM_KB];
  const int c_first = staged ? c_rng[0] : 0, c_last = staged ? c_rng[1] : -1;
  const bool gstaged = staged && c_last >= c_first && c_last - c_first < AB_GC;  // workgroup-uniform
  int node[AB_RW];
  double tn[AB_RW];
#pragma unroll
  for (int j = 0; j < AB_RW; ++j) node[j] = -1, tn[j] = 0.0;
  for (int pass = 0; pass < (n_kb + 3) / 4; ++pass) {
    const int q = 4 * pass + wave;
    if (gstaged) {
      const int64_t kp = kbeg + (int64_t)pass * 4 * GRAM_KB;
      for (int idx = threadIdx.x; idx < AB_GC * 2 * GRAM_KB; idx += 256) {
        const int ci = idx / (2 * GRAM_KB), e = 2 * (idx % (2 * GRAM_KB));
        const int64_t k = kp + e;  // even, and k_len is a multiple of 8: k + 1 < k_len with k
        double2 v = make_double2(0.0, 0.0);
        if (ci <= c_last - c_first && k < k_len) v = *(const double2 *)(G + (size_t)(c_first + ci) * k_len + k);
        *(double2 *)&Gl[pass & 1][ci][e] = v;
      }
      __syncthreads();
    }
    if (q >= n_kb) continue;  // past the panel's k-blocks (later passes' barriers still to come: no break)
    const int64_t kblk = (int64_t)blockIdx.x * kb_wg + q;
    const int64_t k0 = kblk * GRAM_KB + 8 * chunk;
    const int n = k0 < k_len ? (int)(k0 / n_m) : 0;
    double g[8];
    int gc = -1;
#pragma unroll
    for (int j = 0; j < AB_RW; ++j) {
      const int64_t row = row0 + 16 * j;
      float x[8];
      if (whole && cfg[j] >= 0 && k0 < k_len) {
        if (cfg[j] != gc) {
          if (gstaged) {
            const double *Gs = &Gl[pass & 1][cfg[j] - c_first][wave * GRAM_KB + 8 * chunk];
#pragma unroll
            for (int e = 0; e < 8; ++e) g[e] = Gs[e];
          } else {
            const double *Gc = G + (size_t)cfg[j] * k_len + k0;
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
              const double2 t = *(const double2 *)(Gc + e);
              g[e] = t.x;
              g[e + 1] = t.y;
            }
          }
          gc = cfg[j];
        }
        if (node[j] != n) {
          node[j] = n;
          tn[j] = staged ? Tl[(lane >> 2) + 16 * j][n - n_lo] : Tr[j][n];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = (float)(tn[j] * g[e]);
      } else {
        // one by one, stepping across the chi node edges (k0 = n N_M + m)
        const double *Gc = G + (size_t)(cfg[j] >= 0 ? cfg[j] : 0) * k_len;
        int nn = n, mm = (int)(k0 - (int64_t)n * n_m);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int64_t k = k0 + e;
          x[e] = cfg[j] >= 0 && k < k_len ? (float)(Tr[j][nn] * Gc[k]) : 0.0f;
          if (++mm == n_m) mm = 0, ++nn;
        }
      }
      uint32_t hi[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) hi[e] = pack_bf16_rne(x[2 * e], x[2 * e + 1]);
      const size_t off = ((size_t)kblk * r_pad + row) * GRAM_KB + 8 * chunk;
      __builtin_nontemporal_store(u32x4{hi[0], hi[1], hi[2], hi[3]}, (u32x4 *)(A0 + off));
      if (need_lo) {
        uint32_t lo[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          lo[e] = pack_bf16_rne(x[2 * e] - __uint_as_float(hi[e] << 16),
                                x[2 * e + 1] - __uint_as_float(hi[e] & 0xFFFF0000u));
        __builtin_nontemporal_store(u32x4{lo[0], lo[1], lo[2], lo[3]}, (u32x4 *)(A1 + off));
      }
    }
  }
}

// One workgroup per 256-row panel of A-rows: the panel keeps the largest count
// of k-blocks (the k of node n are n N_M .. n N_M + N_M - 1).
__global__ __launch_bounds__(256) void k_panel_ext(const int32_t *__restrict__ last, const int32_t *__restrict__ arow,
                                                  int n_mg, int64_t k_pad, int32_t *__restrict__ ext,
                                                  double *__restrict__ panel_f) {
  __shared__ int32_t best;
  if (threadIdx.x == 0) best = 0;
  __syncthreads();
  const int e = arow[(int64_t)blockIdx.x * 256 + threadIdx.x];
  const int top = e >= 0 ? last[e] : -1;
  const int64_t kb = min(((int64_t)(top + 1) * n_mg + GRAM_KB - 1) / GRAM_KB, k_pad / GRAM_KB);
  if (kb > 0) atomicMax(&best, (int32_t)kb);
  __syncthreads();
  if (threadIdx.x == 0) {
    ext[blockIdx.x] = best;
    if (panel_f) {
      panel_f[blockIdx.x] = 0.0;
      if (blockIdx.x == 0) panel_f[gridDim.x] = 0.0;
    }
  }
}

void launch_panel_ext(const int32_t *last, const int32_t *arow, int64_t r_pad, int n_mg, int64_t k_pad, int32_t *ext,
                      double *panel_f, hipStream_t s) {
  hipLaunchKernelGGL(k_panel_ext, dim3((unsigned)(r_pad / 256)), dim3(256), 0, s, last, arow, n_mg, k_pad, ext,
                     panel_f);
}

void launch_abuild(int fmt, const int32_t *rowR, const double *Ts, const double *G, int64_t n_R, int64_t r_pad,
                   int n_chi, int n_m, int64_t k_pad, int64_t lda, void *A0, void *A1, hipStream_t s,
                   const double *panel_f, double lim, const int32_t *arow, const int32_t *ext) {
  if (fmt == 1 || fmt == 2) {
    // r_pad is a multiple of 64 and k_pad of GRAM_KB (rows are padded to the
    // Gram tile, columns to 64)
    int kb = AB_KB;
    while (kb > 4 && (k_pad / GRAM_KB + kb - 1) / kb * (r_pad / 64) < 512) kb /= 2;
    const dim3 grid((unsigned)((k_pad / GRAM_KB + kb - 1) / kb), (unsigned)(r_pad / 64));
    if (fmt == 1)
      hipLaunchKernelGGL(k_abuild_blk<1>, grid, dim3(256), 0, s, rowR, Ts, G, n_R, n_chi, n_m, k_pad, r_pad,
                         (uint16_t *)A0, (uint16_t *)A1, nullptr, 0.0, arow, ext, kb);
    else
      hipLaunchKernelGGL(k_abuild_blk<2>, grid, dim3(256), 0, s, rowR, Ts, G, n_R, n_chi, n_m, k_pad, r_pad,
                         (uint16_t *)A0, (uint16_t *)A1, panel_f, lim, arow, ext, kb);
    return;
  }
  // r_pad is a multiple of AB_ROWS (rows are padded to the Gram tile)
  const int64_t gx = (k_pad / 8 + 255) / 256;
  int rows = AB_ROWS;
  while (rows > 1 && gx * (r_pad / rows) < 1024) rows /= 2;
  const dim3 grid((unsigned)gx, (unsigned)(r_pad / rows));
  if (fmt == 0)
    hipLaunchKernelGGL(k_abuild<0>, grid, dim3(256), 0, s, rowR, Ts, G, n_R, n_chi, n_m, k_pad, lda, A0, A1, arow, ext,
                       rows);
  else
    hipLaunchKernelGGL(k_abuild<3>, grid, dim3(256), 0, s, rowR, Ts, G, n_R, n_chi, n_m, k_pad, lda, A0, A1, arow, ext,
                       rows);
}

}  // namespace wlc
