// Assembly of the joint P+B covariance (Rizzato et al. 2019, eq. eq:SN2):
//   C = C_Gauss + E (G / Omega) E^T + sigma_b^2 r r^T,
// with E the map from data-vector rows to distinct rows, G the Gram product of
// the one-halo factor, and the Gaussian blocks
//   P-P: delta_{l l'} / N(l) [P^s_ii' P^s_jj' + P^s_ij' P^s_ji']       (eq. CovPPG)
//   B-B: Omega / N_tri sum over the 6 maps sigma of primed onto unprimed legs of
//        prod_a P^s_{i_a i'_sigma(a)}(l_a) delta_K(l_a, l'_sigma(a))     (App. B, Gauss term)
//   P-B: none                                                          (eq. CovPBsynt)
// The result is written scaled, C~[a][b] = 2^(t_a + t_b) C[a][b], with t
// chosen so that every C~[a][a] lies in [1, 4).  Each unordered pair (a, b)
// is evaluated once and written to both halves, so C~ is exactly symmetric.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"

namespace wlc {

__device__ __forceinline__ double gauss_entry(const AsmArgs &A, const int32_t *ra, const int32_t *rb) {
  if (ra[0] != rb[0]) return 0.0;  // different ell-configuration
  const int nz = A.n_z;
  const double *Ps = A.Ps;
  const int kind = A.cfgT[4 * ra[0]];
  if (kind == 2) {
    const int b = ra[5];
    const double *P = Ps + (size_t)b * nz * nz;
    return (P[ra[2] * nz + rb[2]] * P[ra[3] * nz + rb[3]] + P[ra[2] * nz + rb[3]] * P[ra[3] * nz + rb[2]]) /
           A.nmodes[b];
  }
  // M[a][b] = P^s of leg a and primed leg b where their ell-bins agree (else 0),
  // all nine loads at once; the six maps are the terms of its permanent
  double M[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const double v = Ps[((size_t)ra[5 + a] * nz + ra[2 + a]) * nz + rb[2 + b]];
      M[a][b] = ra[5 + a] == rb[5 + b] ? v : 0.0;
    }
  const double s = M[0][0] * M[1][1] * M[2][2] + M[0][0] * M[1][2] * M[2][1] + M[0][1] * M[1][0] * M[2][2] +
                   M[0][1] * M[1][2] * M[2][0] + M[0][2] * M[1][0] * M[2][1] + M[0][2] * M[1][1] * M[2][0];
  return A.omega / A.ntri[ra[0] - A.n_ell] * s;
}

// ---- in-survey terms beyond the one-halo functions (eqs. CovBB, Covpb)
// Index of the distinct row of a bin multiset: pairs i <= j and triples
// i <= j <= k are ranked in the plan's order (first index slowest).
__device__ __forceinline__ int pair_rank(int i, int j, int nz) {
  if (i > j) { const int t = i; i = j; j = t; }
  return i * nz - i * (i - 1) / 2 + (j - i);
}

__device__ __forceinline__ int trip_rank(int a, int b, int c, int nz) {
  // sort three values
  if (a > b) { const int t = a; a = b; b = t; }
  if (b > c) { const int t = b; b = c; c = t; }
  if (a > b) { const int t = a; a = b; b = t; }
  int r = 0;
  for (int x = 0; x < a; ++x) r += (nz - x) * (nz - x + 1) / 2;
  for (int y = a; y < b; ++y) r += nz - y;
  return r + (c - b);
}

// Row of the two-leg trispectrum for legs p <= q (ell-bins) carrying bins
// (j on p, k on q).
__device__ __forceinline__ int64_t twoleg_row(int p, int q, int j, int k, int nl, int nz) {
  const int sp = nz * (nz + 1) / 2;
  if (p == q) return (int64_t)p * sp + pair_rank(j, k, nz);
  const int r = p * (nl - 1) - p * (p - 1) / 2 + (q - p - 1);
  return (int64_t)nl * sp + (int64_t)r * nz * nz + j * nz + k;
}

__device__ __forceinline__ double ngins_entry(const AsmArgs &A, const int32_t *ra, const int32_t *rb) {
  const int nz = A.n_z, nl = A.n_ell;
  const int kind_a = A.cfgT[4 * ra[0]], kind_b = A.cfgT[4 * rb[0]];
  if (kind_a == 2 && kind_b == 2) return 0.0;
  const int sp = nz * (nz + 1) / 2, st = nz * (nz + 1) * (nz + 2) / 6;
  const int64_t np = (int64_t)nl * sp;  // first distinct bispectrum row
  const double *Ps = A.Ps;
  auto ps = [&](int b, int i, int j) { return Ps[((size_t)b * nz + i) * nz + j]; };
  auto bval = [&](int cfg, int z0, int z1, int z2) {
    return A.dR[np + (int64_t)(cfg - nl) * st + trip_rank(z0, z1, z2, nz)];
  };
  if (kind_a == 2 || kind_b == 2) {
    const int32_t *rp = kind_a == 2 ? ra : rb, *rt = kind_a == 2 ? rb : ra;
    const int l = rp[5], i = rp[2], j = rp[3];
    double s = 0.0;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      if (rt[5 + b] != l) continue;
      int zi[3] = {rt[2], rt[3], rt[4]}, zj[3] = {rt[2], rt[3], rt[4]};
      zi[b] = i;
      zj[b] = j;
      s += (ps(l, rt[2 + b], j) * bval(rt[0], zi[0], zi[1], zi[2]) +
            ps(l, i, rt[2 + b]) * bval(rt[0], zj[0], zj[1], zj[2])) / A.nmodes[l];
    }
    return s;
  }
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const int l = ra[5 + a];
      if (l != rb[5 + b]) continue;
      int z1[3] = {ra[2], ra[3], ra[4]}, z2[3] = {rb[2], rb[3], rb[4]};
      z1[a] = rb[2 + b];
      z2[b] = ra[2 + a];
      const double bb = bval(ra[0], z1[0], z1[1], z1[2]) * bval(rb[0], z2[0], z2[1], z2[2]);
      // the two other legs of each row, in leg order (ell-bins non-decreasing)
      const int ax = a == 0 ? 1 : 0, ay = a == 2 ? 1 : 2, bx = b == 0 ? 1 : 0, by = b == 2 ? 1 : 2;
      const int64_t ta = twoleg_row(ra[5 + ax], ra[5 + ay], ra[2 + ax], ra[2 + ay], nl, nz);
      const int64_t tb = twoleg_row(rb[5 + bx], rb[5 + by], rb[2 + bx], rb[2 + by], nl, nz);
      const double t4 = ta >= tb ? A.T2[ta * A.ld_t2 + tb] : A.T2[tb * A.ld_t2 + ta];
      s += (bb + ps(l, ra[2 + a], rb[2 + b]) * t4) / A.nmodes[l];
    }
  return s;
}

// G has been mirrored to exact symmetry, so it is read along rows: for the
// 64 consecutive data rows b of a wavefront the distinct rows e(b) are
// clustered, and the reads touch few cache lines.
__device__ __forceinline__ double gram_at(const AsmArgs &A, int64_t ea, int64_t eb) {
  return A.gm_f32 ? (double)((const float *)A.Gm)[ea * A.ld_g + eb] : ((const double *)A.Gm)[ea * A.ld_g + eb];
}

// Diagonal first: row exponents t_a, and the expanded d, r.
__global__ void k_rowexp(AsmArgs A, int32_t *row_exp2, double *d, double *r) {
  const int64_t a = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (a >= A.n) return;
  const int32_t *ra = A.rowO + 8 * a;
  const int64_t e = ra[1];
  const double g = gram_at(A, e, e);
  const double rr = A.rR[e];
  double c = ldexp(g, -2 * A.sexp[e]) * A.inv_omega + gauss_entry(A, ra, ra) + A.sigma_b2 * rr * rr;
  if (A.ngins) c += ngins_entry(A, ra, ra);
  int t = 0;
  if (c > 0.0 && isfinite(c)) {
    const int E = exp2_of(c);
    const int q = E - 1;
    t = -(q >= 0 ? q / 2 : -((1 - q) / 2));  // -floor((E - 1) / 2)
  }
  row_exp2[a] = t;
  d[a] = A.dR[e];
  r[a] = rr;
}

void launch_rowexp(const AsmArgs &a, int32_t *row_exp2, double *d, double *r, hipStream_t s) {
  hipLaunchKernelGGL(k_rowexp, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, s, a, row_exp2, d, r);
}

// ---- per-tile precision of the bf16 Gram (WLC_BF16_AUTO)
// The one-halo diagonal of distinct row e in FP64 from its factors,
//   G_ee = sum_n Ts[e][n]^2 S[c(e)][n],  S[c][n] = sum_m G[c][n][m]^2
// (the row of A is Ts[e][n] G[c][n][m] over k = (n, m)), then for every data
// row a the share f_a = C1h_aa / C_aa, C_aa = C1h_aa + Gaussian + super-sample
// as in k_rowexp, and per panel of 256 distinct rows the largest f_a.  G_ee
// (gd) comes with the rows' factors.
constexpr int SPLIT_PANEL = 256;  // rows per panel: the bf16 Gram tile

// A workgroup's largest shares are found in LDS first (best [n_panels], 8 bytes
// for each 256 rows of the product): 4550 rows 5 us, with every lane's atomic on
// a handful of global addresses 27.
__global__ void k_split_share(AsmArgs A, const double *__restrict__ gd, double *F, const int32_t *__restrict__ pos,
                              int n_panels) {
  extern __shared__ unsigned long long best[];
  for (int i = threadIdx.x; i < n_panels; i += blockDim.x) best[i] = 0;
  __syncthreads();
  const int64_t a = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  unsigned long long *Fb = (unsigned long long *)F;
  double f = 0.0;
  if (a < A.n) {
    const int32_t *ra = A.rowO + 8 * a;
    const int64_t e = ra[1];
    const double c1h = ldexp(gd[e], -2 * A.sexp[e]) * A.inv_omega;
    const double rr = A.rR[e];
    const double c = c1h + gauss_entry(A, ra, ra) + A.sigma_b2 * rr * rr;
    // a share of 1 (no other term) for a row whose diagonal is not positive
    f = c > 0.0 && isfinite(c) ? c1h / c : 1.0;
    // non-negative doubles order like their bit patterns; the panel of the row's A-row
    atomicMax(&best[(pos ? pos[e] : e) / SPLIT_PANEL], (unsigned long long)__double_as_longlong(f));
  }
  f = wave_max(f);
  if ((threadIdx.x & (WAVE - 1)) == 0)
    atomicMax(&Fb[A.ld_g / SPLIT_PANEL], (unsigned long long)__double_as_longlong(f));
  __syncthreads();
  for (int i = threadIdx.x; i < n_panels; i += blockDim.x)
    if (best[i]) atomicMax(&Fb[i], best[i]);
}

void launch_split_share(const AsmArgs &a, const double *gd, double *F, const int32_t *pos, hipStream_t s) {
  const int n = (int)(a.ld_g / SPLIT_PANEL);
  hipLaunchKernelGGL(k_split_share, dim3((unsigned)((a.n + 255) / 256)), dim3(256), (size_t)n * 8, s, a, gd, F, pos, n);
}

// 64 x 64 output tiles (I >= J); each thread computes 16 entries of one
// column, the transposed copy goes through LDS so both halves are written
// with contiguous rows.  Tiles are numbered row-major over the triangle and
// each XCD (workgroup b runs on XCD b mod 8, each XCD has its own L2) takes
// a contiguous run of them, so the one-halo rows of a tile row are fetched
// into one L2 instead of all eight.  A tile's loads form two rounds: the
// row records and output exponents, then (all depending only on the
// records) the one-halo values and the distinct rows' exponents and
// responses, so a workgroup waits on global memory twice before it writes.
constexpr int AT = 64;
constexpr int ASM_XCD = 8;
// Up to here four entries per thread: a workgroup is a chain of loads, and the
// few of a small matrix are over sooner (818 rows 24.5 us for the phase
// against 34.6 with sixteen, 3750 rows 54 and 56, 7625 rows 146 and 107)
constexpr int64_t ASM_WIDE = 4000;

// Q entries for each thread (4096 / Q threads).
template <typename OutT, int Q>
__global__ __launch_bounds__(AT * AT / Q) void k_assemble(AsmArgs A, const int32_t *__restrict__ row_exp2,
                                                  OutT *__restrict__ C, int64_t n_tiles) {
  __shared__ OutT tileT[AT][AT + 1];
  __shared__ int32_t rowA[AT][8], rowB[AT][8];
  __shared__ int32_t tA[AT], tB[AT], sA[AT], sB[AT];
  __shared__ double rA[AT], rB[AT];
  const int64_t per = (int64_t)gridDim.x / ASM_XCD;
  const int64_t t = (int64_t)(blockIdx.x % ASM_XCD) * per + blockIdx.x / ASM_XCD;
  if (t >= n_tiles) return;  // grid padding (whole workgroup)
  int64_t i = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  while ((i + 1) * (i + 2) / 2 <= t) ++i;
  while (i * (i + 1) / 2 > t) --i;
  const int64_t I = i, J = t - i * (i + 1) / 2;
  const int64_t a0 = I * AT, b0 = J * AT;
  const int tid = threadIdx.x;
  for (int q = tid; q < AT * 8; q += AT * AT / Q) {
    const int r = q / 8, c = q % 8;
    rowA[r][c] = a0 + r < A.n ? A.rowO[(a0 + r) * 8 + c] : 0;
    rowB[r][c] = b0 + r < A.n ? A.rowO[(b0 + r) * 8 + c] : 0;
  }
  if (tid < AT) {
    tA[tid] = a0 + tid < A.n ? row_exp2[a0 + tid] : 0;
  } else if (tid < 2 * AT) {
    tB[tid - AT] = b0 + tid - AT < A.n ? row_exp2[b0 + tid - AT] : 0;
  }
  __syncthreads();
  const int cb = tid & 63;          // column within the tile
  const int rbase = (tid >> 6) * Q;
  const int64_t b = b0 + cb;
  // the Q one-halo values, all loads in flight together with those of the
  // exponents and responses (padding rows map to distinct row 0, so every
  // index is valid)
  // (the one-halo block has the output's type: FP32 for the mixed modes)
  OutT gv[Q];
  const int64_t eb = rowB[cb][1];
  const OutT *G = (const OutT *)A.Gm;
#pragma unroll
  for (int q = 0; q < Q; ++q) gv[q] = G[rowA[rbase + q][1] * A.ld_g + eb];
  if (tid < AT) {
    const bool live = a0 + tid < A.n;
    sA[tid] = live ? A.sexp[rowA[tid][1]] : 0;
    rA[tid] = live ? A.rR[rowA[tid][1]] : 0.0;
  } else if (tid < 2 * AT) {
    const int q = tid - AT;
    const bool live = b0 + q < A.n;
    sB[q] = live ? A.sexp[rowB[q][1]] : 0;
    rB[q] = live ? A.rR[rowB[q][1]] : 0.0;
  }
  __syncthreads();
#pragma unroll 4
  for (int q = 0; q < Q; ++q) {
    const int ra = rbase + q;
    const int64_t a = a0 + ra;
    OutT v = 0;
    const bool live = a < A.n && b < A.n && a >= b;
    if (live) {
      const int tt = tA[ra] + tB[cb];
      const double g = (double)gv[q];
      double rest = A.sigma_b2 * rA[ra] * rB[cb] + gauss_entry(A, rowA[ra], rowB[cb]);
      if (A.ngins) rest += ngins_entry(A, rowA[ra], rowB[cb]);
      v = (OutT)(ldexp(g * A.inv_omega, tt - sA[ra] - sB[cb]) + ldexp(rest, tt));
      C[a * A.n + b] = v;
    }
    tileT[ra][cb] = v;
  }
  __syncthreads();
  // transposed half: C[b][a] for the same pairs, rows of the output contiguous,
  // with non-temporal stores (measured 1 ms faster at N = 82575; both halves
  // non-temporal was 2 ms slower)
#pragma unroll 4
  for (int q = 0; q < Q; ++q) {
    const int rb = rbase + q;  // row of the transposed tile (b index)
    const int ca = cb;         // column (a index)
    const int64_t bb = b0 + rb, aa = a0 + ca;
    if (aa < A.n && bb < A.n && aa > bb) __builtin_nontemporal_store(tileT[ca][rb], &C[bb * A.n + aa]);
  }
}

void launch_assemble(const AsmArgs &a, const int32_t *row_exp2, void *C, hipStream_t s) {
  const int64_t nt = (a.n + AT - 1) / AT;
  const int64_t tiles = nt * (nt + 1) / 2;
  const dim3 grid((unsigned)((tiles + ASM_XCD - 1) / ASM_XCD * ASM_XCD));
  auto run = [&](auto out, auto wide) {
    using T = decltype(out);
    constexpr int Q = decltype(wide)::value ? 4 : 16;
    hipLaunchKernelGGL((k_assemble<T, Q>), grid, dim3(AT * AT / Q), 0, s, a, row_exp2, (T *)C, tiles);
  };
  const bool wide = a.n <= ASM_WIDE;
  if (a.gm_f32)
    wide ? run(0.0f, std::true_type{}) : run(0.0f, std::false_type{});
  else
    wide ? run(0.0, std::true_type{}) : run(0.0, std::false_type{});
}

}  // namespace wlc
