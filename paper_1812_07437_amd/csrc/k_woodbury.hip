// Signal-to-noise (eq. SNprim) through the distinct rows.
//
// The joint covariance is C = C_G + E M E^T: C_G the Gaussian term, zero
// between different ell-configurations (eqs. CovPPG, CovPBsynt and the
// Gaussian term of App. B); E the map from data-vector rows to distinct rows
// (the Limber kernels are symmetric in the bins, so the one-halo term, the
// response and d itself depend only on the multiset of bins); and
// M = C_1h + sigma_b^2 r r^T on the distinct rows.  Since d = E d_R,
//   (S/N)^2 = d_R^T (G^-1 + M)^-1 d_R = u^T (I + Z)^-1 u,
//   G = E^T C_G^-1 E = L L^T,  u = L^T d_R,  Z = L^T M L,
// an identity with no cancellation; the one large factorisation is that of
// I + Z (N_R rows instead of N), done by the bordered Cholesky.
//
// G is block-diagonal over configurations and each block has a closed form
// in Q_b = (P^s_b)^-1.  On the data-vector rows of one configuration the
// Gaussian block is
//   P rows (pairs i <= j):        S2(P_b) / N(l_b)
//   scalene triangle:             (Omega / N_tri) P_1 (x) P_2 (x) P_3
//   l1 = l2 < l3 (rows i <= j, k): (Omega / N_tri) S2(P_1) (x) P_3
//   l1 < l2 = l3 (rows i, j <= k): (Omega / N_tri) P_1 (x) S2(P_2)
//   equilateral (rows i <= j <= k): (Omega / N_tri) S3(P_b)
// with S2(P)[(ij)(kl)] = P_ik P_jl + P_il P_jk and S3(P) the sum over the six
// leg permutations.  These products are symmetric under the permutations of
// equal legs, and on the symmetric subspace their inverses are
//   S2(P)^-1 = (nu nu^T / 4) o S2(Q),  S3(P)^-1 = (mu mu^T / 36) o S3(Q),
// nu and mu counting the distinct orderings of the bins.  G then sums the
// inverse over the rows that share a multiset of bins.
//
// Rows are scaled by powers of two throughout (G by D = diag(2^tau) so that
// its diagonal lies in [1, 4), M by D^-1), so that every factor stays near
// unit size; the scaling is exact.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace wlc {

// ------------------------------------------------------------------ Q
constexpr int QMAX = WOOD_NZ_MAX;

// Q_b = (P^s_b)^-1 for every ell-bin (n_z <= QMAX), one wavefront each, lane i
// with row i of the Cholesky factor and column i of its inverse, in LDS (ten bins
// 5 us; one thread for each ell-bin, its matrix in scratch memory, 20).
__global__ __launch_bounds__(WAVE) void k_qinv(const double *__restrict__ Ps, int nz, double *__restrict__ Q,
                                               int *__restrict__ flag) {
  __shared__ double L[QMAX][QMAX + 1], X[QMAX][QMAX + 1];
  const int b = blockIdx.x, i = threadIdx.x;
  const double *P = Ps + (size_t)b * nz * nz;
  for (int e = i; e < nz * nz; e += WAVE) L[e / nz][e % nz] = P[e];
  __syncthreads();
  bool bad = false;
  for (int k = 0; k < nz; ++k) {
    double v = L[k][k];
    if (!(v > 0.0)) {
      bad = true;
      v = 1.0;
    }
    const double d = sqrt(v);
    const double l = i > k && i < nz ? L[i][k] / d : 0.0;
    __syncthreads();
    if (i == k) L[k][k] = d;
    if (i > k && i < nz) L[i][k] = l;
    __syncthreads();
    if (i > k && i < nz)
      for (int j = k + 1; j <= i; ++j) L[i][j] -= l * L[j][k];
    __syncthreads();
  }
  if (i < nz) {  // column i of X = L^-1
    X[i][i] = 1.0 / L[i][i];
    for (int r = i + 1; r < nz; ++r) {
      double t = 0.0;
      for (int k = i; k < r; ++k) t -= L[r][k] * X[k][i];
      X[r][i] = t / L[r][r];
    }
  }
  __syncthreads();
  // Q = X^T X
  for (int e = i; e < nz * nz; e += WAVE) {
    const int r = e / nz, c = e % nz;
    double t = 0.0;
    for (int k = max(r, c); k < nz; ++k) t += X[k][r] * X[k][c];
    Q[(size_t)b * nz * nz + e] = t;
  }
  if (bad && i == 0) atomicOr(flag, 1);
}

// ------------------------------------------------------------------ G
__device__ __forceinline__ void decode_pair(int m, int nz, int &i, int &j) {
  for (i = 0; i < nz; ++i) {
    const int cnt = nz - i;
    if (m < cnt) {
      j = i + m;
      return;
    }
    m -= cnt;
  }
}

__device__ __forceinline__ void decode_trip(int m, int nz, int &i, int &j, int &k) {
  for (i = 0; i < nz; ++i)
    for (j = i; j < nz; ++j) {
      const int cnt = nz - j;
      if (m < cnt) {
        k = j + m;
        return;
      }
      m -= cnt;
    }
}

struct Qv {
  const double *Q;
  int nz;
  __device__ double operator()(int b, int x, int y) const { return Q[((size_t)b * nz + x) * nz + y]; }
};

__device__ __forceinline__ double s2(const Qv &q, int b, int i, int j, int k, int l) {
  return q(b, i, k) * q(b, j, l) + q(b, i, l) * q(b, j, k);
}

// number of distinct orderings of a sorted triple
__device__ __forceinline__ int orderings(const int m[3]) {
  return m[0] == m[2] ? 1 : m[0] == m[1] || m[1] == m[2] ? 3 : 6;
}

// On a triangle's rows the entry of G is
//   sum over the distinct orderings a of m and b of m' of Q_1(a_1, b_1) Q_2(a_2, b_2) Q_3(a_3, b_3),
// halved for two equal legs and a sixth of it for three: a row of an (i <= j, k) or
// (i <= j <= k) block stands for nu or mu orderings, and in the sum over all of
// them the two terms of S2 (the six of S3) are the same.  The orderings are taken
// as all 36 pairs of permutations, n n' / 36 of their sum, from 27 values that
// are loaded together (64 triangles of 35 rows 7 us; the distinct orderings, listed in
// scratch memory, 37).
__global__ void k_gblock(BlockMap B, const int32_t *__restrict__ cfgT, Qv q, const double *__restrict__ nmodes,
                         const double *__restrict__ ntri, double omega, double *__restrict__ Gb) {
  const int c = blockIdx.y;
  const int s = B.size(c);
  const int nz = q.nz;
  double *G = Gb + B.off(c);
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < (int64_t)s * s;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int mi = (int)(e / s), mj = (int)(e % s);
    if (mj > mi) continue;
    double v = 0.0;
    if (c < B.nl) {
      int i, j, k, l;
      decode_pair(mi, nz, i, j);
      decode_pair(mj, nz, k, l);
      const double nu = (i == j ? 1.0 : 2.0) * (k == l ? 1.0 : 2.0);
      v = nmodes[c] * nu * 0.25 * s2(q, c, i, j, k, l);
    } else {
      const int l1 = cfgT[4 * c + 1], l2 = cfgT[4 * c + 2], l3 = cfgT[4 * c + 3];
      int m[3], mp[3];
      decode_trip(mi, nz, m[0], m[1], m[2]);
      decode_trip(mj, nz, mp[0], mp[1], mp[2]);
      double a[3][3], b[3][3], d[3][3];
#pragma unroll
      for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int y = 0; y < 3; ++y) {
          a[x][y] = q(l1, m[x], mp[y]);
          b[x][y] = q(l2, m[x], mp[y]);
          d[x][y] = q(l3, m[x], mp[y]);
        }
#pragma unroll
      for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int y = 0; y < 3; ++y) {
          const int x1 = (x + 1) % 3, x2 = (x + 2) % 3, y1 = (y + 1) % 3, y2 = (y + 2) % 3;
          v += a[x][y] * (b[x1][y1] * d[x2][y2] + b[x1][y2] * d[x2][y1] + b[x2][y1] * d[x1][y2] + b[x2][y2] * d[x1][y1]);
        }
      v *= (double)(orderings(m) * orderings(mp)) / (l1 == l3 ? 216.0 : l1 == l2 || l2 == l3 ? 72.0 : 36.0);
      v *= ntri[c - B.nl] / omega;
    }
    G[(int64_t)mi * s + mj] = v;
  }
}

// ------------------------------------------------------------------ blocks
// Per block (one workgroup): row scales tau with G_ee 2^(2 tau) in [1, 4),
// the scaled block factored in place (lower), u = L^T D^-1 d_R into the
// border row, and r scaled by D^-1.
//
// LDS: the block lies in LDS (up to GCHOL_MAX rows), else it stays in global
// memory.  Bound by the chain of its columns, one barrier each: column k is
// scaled while column k + 1 is eliminated with, and an elimination divides by the
// pivot instead (blocks of 35 rows 27 us, of 84 115; in global memory with three
// barriers 42 and 320).
constexpr int GCHOL_MAX = 138;  // of 160 KB 138 rows take 138 139 8 bytes; eight bins have 120 rows, nine 165

template <bool LDS>
__global__ __launch_bounds__(256) void k_gchol(BlockMap B, double *__restrict__ Gb, const double *__restrict__ dR,
                                               const double *__restrict__ rR, int32_t *__restrict__ tau,
                                               double *__restrict__ rhat, double *__restrict__ urow,
                                               int *__restrict__ flag) {
  extern __shared__ double lds[];
  const int c = blockIdx.x;
  const int s = B.size(c);
  const int64_t b0 = B.start(c);
  double *G = Gb + B.off(c), *A = LDS ? lds : G;
  const int ld = LDS ? s | 1 : s;
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  for (int e = tid; e < s; e += 256) {
    const double g = G[(int64_t)e * s + e];
    int t = 0;
    if (g > 0.0 && isfinite(g)) {
      const int q = exp2_of(g) - 1;
      t = -(q >= 0 ? q / 2 : -((1 - q) / 2));  // -floor((E - 1) / 2)
    }
    tau[b0 + e] = t;
    rhat[b0 + e] = ldexp(rR[b0 + e], -t);
  }
  __syncthreads();
  for (int i = ty; i < s; i += 16)
    for (int j = tx; j <= i; j += 16)
      A[(int64_t)i * ld + j] = ldexp(G[(int64_t)i * s + j], tau[b0 + i] + tau[b0 + j]);
  __syncthreads();
  bool bad = false;
  double rp = 1.0;  // of the column before
  for (int k = 0; k < s; ++k) {
    double v = A[(int64_t)k * ld + k];
    if (!(v > 0.0)) {
      bad = true;
      v = 1.0;
    }
    const double rv = 1.0 / v;
    // column k - 1, no longer needed as it was
    if (k > 0)
      for (int i = k + tid; i < s; i += 256) A[(int64_t)i * ld + k - 1] *= rp;
    for (int i = k + 1 + ty; i < s; i += 16) {
      const double f = A[(int64_t)i * ld + k] * rv;
      for (int j = k + 1 + tx; j <= i; j += 16) A[(int64_t)i * ld + j] -= f * A[(int64_t)j * ld + k];
    }
    rp = 1.0 / sqrt(v);
    __syncthreads();
    if (tid == 0) A[(int64_t)k * ld + k] = sqrt(v);  // read by no later step
  }
  __syncthreads();
  if (LDS)
    for (int i = ty; i < s; i += 16)
      for (int j = tx; j <= i; j += 16) G[(int64_t)i * s + j] = A[(int64_t)i * ld + j];
  for (int e = tid; e < s; e += 256) {
    double u = 0.0;
    for (int f = e; f < s; ++f) u += A[(int64_t)f * ld + e] * ldexp(dR[b0 + f], -tau[b0 + f]);
    urow[b0 + e] = u;
  }
  if (tid == 0 && bad) atomicOr(flag, 1);
}

// ------------------------------------------------------------------ products
// MODE 0:  T[e][g] = sum_{h in block(e), h >= e} L[h][e] Mhat[g][h]   (tiles with
//          columns up to the end of the last block of their rows: no entry of W
//          takes more)
// MODE 1:  W[e][f] = delta_ef + sum_{g in block(f), g >= f} T[e][g] L[g][f]   (e >= f)
// with Mhat[g][h] = 2^-(s_g + s_h + tau_g + tau_h) Gm[g][h] / Omega
//                  + sigma_b^2 rhat_g rhat_h,
// Gm the mirrored (symmetric) Gram output.  64 x 64 tiles on
// v_mfma_f64_16x16x4 (four wavefronts of 32 x 32); the contraction runs over
// the configuration blocks that the tile's rows (MODE 0) or columns (MODE 1)
// touch, in LDS stages of 16.
//
// Bound by the loads of a stage: 2390 rows 43 + 24 us, 12768 rows 1.24 + 0.76 ms
// (with every tile of T, and each stage's loads waited for before the products
// of the one before, 60 + 25 us and 2.06 + 0.78 ms).
struct WbArgs {
  BlockMap B;
  const double *Gb;        // factored blocks
  const void *Gm;          // symmetric Gram, f32 or f64, pitch ld_g
  int gm_f32;
  int64_t ld_g;
  const int32_t *sexp;     // Gram row exponents
  const int32_t *tau;
  const double *rhat;
  double inv_omega, sigma_b2;
  double *T;               // [n_R][ld_t]
  int64_t ld_t;
  double *W;               // [n_R + 1][ld_w]
  int64_t ld_w;
};

constexpr int WK = 16;
constexpr int WLD = WK + 1;

template <int MODE>
__global__ __launch_bounds__(256) void k_wb_prod(WbArgs a) {
  __shared__ double lds[2][64 * WLD];
  const int64_t nR = a.B.n_R;
  const int64_t nt = (nR + 63) / 64;
  int64_t ti, tj;
  if (MODE == 0) {
    ti = blockIdx.x / nt;
    tj = blockIdx.x % nt;
  } else {
    const int64_t t = blockIdx.x;
    int64_t i = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    while (i * (i + 1) / 2 > t) --i;
    ti = i;
    tj = t - i * (i + 1) / 2;
  }
  const int64_t e0 = ti * 64, f0 = tj * 64;
  if (MODE == 0) {  // past the blocks of the tile's rows: no W takes it
    const int cl = a.B.blk(min(nR, e0 + 64) - 1);
    if (f0 >= a.B.start(cl) + a.B.size(cl)) return;
  }
  // contraction range: the blocks spanned by the rows (MODE 0) or columns (MODE 1)
  const int64_t s0 = MODE == 0 ? e0 : f0;
  const int64_t s1 = min(nR, s0 + 64) - 1;
  const int cb0 = a.B.blk(s0), cb1 = a.B.blk(s1);
  const int64_t k0 = a.B.start(cb0), k1 = a.B.start(cb1) + a.B.size(cb1);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  f64x4 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
  // Per loaded element j of this thread: its row r = q / WK of the tile is
  // fixed, so the block facts of the L row (e in MODE 0, f in MODE 1) and
  // the scale of the Mhat row f (MODE 0) are taken once here, and the k
  // loop does no index division.
  int64_t lb0[4], lb1[4], lbase[4];  // block [lb0, lb1) holding the L row, Gb index of L[lb0][row]
  int lsz[4];
  double fscale[4], frh[4];          // MODE 0: 2^-(s_f + tau_f) / Omega and sigma_b^2 rhat_f
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = (tid + 256 * j) / WK;
    const int64_t lr = (MODE == 0 ? e0 : f0) + r;  // the row whose L column is read
    lb0[j] = lb1[j] = lbase[j] = 0;
    lsz[j] = 0;
    if (lr < nR) {
      const int c = a.B.blk(lr);
      lb0[j] = a.B.start(c);
      lsz[j] = a.B.size(c);
      lb1[j] = lb0[j] + lsz[j];
      lbase[j] = a.B.off(c) + (lr - lb0[j]);
    }
    fscale[j] = frh[j] = 0.0;
    if (MODE == 0 && f0 + r < nR) {
      const int64_t f = f0 + r;
      fscale[j] = ldexp(a.inv_omega, -(a.sexp[f] + a.tau[f]));
      frh[j] = a.sigma_b2 * a.rhat[f];
    }
  }
  double lw[4], gw[4], rk = 0.0;
  float gf[4];
  int sk = 0;
  auto gload = [&](int64_t kq) {
    // every element of this thread sits in column k = kq + tid % WK of the
    // stage, so the column's Mhat factors are loaded once.  All loads are
    // unconditional, from indices clamped into range, and masked by
    // multiplication when they are put into LDS (the values are finite), so they are in
    // flight together, under the products of the stage before.
    const int64_t k = kq + tid % WK;
    const int64_t kc = k < k1 ? k : k1 - 1;
    if (MODE == 0) {
      sk = a.sexp[kc] + a.tau[kc];
      rk = a.rhat[kc];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t lr = (MODE == 0 ? e0 : f0) + (tid + 256 * j) / WK;
      // L[k][lr]: nonzero only inside lr's block, on or below its diagonal;
      // elsewhere the block's diagonal entry L[lr][lr] is read instead
      const bool lin = k >= lr && k < lb1[j];
      lw[j] = a.Gb[lbase[j] + ((lin ? k : lr) - lb0[j]) * lsz[j]];
    }
    if (MODE == 0) {
      if (a.gm_f32) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          gf[j] = ((const float *)a.Gm)[min(f0 + (tid + 256 * j) / WK, nR - 1) * a.ld_g + kc];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) gw[j] = ((const double *)a.Gm)[min(f0 + (tid + 256 * j) / WK, nR - 1) * a.ld_g + kc];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) gw[j] = a.T[min(e0 + (tid + 256 * j) / WK, nR - 1) * a.ld_t + kc];
    }
  };
  auto lstore = [&](int64_t kq) {
    const int64_t k = kq + tid % WK;
    const bool kin = k < k1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int q = tid + 256 * j, r = q / WK;
      const int64_t e = e0 + r, f = f0 + r;
      const int64_t lr = MODE == 0 ? e : f;
      const double lv = lw[j] * ((k >= lr && k < lb1[j] && kin) ? 1.0 : 0.0);
      double pa, pb;
      if (MODE == 0) {
        const double g = a.gm_f32 ? (double)gf[j] : gw[j];
        pa = lv;
        pb = (ldexp(g * fscale[j], -sk) + frh[j] * rk) * ((f < nR && kin) ? 1.0 : 0.0);
      } else {
        pa = gw[j] * ((e < nR && kin) ? 1.0 : 0.0);
        pb = lv;
      }
      lds[0][r * WLD + q % WK] = pa;
      lds[1][r * WLD + q % WK] = pb;
    }
  };
  gload(k0);
  for (int64_t kq = k0; kq < k1; kq += WK) {
    __syncthreads();
    lstore(kq);
    __syncthreads();
    if (kq + WK < k1) gload(kq + WK);
#pragma unroll
    for (int kk = 0; kk < WK; kk += 4) {
      const int kc = kk + (lane >> 4);
      double av[2], bv[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        av[x] = lds[0][(wr + x * 16 + (lane & 15)) * WLD + kc];
        bv[x] = lds[1][(wc + x * 16 + (lane & 15)) * WLD + kc];
      }
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x], bv[y], acc[x][y], 0, 0, 0);
    }
  }
  // accumulator value v of lane l: row l / 16 + 4 v, column l % 16; W goes
  // out non-temporal (fewer dirty lines under the kernels after it)
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t e = e0 + wr + x * 16 + (lane >> 4) + 4 * v;
        const int64_t f = f0 + wc + y * 16 + (lane & 15);
        if (e >= nR || f >= nR) continue;
        if (MODE == 0) a.T[e * a.ld_t + f] = acc[x][y][v];
        else if (e >= f) __builtin_nontemporal_store(acc[x][y][v] + (e == f ? 1.0 : 0.0), &a.W[e * a.ld_w + f]);
      }
}

// ------------------------------------------------------------------ driver
void launch_woodbury(const WoodArgs &w, hipStream_t s) {
  const BlockMap &B = w.B;
  const int n_cfg = B.nl + B.n_tri;
  hipLaunchKernelGGL(k_qinv, dim3((unsigned)w.n_ell), dim3(WAVE), 0, s, w.Ps, w.nz, w.Q, w.flag);
  const int smax = B.sb > B.sp ? B.sb : B.sp;
  const unsigned gx = (unsigned)((smax * smax + 255) / 256);
  hipLaunchKernelGGL(k_gblock, dim3(gx, (unsigned)n_cfg), dim3(256), 0, s, B, w.cfgT, Qv{w.Q, w.nz}, w.nmodes,
                     w.ntri, w.omega, w.Gb);
  if (smax <= GCHOL_MAX)
    hipLaunchKernelGGL(k_gchol<true>, dim3((unsigned)n_cfg), dim3(256), (size_t)smax * (smax | 1) * 8, s, B, w.Gb, w.dR,
                       w.rR, w.tau, w.rhat, w.W + B.n_R * w.ld_w, w.flag);
  else
    hipLaunchKernelGGL(k_gchol<false>, dim3((unsigned)n_cfg), dim3(256), 0, s, B, w.Gb, w.dR, w.rR, w.tau, w.rhat,
                       w.W + B.n_R * w.ld_w, w.flag);
  WbArgs a{B, w.Gb, w.Gm, w.gm_f32, w.ld_g, w.sexp, w.tau, w.rhat, 1.0 / w.omega, w.sigma_b2, w.T, w.ld_t, w.W,
           w.ld_w};
  const int64_t nt = (B.n_R + 63) / 64;
  hipLaunchKernelGGL(k_wb_prod<0>, dim3((unsigned)(nt * nt)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_wb_prod<1>, dim3((unsigned)(nt * (nt + 1) / 2)), dim3(256), 0, s, a);
}

}  // namespace wlc
