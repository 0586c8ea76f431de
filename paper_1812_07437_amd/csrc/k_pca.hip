// Principal components of the joint covariance (Rizzato et al. 2019, arXiv
// 1812.07437, Sec. 6): C = sum_a lambda_a S_a S_a^T (eq. SNPCA), the new
// observables D^_a = S_a . D (eq. NewObs) and their (S/N)^2_a = D^_a^2 /
// lambda_a (eq. SNperEign), with the cumulative curve of eq. CumulSN.
//
// The eigenvalues span tens of decades.  A tridiagonal eigensolver resolves
// only those above about 1e-16 of the largest, so this path uses one-sided
// (Hestenes) Jacobi, which keeps relative accuracy on graded matrices
// (Demmel and Veselic 1992): with C = Delta C^ Delta (Delta = 2^-t, the row
// scaling of the covariance) and C^ = L L^T from the bordered Cholesky,
// C = W W^T for W = Delta L.  Column rotations W -> W Q make the columns w_a
// orthogonal; then lambda_a = |w_a|^2.  Since d = W y (y = L^-1 2^t d, the
// Cholesky's own forward substitution), D^_a / sqrt(lambda_a) is component a of
// Q^T y: y is rotated along.  The rows are taken in decreasing order of the
// diagonal of C before the factorisation, so that the columns of W come graded
// and the rotations start small (Veselic and Hari 1989): 818 rows of the paper's
// binning converge in 7 sweeps of a plain cyclic Jacobi instead of 11 on the
// rows of Delta L, with the same accuracy (327 rows against 80-bit arithmetic:
// 3.3e-13 on the worst of 17 decades of eigenvalues, 3.1e-13 on the rows).
//
// The eigenvectors need the other side.  w_a / |w_a| has an error of tol in every
// entry, but its entry at a row k of much larger variance is as small as
// sqrt(lambda_a / C_kk), and S_a . d, where d_k is as much larger, takes it at
// its own size.  With vectors the method therefore works on W^T = L^T Delta:
// rotations W^T -> W^T V of its columns, those of the rows of W, are accumulated
// in V, whose columns are the eigenvectors, and an angle between columns of
// different norms is itself as small as their ratio.  Then lambda_a = |w_a|^2
// for the columns w_a of W^T V, and D^_a = w_a . y with y as it is.  Largest error of
// (S_a . d)^2 / lambda_a over the whole S/N at 818, 2420 and 4550 rows: 2e-15, 8e-15
// and 1e-14, from w_a / |w_a| 3e-5, 4e-5 and 8e-6.  It costs sweeps (11, 17 and 18
// instead of 7, 10 and 15, the diagonal's order or the natural one alike) and the
// second product of a round: 12.6, 103 and 473 ms against 6.9, 44 and 259.
//
// Storage: the columns of W (with vectors of W^T, and of V) are the rows of X
// (and of V; zero-padded to n_pad), so every vector the method touches is a contiguous row.  Rows are grouped in blocks of
// 32; each round pairs all blocks (a round-robin tournament over n_blk =
// n_pad / 32 blocks, n_blk - 1 rounds per sweep); for each pair (p, q) the
// 64 x 64 Gram matrix of its rows is formed on FP64 MFMA, rotated towards
// diagonal form by cyclic two-sided Jacobi in LDS (relative accuracy again:
// rotations are driven by |M_jl| / sqrt(M_jj M_ll)), and the 64 x 64 rotation is
// applied to its rows of X on FP64 MFMA.  The first round of a sweep rotates
// every pair of a 64-row pair of blocks, the others those across the two
// blocks, so that a sweep rotates every pair of columns once.  Sweeps repeat
// until no pair has a scaled off-diagonal entry above tol.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace wlc {

constexpr int PB = 32;        // rows per block
constexpr int PR = 2 * PB;    // rows per pair
constexpr int PLD = PR + 1;   // padded LDS row

// Round-robin tournament: position 0 is fixed, the others rotate by r.
__device__ __forceinline__ int rr_at(int pos, int r, int n) { return pos == 0 ? 0 : 1 + (pos - 1 + r) % (n - 1); }

// Where a diagonal entry C 2^-2t of C_true stands: its exponent and mantissa,
// compared one after the other, so that no scale rounds or overflows; entries
// that are not positive (or no number: the factorisation refuses them later)
// come last, infinite ones first.
__device__ __forceinline__ void diag_key(double c, int t, int &e, double &f) {
  f = frexp(c, &e);
  e -= 2 * t;
  if (!(c > 0.0)) { e = INT32_MIN; f = 0.0; }
  if (c == __builtin_inf()) { e = INT32_MAX; f = 0.0; }
}

// One wavefront per row: the rank of the row in decreasing order of the
// diagonal of C_true (ties by index), as the permutation that puts the rows in
// that order.
template <typename InT>
__global__ void k_pca_order(const InT *__restrict__ C, const int32_t *__restrict__ t, int64_t n,
                            int32_t *__restrict__ perm) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t a = (int64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE;
  if (a >= n) return;
  int ea, eb;
  double fa, fb;
  diag_key((double)C[a * n + a], t[a], ea, fa);
  int rank = 0;
  for (int64_t b = lane; b < n; b += WAVE) {
    diag_key((double)C[b * n + b], t[b], eb, fb);
    rank += eb > ea || (eb == ea && (fb > fa || (fb == fa && b < a)));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) rank += __shfl_xor(rank, o, WAVE);
  if (lane == 0) perm[rank] = (int32_t)a;
}

// X from the bordered factor Wm of the ordered rows (rows 0..n-1: L in the lower
// triangle, row n: y): X[j][k] = 2^-t_k Wm[k][j] for j <= k < n, else 0, by way of
// LDS; with VECTORS its transpose; y_pad = row n of Wm.  A 64 x 64 block per
// workgroup.
template <bool VECTORS>
__global__ __launch_bounds__(256) void k_pca_init(const double *__restrict__ Wm, int64_t ld,
                                                  const int32_t *__restrict__ t, const int32_t *__restrict__ perm,
                                                  int64_t n, int64_t n_pad, double *__restrict__ X,
                                                  double *__restrict__ y) {
  __shared__ double tile[64][65];
  const int64_t j0 = (int64_t)blockIdx.y * 64, k0 = (int64_t)blockIdx.x * 64;
  const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
  for (int r = r0; r < 64; r += 4) {
    const int64_t k = k0 + r, j = j0 + c;
    const double x = k < n && j <= k ? ldexp(Wm[k * ld + j], -t[perm[k]]) : 0.0;
    if constexpr (VECTORS) X[k * n_pad + j] = x;
    else tile[r][c] = x;
  }
  __syncthreads();
  if constexpr (!VECTORS)
    for (int r = r0; r < 64; r += 4) X[(j0 + r) * n_pad + k0 + c] = tile[c][r];
  if (blockIdx.x == 0 && threadIdx.x < 64) {
    const int64_t j = j0 + threadIdx.x;
    y[j] = j < n ? Wm[n * ld + j] : 0.0;
  }
}

__global__ void k_pca_identity(int64_t n_pad, double *__restrict__ V) {
  const int64_t j = blockIdx.y, k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n_pad) V[j * n_pad + k] = j == k ? 1.0 : 0.0;
}

__device__ __forceinline__ void atomic_max_nonneg(double *addr, double v) {
  // non-negative doubles order like their bit patterns
  atomicMax(reinterpret_cast<unsigned long long *>(addr), (unsigned long long)__double_as_longlong(v));
}

// A round is three launches.  (a) k_pca_gram: partial 64 x 64 Gram matrices
// of each block pair over column slices (FP64 MFMA); (b) k_pca_rot or
// k_pca_cross, one workgroup per pair: sum the slices in fixed order, measure the largest
// scaled off-diagonal entry, and unless it is below tol rotate M in LDS, store
// Q and rotate the pair's components of y, if given (reordering the rotated columns by
// norm, as in de Rijk's sorting, was measured to break the convergence of the
// cyclic tournament here); (c) k_pca_apply: rows of X (and V) <- Q^T rows, skipped for
// pairs that did not rotate.
__device__ __forceinline__ int64_t pair_row(int bp, int bq, int j) {
  return j < PB ? (int64_t)bp * PB + j : (int64_t)bq * PB + (j - PB);
}

constexpr int PART = PCA_PART;

// Gram of a pair.  The pair's 64 rows are copied one 64-column chunk ahead into two LDS buffers of [64 rows][64
// doubles], unpadded, with the 16-byte chunk s of row l at slot s ^ (l & 15),
// so the 16 consecutive rows one MFMA operand read touches at one column
// fall on 16 distinct bank groups.  A wavefront copy fills two rows.
//
// Bound at few pairs by the chain of a slice's chunks, at many by reading X: 8 us
// a round at 832 columns, 16 at 2432 (47 MB); 10.6 and 21 us with the full
// 64 x 64 square, one quadrant per wavefront.
__device__ __forceinline__ int gram_slot(int l, int k) { return l * PR + 2 * ((k >> 1) ^ (l & 15)) + (k & 1); }

__global__ __launch_bounds__(256) void k_pca_gram(const double *__restrict__ X, int64_t n_pad, int n_blk, int r,
                                                    double *__restrict__ part) {
  __shared__ __attribute__((aligned(16))) double st0[2 * PART];
  __shared__ __attribute__((aligned(16))) double st1[2 * PART];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pi = blockIdx.x, ks = blockIdx.y;
  const int bp = rr_at(pi, r, n_blk), bq = rr_at(n_blk - 1 - pi, r, n_blk);
  // this slice's 64-column chunks
  const int all = (int)(n_pad / PR), first = (int)((int64_t)all * ks / gridDim.y);
  const int64_t c0 = (int64_t)first * PR;
  const int nch = (int)((int64_t)all * (ks + 1) / gridDim.y) - first;
  // copy i of this wavefront: rows l0 = 2 (4 i + w) and l0 + 1 of the pair
  // (one 32-row block, so consecutive rows of X), one descriptor per copy
  const double *rows[8];
  uint32_t off[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int l0 = 2 * (i * 4 + wave), l = l0 + (lane >> 5);
    rows[i] = X + pair_row(bp, bq, l0) * n_pad;
    off[i] = (uint32_t)(((lane >> 5) * n_pad + 2 * ((lane & 31) ^ (l & 15))) * 8);
  }
  auto issue = [&](int ci, double *buf) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          __builtin_amdgcn_make_buffer_rsrc((void *)rows[i], 0, (int)(2 * n_pad * 8), 0x00020000),
          (__attribute__((address_space(3))) void *)(buf + (i * 4 + wave) * 2 * PR), 16, off[i],
          (int)((c0 + (int64_t)ci * PR) * 8), 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // each wavefront sums the ten 16 x 16 tiles of the lower triangle over a
  // quarter of the chunk's columns: one read per row block and step serves
  // as both operands
  f64x4 acc[10];
#pragma unroll
  for (int x = 0; x < 10; ++x) acc[x] = f64x4{0.0, 0.0, 0.0, 0.0};
  auto compute = [&](const double *buf) {
#pragma unroll
    for (int kk = 0; kk < PR / 4; kk += 4) {
      const int k = wave * (PR / 4) + kk + (lane >> 4);
      double a[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) a[x] = buf[gram_slot(x * 16 + (lane & 15), k)];
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int z = 0; z <= x; ++z)
          acc[x * (x + 1) / 2 + z] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x], a[z], acc[x * (x + 1) / 2 + z], 0, 0, 0);
    }
  };
  if (nch > 0) issue(0, st0);
  int ci = 0;
  for (; ci + 1 < nch; ci += 2) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's copy of chunk ci
    __syncthreads();
    issue(ci + 1, st1);
    compute(st0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    if (ci + 2 < nch) issue(ci + 2, st0);
    compute(st1);
  }
  if (ci < nch) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    compute(st0);
  }
  // the wavefronts' sums in order, through LDS; tile x (x + 1) / 2 + z of the
  // result is 64 lanes of four values (row l / 16 + 4 v, column l % 16)
  __syncthreads();
  double *P = part + ((int64_t)pi * gridDim.y + ks) * PART;
  double *sum = wave < 2 ? st0 : st1;  // 20 KB per wavefront
#pragma unroll
  for (int x = 0; x < 10; ++x)
#pragma unroll
    for (int v = 0; v < 4; v += 2)
      *reinterpret_cast<double2 *>(&sum[(wave & 1) * PART + x * 256 + v * 64 + 2 * lane]) =
          make_double2(acc[x][v], acc[x][v + 1]);
  __syncthreads();
  for (int e = 2 * tid; e < PART; e += 512) {
    double2 o = *reinterpret_cast<const double2 *>(&st0[e]);
    const double2 o1 = *reinterpret_cast<const double2 *>(&st0[PART + e]);
    const double2 o2 = *reinterpret_cast<const double2 *>(&st1[e]), o3 = *reinterpret_cast<const double2 *>(&st1[PART + e]);
    o.x = ((o.x + o1.x) + o2.x) + o3.x;
    o.y = ((o.y + o1.y) + o2.y) + o3.y;
    *reinterpret_cast<double2 *>(&P[e]) = o;
  }
}

constexpr int RT = 512;       // threads of the rotation kernel
constexpr int QLD = PR + 2;   // padded row of Q^T (16-byte aligned)

// 1 / sqrt(x) for x in the normal range: estimate and one third-order step
__device__ __forceinline__ double rsqrt_near(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// The rotation that zeroes m = M_jl between a = M_jj and b = M_ll:
// x_j' = c x_j - s x_l, x_l' = s x_j + c x_l, |angle| <= pi / 4, t = s / c.  With
// h = sqrt((b - a)^2 + 4 m^2): cos 2 theta = |b - a| / h, c = sqrt((1 + cos) / 2),
// s = m / (h c), signed.  The exponents are taken out first, so neither squares
// nor h leave the range, and (c, s) is brought back to unit length to rounding.
__device__ __forceinline__ void jacobi_angle(double a, double b, double m, double &c, double &s, double &t) {
  const double d0 = b - a;
  const int em = __builtin_amdgcn_frexp_exp(m) + 1;
  const int e = d0 == 0.0 ? em : max(__builtin_amdgcn_frexp_exp(d0), em);
  const double d = ldexp(d0, -e), m2 = ldexp(m, 1 - e);
  const double rh = rsqrt_near(fma(d, d, m2 * m2));
  const double u = fma(0.5 * fabs(d), rh, 0.5);
  const double ru = rsqrt_near(u);
  const double sg = d0 >= 0.0 ? 0.5 : -0.5;
  c = u * ru;
  s = sg * m2 * rh * ru;
  const double f = 0.5 * fma(-s, s, fma(-c, c, 1.0));
  c = fma(c, f, c);
  s = fma(s, f, s);
  t = sg * m2 * rh * ru * ru;
}

// Whether m = M_jl is above tol of sqrt(a b), a = M_jj and b = M_ll (false where one
// of them is zero): squares of mantissas, and the exponents apart, since a b, and
// m^2 long before it, leaves the range of a double well within that of C.
__device__ __forceinline__ bool above_tol(double a, double b, double m, double tol2) {
  const double x = __builtin_amdgcn_frexp_mant(m);
  const int e = 2 * __builtin_amdgcn_frexp_exp(m) - __builtin_amdgcn_frexp_exp(a) - __builtin_amdgcn_frexp_exp(b);
  return ldexp(x * x, e) > tol2 * (__builtin_amdgcn_frexp_mant(a) * __builtin_amdgcn_frexp_mant(b)) && a > 0.0 && b > 0.0;
}

// |m| / sqrt(a b), exponents apart as above; 0 where a or b is zero
__device__ __forceinline__ double scaled_entry(double a, double b, double m) {
  const int e = __builtin_amdgcn_frexp_exp(a) + __builtin_amdgcn_frexp_exp(b);
  const double p = __builtin_amdgcn_frexp_mant(a) * __builtin_amdgcn_frexp_mant(b);
  return p > 0.0 ? ldexp(fabs(m), -(e >> 1)) / sqrt(e & 1 ? 2.0 * p : p) : 0.0;
}

// What both rotation kernels begin with, on T threads: M (lower triangle, row >=
// column) from the slices, in order, and the pair's largest scaled off-diagonal
// entry; whether it is above tol (else the pair is orthogonal).
template <int T>
__device__ __forceinline__ bool rot_begin(const double *__restrict__ part, int n_ks, double tol, int pi,
                                          double *__restrict__ M, double *__restrict__ diag, double *__restrict__ red,
                                          int32_t *__restrict__ rot, double *__restrict__ conv) {
  constexpr int NV = (PART / 2 + T - 1) / T;
  const int tid = threadIdx.x;
  const double *P = part + (int64_t)pi * n_ks * PART;
  double2 v[NV];
  int row[NV], col[NV], at[NV];  // of v.x; v.y is four rows below
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const int e = 2 * min(tid + T * q, PART / 2 - 1);
    const int tile = e >> 8, l = (e & 127) >> 1;
    const int x = (tile >= 1) + (tile >= 3) + (tile >= 6);
    row[q] = 16 * x + (l >> 4) + 8 * ((e >> 7) & 1);
    col[q] = 16 * (tile - x * (x + 1) / 2) + (l & 15);
    at[q] = e;
    v[q] = *reinterpret_cast<const double2 *>(P + e);
  }
#pragma unroll 2
  for (int k = 1; k < n_ks; ++k)
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const double2 w = *reinterpret_cast<const double2 *>(P + (int64_t)k * PART + at[q]);
      v[q].x += w.x;
      v[q].y += w.y;
    }
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    if (row[q] >= col[q]) M[row[q] * PLD + col[q]] = v[q].x;
    if (row[q] + 4 >= col[q]) M[(row[q] + 4) * PLD + col[q]] = v[q].y;
    if (row[q] == col[q]) diag[row[q]] = v[q].x;
    if (row[q] + 4 == col[q]) diag[col[q]] = v[q].y;
  }
  __syncthreads();
  double off = 0.0;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const double dc = diag[col[q]];
    if (col[q] < row[q]) off = fmax(off, scaled_entry(diag[row[q]], dc, v[q].x));
    if (col[q] < row[q] + 4) off = fmax(off, scaled_entry(diag[row[q] + 4], dc, v[q].y));
  }
  off = wave_max(off);
  if ((tid & 63) == 0) red[tid / WAVE] = off;
  __syncthreads();
  double off0 = red[0];
#pragma unroll
  for (int q = 1; q < T / WAVE; ++q) off0 = fmax(off0, red[q]);
  if (tid == 0) {
    atomic_max_nonneg(conv, off0);
    rot[pi] = off0 > tol ? 1 : 0;
  }
  return off0 > tol;
}

// block between pairs bi > bk, numbered e < 496 (else bi is past the last pair)
__device__ __forceinline__ void rot_block(int e, int &bi, int &bk) {
  bi = 1;
  bk = e;
  while (bk >= bi) {
    bk -= bi;
    ++bi;
  }
}

// All 2016 pairs of a pair of blocks (the first round of a sweep), one workgroup
// for each, in 63 round-robin steps.  A step rotates 32 disjoint pairs of indices: 32
// threads find the angles and update their own 2 x 2 block, then every thread
// updates one of the 496 blocks between two pairs, and its share of Q (stored
// transposed, so that a thread takes four rows of both columns at once).  65 us:
// bound by the chain of a step, as the kernel below.
__global__ __launch_bounds__(RT) void k_pca_rot(const double *__restrict__ part, int n_ks, double tol, int n_blk, int r,
                                                double *__restrict__ y, double *__restrict__ Qg,
                                                int32_t *__restrict__ rot, double *__restrict__ conv) {
  __shared__ double M[PR * PLD];
  __shared__ __attribute__((aligned(16))) double QT[PR * QLD];
  __shared__ __attribute__((aligned(16))) double2 cs[PR / 2];
  __shared__ double diag[PR], red[RT / WAVE], ys[PR];
  const int tid = threadIdx.x, pi = blockIdx.x;
  if (!rot_begin<RT>(part, n_ks, tol, pi, M, diag, red, rot, conv)) return;
  for (int e = tid; e < PR * PR; e += RT) QT[e / PR * QLD + e % PR] = e / PR == e % PR ? 1.0 : 0.0;
  int bi, bk;
  rot_block(tid, bi, bk);
  const int qp = tid >> 4, q0 = 4 * (tid & 15);  // Q: pair, first of four rows
  const double tol2 = tol * tol;
  auto lower = [](int i, int k) { return max(i, k) * PLD + min(i, k); };
#pragma unroll 1
  for (int ir = 0; ir < PR - 1; ++ir) {
    auto first = [&](int q) { return rr_at(q, ir, PR); };
    auto second = [&](int q) { return rr_at(PR - 1 - q, ir, PR); };
    if (tid < PR / 2) {
      const int j = first(tid), l = second(tid), jl = lower(j, l);
      const double mjj = M[j * PLD + j], mll = M[l * PLD + l], mjl = M[jl];
      double c = 1.0, sn = 0.0;
      if (above_tol(mjj, mll, mjl, tol2)) {
        double tt;
        jacobi_angle(mjj, mll, mjl, c, sn, tt);
        M[j * PLD + j] = fma(-tt, mjl, mjj);
        M[l * PLD + l] = fma(tt, mjl, mll);
        M[jl] = 0.0;
      }
      cs[tid] = make_double2(c, sn);
    }
    __syncthreads();
    if (bi < PR / 2) {
      const int i0 = first(bi), i1 = second(bi), k0 = first(bk), k1 = second(bk);
      const int p00 = lower(i0, k0), p01 = lower(i0, k1), p10 = lower(i1, k0), p11 = lower(i1, k1);
      const double2 ci = cs[bi], ck = cs[bk];
      const double a00 = M[p00], a01 = M[p01], a10 = M[p10], a11 = M[p11];
      const double r00 = ci.x * a00 - ci.y * a10, r10 = ci.y * a00 + ci.x * a10;
      const double r01 = ci.x * a01 - ci.y * a11, r11 = ci.y * a01 + ci.x * a11;
      M[p00] = ck.x * r00 - ck.y * r01;
      M[p01] = ck.y * r00 + ck.x * r01;
      M[p10] = ck.x * r10 - ck.y * r11;
      M[p11] = ck.y * r10 + ck.x * r11;
    }
    const double2 cq = cs[qp];
    if (cq.y != 0.0) {
      double *a = &QT[first(qp) * QLD + q0], *b = &QT[second(qp) * QLD + q0];
      const double2 x0 = *reinterpret_cast<double2 *>(a), x1 = *reinterpret_cast<double2 *>(a + 2);
      const double2 z0 = *reinterpret_cast<double2 *>(b), z1 = *reinterpret_cast<double2 *>(b + 2);
      *reinterpret_cast<double2 *>(a) = make_double2(cq.x * x0.x - cq.y * z0.x, cq.x * x0.y - cq.y * z0.y);
      *reinterpret_cast<double2 *>(a + 2) = make_double2(cq.x * x1.x - cq.y * z1.x, cq.x * x1.y - cq.y * z1.y);
      *reinterpret_cast<double2 *>(b) = make_double2(cq.y * x0.x + cq.x * z0.x, cq.y * x0.y + cq.x * z0.y);
      *reinterpret_cast<double2 *>(b + 2) = make_double2(cq.y * x1.x + cq.x * z1.x, cq.y * x1.y + cq.x * z1.y);
    }
    __syncthreads();
  }
  double *out = Qg + (int64_t)pi * PR * PR;
  for (int e = tid; e < PR * PR; e += RT) out[e] = QT[(e % PR) * QLD + e / PR];
  if (!y) return;
  // y of the pair <- Q^T y
  const int bp = rr_at(pi, r, n_blk), bq = rr_at(n_blk - 1 - pi, r, n_blk);
  if (tid < PR) ys[tid] = y[pair_row(bp, bq, tid)];
  __syncthreads();
  if (tid < PR) {
    double o = 0.0;
#pragma unroll 8
    for (int l = 0; l < PR; ++l) o += QT[tid * QLD + l] * ys[l];
    y[pair_row(bp, bq, tid)] = o;
  }
}

// The 1024 pairs across the two blocks (the other rounds) in 32 steps, step k
// rotating j < 32 with 32 + (j + k) mod 32.  M is kept twice, a step reading the
// one and writing the other, so that while eight wavefronts apply step k (as
// above, but for the pairs' own 2 x 2 blocks) the first one already finds the
// angles of step k + 1: lane j holds M_jj and, of its partner, M_ll; the partner's
// neighbour hands over the next M_ll, and the next M_jl is one entry of the block
// between the two pairs.  One barrier per step.  Q is in registers: a thread has
// two rows of columns j and j + 16 and of their partners, and the partners' columns
// move one pair on after every step.
//
// Bound by the chain of a step (four reads of LDS, an angle with two reciprocal
// square roots, a barrier) and LDS about equally: 18.5 us with six slices to sum, 21.7
// with Q in LDS, 25.4 with angles and updates one after the other; 1024 threads, two divisions and two square roots per
// angle and all 63 steps in every round took 100 (a barrier over 16 wavefronts
// takes 265 ns, one over eight a fraction of it).
constexpr int CT = RT + WAVE;
// the next lane's value among 16 (the last one's: the first one's)
__device__ __forceinline__ double next_of_16(double x) {
  const int64_t b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x12F, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x12F, 0xf, 0xf, true);
  return __longlong_as_double(((int64_t)hi << 32) | (uint32_t)lo);
}
// the next lane's value (the last lane: the first one's)
__device__ __forceinline__ double next_lane(double x) {
  const int64_t b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x134, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x134, 0xf, 0xf, true);
  return __longlong_as_double(((int64_t)hi << 32) | (uint32_t)lo);
}
__global__ __launch_bounds__(CT) void k_pca_cross(const double *__restrict__ part, int n_ks, double tol, int n_blk,
                                                  int r, double *__restrict__ y, double *__restrict__ Qg,
                                                  int32_t *__restrict__ rot, double *__restrict__ conv) {
  constexpr int H = PR / 2;
  __shared__ double M0[2 * PR * PLD];
  __shared__ __attribute__((aligned(16))) double2 cs[2][H];
  __shared__ double diag[PR], red[CT / WAVE], ys[H][PR + 1];
  const int tid = threadIdx.x, pi = blockIdx.x;
  if (!rot_begin<CT>(part, n_ks, tol, pi, M0, diag, red, rot, conv)) return;
  auto lower = [](int i, int k) { return max(i, k) * PLD + min(i, k); };
  const int bp = rr_at(pi, r, n_blk), bq = rr_at(n_blk - 1 - pi, r, n_blk);
  if (tid < WAVE) {
    const int j = tid & (H - 1), jn = (j + 1) & (H - 1);  // both halves alike
    const double tol2 = tol * tol;
    double mjj = M0[j * PLD + j], mll = M0[(H + j) * PLD + H + j], mjl = M0[(H + j) * PLD + j];
    double c, s, t;
    bool on;
    auto angle = [&]() {
      on = above_tol(mjj, mll, mjl, tol2);
      jacobi_angle(mjj, mll, mjl, c, s, t);  // no number where both are zero
      c = on ? c : 1.0;
      s = on ? s : 0.0;
      t = on ? t : 0.0;
    };
    __builtin_amdgcn_s_setprio(3);  // the others wait for this wavefront
    angle();
    cs[0][j] = make_double2(c, s);
    double cn = next_lane(c), sn = next_lane(s), next = next_lane(fma(t, mjl, mll));
    __syncthreads();
#pragma unroll 1
    for (int k = 0; k < H; ++k) {
      const double *M = M0 + (k & 1) * PR * PLD;
      double *out = M0 + ((k + 1) & 1) * PR * PLD;
      const int l = H + ((j + k) & (H - 1)), ln = H + ((j + k + 1) & (H - 1));
      const double a00 = M[lower(j, jn)], a10 = M[l * PLD + jn], a01 = M[ln * PLD + j], a11 = M[lower(l, ln)];
      out[l * PLD + j] = on ? 0.0 : mjl;
      mjj = fma(-t, mjl, mjj);
      mll = next;
      mjl = sn * (c * a00 - s * a10) + cn * (c * a01 - s * a11);
      angle();
      cs[(k + 1) & 1][j] = make_double2(c, s);
      cn = next_lane(c);
      sn = next_lane(s);
      next = next_lane(fma(t, mjl, mll));
      __syncthreads();
    }
  } else {
    const int e = tid - WAVE;
    int bi, bk;
    rot_block(e, bi, bk);
    // rows row and row + 1 of Q, columns j + 16 p and their partners
    const int j = e & 15, row = 2 * (e >> 4);
    double x[2][2], z[2][2];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        x[p][i] = row + i == j + 16 * p ? 1.0 : 0.0;
        z[p][i] = row + i == H + j + 16 * p ? 1.0 : 0.0;
      }
    const double y0 = y ? y[pair_row(bp, bq, row)] : 0.0, y1 = y ? y[pair_row(bp, bq, row + 1)] : 0.0;
    __syncthreads();
#pragma unroll 1
    for (int k = 0; k < H; ++k) {
      const double *M = M0 + (k & 1) * PR * PLD;
      double *out = M0 + ((k + 1) & 1) * PR * PLD;
      const double2 *cur = cs[k & 1];
      if (bi < H) {
        const int li = H + ((bi + k) & (H - 1)), lk = H + ((bk + k) & (H - 1));
        const int p00 = bi * PLD + bk, p01 = lk * PLD + bi, p10 = li * PLD + bk, p11 = lower(li, lk);
        const double2 ci = cur[bi], ck = cur[bk];
        const double a00 = M[p00], a01 = M[p01], a10 = M[p10], a11 = M[p11];
        const double r00 = ci.x * a00 - ci.y * a10, r10 = ci.y * a00 + ci.x * a10;
        const double r01 = ci.x * a01 - ci.y * a11, r11 = ci.y * a01 + ci.x * a11;
        out[p00] = ck.x * r00 - ck.y * r01;
        out[p01] = ck.y * r00 + ck.x * r01;
        out[p10] = ck.x * r10 - ck.y * r11;
        out[p11] = ck.y * r10 + ck.x * r11;
      }
      const double2 c0 = cur[j], c1 = cur[j + 16];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const double u = x[0][i], v = x[1][i];
        x[0][i] = c0.x * u - c0.y * z[0][i];
        x[1][i] = c1.x * v - c1.y * z[1][i];
        // the partners' columns go to the pairs before: lane j + 1's, and
        // across the ends of the 16 lanes
        const double n0 = next_of_16(c0.y * u + c0.x * z[0][i]), n1 = next_of_16(c1.y * v + c1.x * z[1][i]);
        z[0][i] = j == 15 ? n1 : n0;
        z[1][i] = j == 15 ? n0 : n1;
      }
      __syncthreads();
    }
    double *out = Qg + (int64_t)pi * PR * PR + row * PR + j;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        out[i * PR + 16 * p] = x[p][i];
        out[i * PR + 16 * p + H] = z[p][i];
      }
      ys[e >> 4][j + 16 * p] = x[p][0] * y0 + x[p][1] * y1;
      ys[e >> 4][j + 16 * p + H] = z[p][0] * y0 + z[p][1] * y1;
    }
  }
  if (!y) return;
  __syncthreads();
  // y of the pair <- Q^T y
  if (tid < PR) {
    double o = 0.0;
#pragma unroll 8
    for (int l = 0; l < H; ++l) o += ys[l][tid];
    y[pair_row(bp, bq, tid)] = o;
  }
}

// Per mode a < n: lambda_a = |x_a|^2 and (S/N)^2_a = y_a^2 (y rotated along), with
// VECTORS (x_a . y)^2 / lambda_a.
template <bool VECTORS>
__global__ void k_pca_modes(const double *__restrict__ X, const double *__restrict__ y, int64_t n, int64_t n_pad,
                            double *__restrict__ lam, double *__restrict__ snr2) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t a = (int64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE;
  if (a >= n) return;
  const double *x = X + a * n_pad;
  double nn = 0.0, dy = 0.0;
  for (int64_t k = lane; k < n_pad; k += WAVE) {
    nn += x[k] * x[k];
    if (VECTORS) dy += x[k] * y[k];
  }
  nn = wave_sum(nn);
  if (VECTORS) dy = wave_sum(dy);
  if (lane == 0) {
    lam[a] = nn;
    const double v = VECTORS ? dy / sqrt(nn) : y[a];
    snr2[a] = nn > 0.0 ? v * v : 0.0;
  }
}

// Rank of each mode by ascending lambda (ties by index) and by descending
// (S/N)^2, one wavefront per mode.
__global__ void k_pca_rank(const double *__restrict__ lam, const double *__restrict__ snr2, int64_t n,
                           int32_t *__restrict__ rank_lam, int32_t *__restrict__ rank_snr) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t a = (int64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE;
  if (a >= n) return;
  const double la = lam[a], sa = snr2[a];
  int rl = 0, rs = 0;
  for (int64_t b = lane; b < n; b += WAVE) {
    const double lb = lam[b], sb = snr2[b];
    rl += (lb < la) || (lb == la && b < a);
    rs += (sb > sa) || (sb == sa && b < a);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    rl += __shfl_xor(rl, o, WAVE);
    rs += __shfl_xor(rs, o, WAVE);
  }
  if (lane == 0) {
    rank_lam[a] = rl;
    rank_snr[a] = rs;
  }
}

__global__ void k_pca_scatter(const double *__restrict__ lam, const double *__restrict__ snr2,
                              const int32_t *__restrict__ rank_lam, const int32_t *__restrict__ rank_snr, int64_t n,
                              double *__restrict__ lam_out, double *__restrict__ snr2_out,
                              double *__restrict__ desc) {
  const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= n) return;
  lam_out[rank_lam[a]] = lam[a];
  snr2_out[rank_lam[a]] = snr2[a];
  desc[rank_snr[a]] = snr2[a];
}

// Cumulative sum in place by one wavefront, 64 values at a time.
__global__ void k_pca_cumsum(double *__restrict__ v, int64_t n) {
  const int lane = threadIdx.x;
  double s = 0.0;
  double next = lane < n ? v[lane] : 0.0;
  for (int64_t b = 0; b < n; b += WAVE) {
    double x = next;
    next = b + WAVE + lane < n ? v[b + WAVE + lane] : 0.0;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const double u = __shfl_up(x, o, WAVE);
      if (lane >= o) x += u;
    }
    x += s;
    if (b + lane < n) v[b + lane] = x;
    s = __shfl(x, WAVE - 1, WAVE);
  }
}

// Eigenvector rows in ascending-lambda order, back in the data
// vector's order, with the sign that makes the largest entry in magnitude
// positive (the first of them in the data vector's order).
__global__ void k_pca_vectors(const double *__restrict__ V, const int32_t *__restrict__ rank_lam,
                              const int32_t *__restrict__ perm, int64_t n, int64_t n_pad, double *__restrict__ S) {
  __shared__ double bv[256];
  __shared__ int64_t bi[256];
  __shared__ int64_t bk[256];
  const int64_t a = blockIdx.x;
  const double *v = V + a * n_pad;
  double best = -1.0;
  int64_t at = n, bat = 0;
  for (int64_t k = threadIdx.x; k < n; k += blockDim.x) {
    const double m = fabs(v[k]);
    if (m > best || (m == best && perm[k] < at)) { best = m; at = perm[k]; bat = k; }
  }
  bv[threadIdx.x] = best;
  bi[threadIdx.x] = at;
  bk[threadIdx.x] = bat;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      const double o = bv[threadIdx.x + w];
      const int64_t oi = bi[threadIdx.x + w];
      if (o > bv[threadIdx.x] || (o == bv[threadIdx.x] && oi < bi[threadIdx.x])) {
        bv[threadIdx.x] = o;
        bi[threadIdx.x] = oi;
        bk[threadIdx.x] = bk[threadIdx.x + w];
      }
    }
    __syncthreads();
  }
  const double sg = v[bk[0]] < 0.0 ? -1.0 : 1.0;
  double *out = S + (int64_t)rank_lam[a] * n;
  for (int64_t k = threadIdx.x; k < n; k += blockDim.x) out[perm[k]] = sg * v[k];
}

void launch_pca_order(const void *C, int c_f32, const int32_t *t, int64_t n, int32_t *perm, hipStream_t s) {
  const dim3 grid((unsigned)((n + 3) / 4));
  if (c_f32)
    hipLaunchKernelGGL(k_pca_order<float>, grid, dim3(256), 0, s, (const float *)C, t, n, perm);
  else
    hipLaunchKernelGGL(k_pca_order<double>, grid, dim3(256), 0, s, (const double *)C, t, n, perm);
}

void launch_pca_init(const double *Wm, int64_t ld, const int32_t *t, const int32_t *perm, int64_t n, int64_t n_pad,
                     bool vectors, double *X, double *y, hipStream_t s) {
  const dim3 grid((unsigned)(n_pad / 64), (unsigned)(n_pad / 64));
  if (vectors)
    hipLaunchKernelGGL(k_pca_init<true>, grid, dim3(256), 0, s, Wm, ld, t, perm, n, n_pad, X, y);
  else
    hipLaunchKernelGGL(k_pca_init<false>, grid, dim3(256), 0, s, Wm, ld, t, perm, n, n_pad, X, y);
}

void launch_pca_identity(int64_t n_pad, double *V, hipStream_t s) {
  hipLaunchKernelGGL(k_pca_identity, dim3((unsigned)((n_pad + 255) / 256), (unsigned)n_pad), dim3(256), 0, s, n_pad, V);
}

// Rotation of a pair's rows.  Q's fragments stay in
// registers; the pair's 64 rows are copied from global memory straight into
// LDS (buffer loads with the LDS flag: lane l of a wavefront writes 16 bytes
// at the wavefront's LDS base + 16 l), one 64-column chunk ahead, into two
// buffers of [64 rows][64 doubles], unpadded, with the 16-byte chunk s of
// row l at slot s ^ (8 (l & 1)): the four rows one MFMA operand read touches
// fall on alternate halves of the banks.  A wavefront copy fills two rows.
__device__ __forceinline__ int apply_slot(int l, int col) { return l * PR + 2 * ((col >> 1) ^ (8 * (l & 1))) + (col & 1); }

// `per` chunks per workgroup, of X for blockIdx.z = 0 and of V for 1.
__global__ __launch_bounds__(256) void k_pca_apply(double *__restrict__ X, double *__restrict__ V, int64_t n_pad,
                                                     int per, int n_blk, int r, const double *__restrict__ Qg,
                                                     const int32_t *__restrict__ rot) {
  __shared__ __attribute__((aligned(16))) double st0[PR * PR];
  __shared__ __attribute__((aligned(16))) double st1[PR * PR];
  const int pi = blockIdx.x;
  if (!rot[pi]) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bp = rr_at(pi, r, n_blk), bq = rr_at(n_blk - 1 - pi, r, n_blk);
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  double *Y = blockIdx.z == 0 ? X : V;
  // Q fragments: step kk, block x: Q[kk + lane / 16][wr + 16 x + lane % 16]
  const double *q = Qg + (int64_t)pi * PR * PR;
  double qa[PR / 4][2];
#pragma unroll
  for (int kk = 0; kk < PR / 4; ++kk)
#pragma unroll
    for (int x = 0; x < 2; ++x) qa[kk][x] = q[(4 * kk + (lane >> 4)) * PR + wr + x * 16 + (lane & 15)];
  // copies: wavefront w fills LDS rows 2 (8 i + w) + lane / 32 ... for i < 8
  // copy i of this wavefront: rows l0 = 2 (4 i + w) and l0 + 1 of the pair
  // (one 32-row block, so consecutive rows of Y), one descriptor per copy
  const double *rows[8];
  uint32_t off[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int l0 = 2 * (i * 4 + wave), l = l0 + (lane >> 5);
    rows[i] = Y + pair_row(bp, bq, l0) * n_pad;
    off[i] = (uint32_t)(((lane >> 5) * n_pad + 2 * ((lane & 31) ^ (8 * (l & 1)))) * 8);
  }
  const int64_t cbase = (int64_t)blockIdx.y * per * PR;
  const int nch = (int)min((int64_t)per, (n_pad - cbase) / PR);
  auto issue = [&](int ci, double *buf) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          __builtin_amdgcn_make_buffer_rsrc((void *)rows[i], 0, (int)(2 * n_pad * 8), 0x00020000),
          (__attribute__((address_space(3))) void *)(buf + (i * 4 + wave) * 2 * PR), 16, off[i],
          (int)((cbase + (int64_t)ci * PR) * 8), 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto compute = [&](const double *buf, int ci) {
    f64x4 acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int z = 0; z < 2; ++z) acc[x][z] = f64x4{0.0, 0.0, 0.0, 0.0};
    // out[j][c] = sum_l Q[l][j] stage[l][c]
#pragma unroll
    for (int kk = 0; kk < PR / 4; ++kk) {
      const int l = 4 * kk + (lane >> 4);
      double b[2];
#pragma unroll
      for (int z = 0; z < 2; ++z) b[z] = buf[apply_slot(l, wc + z * 16 + (lane & 15))];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int z = 0; z < 2; ++z) acc[x][z] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[kk][x], b[z], acc[x][z], 0, 0, 0);
    }
    const int64_t c0 = cbase + (int64_t)ci * PR;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int z = 0; z < 2; ++z)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int j = wr + x * 16 + (lane >> 4) + 4 * v, c = wc + z * 16 + (lane & 15);
          Y[pair_row(bp, bq, j) * n_pad + c0 + c] = acc[x][z][v];
        }
  };
  // the chunk written back is never one being copied (the copies run one
  // chunk ahead, on other columns)
  if (nch > 0) issue(0, st0);
  int ci = 0;
  for (; ci + 1 < nch; ci += 2) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's copy of chunk ci
    __syncthreads();
    issue(ci + 1, st1);
    compute(st0, ci);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    if (ci + 2 < nch) issue(ci + 2, st0);
    compute(st1, ci + 1);
  }
  if (ci < nch) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    compute(st0, ci);
  }
}

// Column slices of the Gram.  A slice costs its share of the chunks (1.1 us
// each, on one workgroup) and 20 KB for the rotation kernel to read back on one
// CU (0.35 us): about sqrt(3 chunks) slices, as long as the workgroups fit
// the chip four times.
int pca_slices(int64_t n_pad) {
  const int pairs = (int)(n_pad / PR), chunks = (int)(n_pad / PR);
  int ks = 1;
  while ((ks + 1) * (ks + 1) <= 3 * chunks && ks + 1 <= chunks && pairs * (ks + 1) <= 1024) ++ks;
  return ks;
}

void launch_pca_round(double *X, double *V, double *y, int64_t n_pad, int r, double tol, double *conv, double *part, double *Qg,
                      int32_t *rot, hipStream_t s) {
  const int n_blk = (int)(n_pad / PB), pairs = n_blk / 2, ks = pca_slices(n_pad), chunks = (int)(n_pad / PR);
  hipLaunchKernelGGL(k_pca_gram, dim3((unsigned)pairs, (unsigned)ks), dim3(256), 0, s, X, n_pad, n_blk, r, part);
  if (r == 0)
    hipLaunchKernelGGL(k_pca_rot, dim3((unsigned)pairs), dim3(RT), 0, s, part, ks, tol, n_blk, r, y, Qg, rot, conv);
  else
    hipLaunchKernelGGL(k_pca_cross, dim3((unsigned)pairs), dim3(CT), 0, s, part, ks, tol, n_blk, r, y, Qg, rot, conv);
  // chunks per workgroup: eight amortise the 32 KB of Q, fewer while the chip
  // is not filled twice
  const int sides = V ? 2 : 1;
  int per = (int)std::min<int64_t>(8, std::max<int64_t>(1, (int64_t)pairs * chunks * sides / 512));
  hipLaunchKernelGGL(k_pca_apply, dim3((unsigned)pairs, (unsigned)((chunks + per - 1) / per), sides), dim3(256), 0, s,
                     X, V, n_pad, per, n_blk, r, Qg, rot);
}

void launch_pca_finish(const double *X, const double *V, const double *y, const int32_t *perm, int64_t n, int64_t n_pad, double *lam,
                       double *snr2, int32_t *rank_lam, int32_t *rank_snr, double *lam_out, double *snr2_out,
                       double *desc, double *S, hipStream_t s) {
  const dim3 waves((unsigned)((n + 3) / 4));
  if (V)
    hipLaunchKernelGGL(k_pca_modes<true>, waves, dim3(256), 0, s, X, y, n, n_pad, lam, snr2);
  else
    hipLaunchKernelGGL(k_pca_modes<false>, waves, dim3(256), 0, s, X, y, n, n_pad, lam, snr2);
  hipLaunchKernelGGL(k_pca_rank, waves, dim3(256), 0, s, lam, snr2, n, rank_lam, rank_snr);
  hipLaunchKernelGGL(k_pca_scatter, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, lam, snr2, rank_lam, rank_snr,
                     n, lam_out, snr2_out, desc);
  hipLaunchKernelGGL(k_pca_cumsum, dim3(1), dim3(64), 0, s, desc, n);
  if (V) hipLaunchKernelGGL(k_pca_vectors, dim3((unsigned)n), dim3(256), 0, s, V, rank_lam, perm, n, n_pad, S);
}

}  // namespace wlc
