// One-halo covariance through its factorisation along the line of sight.
//
// A row of the flattened one-halo factor is A[row][(n, m)] = T_row(chi_n)
// G_c(chi_n, M_m), c the row's ell-configuration (eq. General1h with the
// Limber kernel of eq. nProjection), so
//   (A A^T)[a][b] = sum_n T_a(n) T_b(n) H_n[c(a)][c(b)],
//   H_n[c][c'] = sum_m G_c(n, m) G_c'(n, m).
// H is small (configurations x configurations x chi nodes), and the second
// sum is a product over the chi nodes only: N_M times fewer operations than
// the flattened Gram, and computed here in FP64 from the same factors T
// (which carry the rows' power-of-two scales) and G.
//
// Distinct rows are grouped by configuration with uniform block sizes
// (sp rows per power-spectrum configuration, sb per triangle).  Blocks are
// cut into sub-tiles of 64 rows; sub-tile rows are numbered configuration
// by configuration, so a pair of sub-tile rows R >= R' covers configurations
// c >= c' and one weight vector h = H[c][c'][.] applies to the whole pair:
// each pair is an FP64 MFMA product over n of up to 64 x 64, with one operand scaled
// by h; only its 16 x 16 tiles that hold rows are computed (15 or 35 rows a block at
// five redshift bins).
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace wlc {

// ------------------------------------------------------------------ H
// H[c][c'][n] = sum_m G[c][n][m] G[c'][n][m] for 32-blocks of c >= c': one
// workgroup per pair of blocks and HN chi nodes, a wavefront per node.  A lane's
// operands are four consecutive m of one row (a contraction takes its terms
// in any order: step q of lane group g holds m = 16 i + 4 g + q on both sides), so
// the 16 rows of a tile are read in whole 128-byte lines, without LDS; the
// results of the HN nodes are put together in LDS and leave as 64-byte runs of n.
//
// Bound by the loads of G: 74 configurations, 256 nodes, 129 columns 22 us (as FP64
// vector products with all c and c' 117).
constexpr int HN = 8;
constexpr int HB = 32;
typedef double h64x4 __attribute__((ext_vector_type(4), aligned(8)));  // rows of any pitch

__global__ __launch_bounds__(HN * 64) void k_hfactor(const double *__restrict__ G, int n_cfg, int n_chi, int n_m,
                                                     double *__restrict__ H) {
  __shared__ double out[HB * HB][HN + 1];
  int bi = (int)((sqrtf(8.0f * (float)blockIdx.x + 1.0f) - 1.0f) * 0.5f);
  while ((bi + 1) * (bi + 2) / 2 <= (int)blockIdx.x) ++bi;
  while (bi * (bi + 1) / 2 > (int)blockIdx.x) --bi;
  const int c0 = bi * HB, p0 = ((int)blockIdx.x - bi * (bi + 1) / 2) * HB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n0 = blockIdx.y * HN, n = min(n0 + wave, n_chi - 1);
  const double *ga[2], *gb[2];
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    ga[x] = G + ((size_t)min(c0 + 16 * x + (lane & 15), n_cfg - 1) * n_chi + n) * n_m;
    gb[x] = G + ((size_t)min(p0 + 16 * x + (lane & 15), n_cfg - 1) * n_chi + n) * n_m;
  }
  f64x4 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
  auto step = [&](const f64x4 *a, const f64x4 *b) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x][q], b[y][q], acc[x][y], 0, 0, 0);
  };
  int m = 4 * (lane >> 4);
  const int whole = n_m & ~15;
#pragma unroll 2
  for (int i = 0; i < whole; i += 16, m += 16) {
    f64x4 a[2], b[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      a[x] = *(const h64x4 *)(ga[x] + m);
      b[x] = *(const h64x4 *)(gb[x] + m);
    }
    step(a, b);
  }
  if (whole < n_m) {
    f64x4 a[2], b[2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool in = m + q < n_m;
        a[x][q] = in ? ga[x][m + q] : 0.0;
        b[x][q] = in ? gb[x][m + q] : 0.0;
      }
    step(a, b);
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        out[(16 * x + (lane >> 4) + 4 * v) * HB + 16 * y + (lane & 15)][wave] = acc[x][y][v];
  __syncthreads();
  for (int q = threadIdx.x; q < HB * HB * HN; q += HN * 64) {
    const int e = q / HN, w = q % HN, c = c0 + e / HB, cp = p0 + e % HB;
    if (c < n_cfg && cp < n_cfg && n0 + w < n_chi) H[((size_t)c * n_cfg + cp) * n_chi + n0 + w] = out[e][w];
  }
}

// ------------------------------------------------------------------ C_1h
struct SubRow {
  int c;       // configuration
  int64_t e0;  // first distinct row
  int cnt;     // rows in this sub-tile (<= 64)
};

__device__ __forceinline__ SubRow sub_row(int64_t R, int nl, int sp, int sb, int tp, int tb) {
  SubRow s;
  if (R < (int64_t)nl * tp) {
    const int c = (int)(R / tp), ti = (int)(R % tp);
    s.c = c;
    s.e0 = (int64_t)c * sp + ti * 64;
    s.cnt = min(64, sp - ti * 64);
  } else {
    const int64_t q = R - (int64_t)nl * tp;
    const int t = (int)(q / tb), ti = (int)(q % tb);
    s.c = nl + t;
    s.e0 = (int64_t)nl * sp + (int64_t)t * sb + ti * 64;
    s.cnt = min(64, sb - ti * 64);
  }
  return s;
}

// Bound by the products (a third to a half of a block's 16 x 16 tiles is
// padding) and the latency of each stage's loads.  2390 rows, 256 nodes: 91 us, against 127 with
// all 64 x 64 computed and the loads waited for before the products of the
// stage in hand.
constexpr int CK = 16;        // chi nodes per LDS stage
constexpr int CLD = CK + 1;   // padded row

__global__ __launch_bounds__(256) void k_chifact(const double *__restrict__ Ts, const double *__restrict__ H,
                                                 int n_cfg, int n_chi, int nl, int sp, int sb, int tp, int tb,
                                                 double *__restrict__ out, int64_t ld) {
  __shared__ double lds[2][64 * CLD];  // [A' rows, B rows][64][CK]
  int64_t R, Rp;
  {
    const int64_t t = blockIdx.x;
    int64_t i = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    while (i * (i + 1) / 2 > t) --i;
    R = i;
    Rp = t - i * (i + 1) / 2;
  }
  const SubRow A = sub_row(R, nl, sp, sb, tp, tb), B = sub_row(Rp, nl, sp, sb, tp, tb);
  const double *h = H + ((size_t)A.c * n_cfg + B.c) * n_chi;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the 16 x 16 tiles that hold rows, dealt to the four wavefronts in turn
  const int ta = (A.cnt + 15) / 16, tbl = (B.cnt + 15) / 16;
  f64x4 acc[4];
  int off_a[4], off_b[4], mine = 0;
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    acc[x] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int q = wave + 4 * x;
    off_a[x] = min(q / tbl, ta - 1) * 16;
    off_b[x] = q % tbl * 16;
    if (q < ta * tbl) mine = x + 1;
  }

  // staging: 64 rows x CK nodes per side, 4 per thread; element q is row
  // q / CK, node q % CK
  // (loads unconditional, from indices clamped into range, and masked by
  // multiplication when they are put into LDS: the factors are finite, and all
  // 12 loads of a thread are in flight together, under the products of the
  // stage before)
  double la[4], lb[4], hv[4];
  auto gload = [&](int n0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int q = tid + 256 * j;
      const int r = q / CK, n = min(n0 + q % CK, n_chi - 1);
      la[j] = Ts[(size_t)(A.e0 + min(r, A.cnt - 1)) * n_chi + n];
      lb[j] = Ts[(size_t)(B.e0 + min(r, B.cnt - 1)) * n_chi + n];
      hv[j] = h[n];
    }
  };
  gload(0);
  for (int n0 = 0; n0 < n_chi; n0 += CK) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int q = tid + 256 * j;
      const int r = q / CK;
      const bool kin = n0 + q % CK < n_chi;
      lds[0][r * CLD + q % CK] = la[j] * hv[j] * ((kin && r < A.cnt) ? 1.0 : 0.0);
      lds[1][r * CLD + q % CK] = lb[j] * ((kin && r < B.cnt) ? 1.0 : 0.0);
    }
    __syncthreads();
    if (n0 + CK < n_chi) gload(n0 + CK);
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      if (x >= mine) break;
#pragma unroll
      for (int kk = 0; kk < CK; kk += 4) {
        const int kc = kk + (lane >> 4);
        const double a = lds[0][(off_a[x] + (lane & 15)) * CLD + kc];
        const double b = lds[1][(off_b[x] + (lane & 15)) * CLD + kc];
        acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[x], 0, 0, 0);
      }
    }
  }
  // accumulator value v of lane l: row l / 16 + 4 v, column l % 16; the
  // product is written non-temporal (the later kernels then run 2.6 ms faster
  // at large10: fewer dirty lines left to write back under them)
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    if (x >= mine) break;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = off_a[x] + (lane >> 4) + 4 * v;
      const int c = off_b[x] + (lane & 15);
      if (r < A.cnt && c < B.cnt) __builtin_nontemporal_store(acc[x][v], &out[(A.e0 + r) * ld + B.e0 + c]);
    }
  }
}

void launch_chifact(const double *Ts, const double *G, double *H, int n_cfg, int n_chi, int n_m, int nl, int sp,
                    int sb, int n_tri, double *out, int64_t ld, hipStream_t s) {
  const unsigned nb = (unsigned)((n_cfg + HB - 1) / HB);
  hipLaunchKernelGGL(k_hfactor, dim3(nb * (nb + 1) / 2, (unsigned)((n_chi + HN - 1) / HN)), dim3(HN * 64), 0, s, G,
                     n_cfg, n_chi, n_m, H);
  const int tp = (sp + 63) / 64, tb = sb > 0 ? (sb + 63) / 64 : 1;
  const int64_t ns = (int64_t)nl * tp + (int64_t)n_tri * tb;
  const int64_t items = ns * (ns + 1) / 2;
  if (items > 0)
    hipLaunchKernelGGL(k_chifact, dim3((unsigned)items), dim3(256), 0, s, Ts, H, n_cfg, n_chi, nl, sp, sb, tp, tb,
                       out, ld);
}

}  // namespace wlc
