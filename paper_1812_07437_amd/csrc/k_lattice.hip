// Integer lattice counts of modes and triangles (Rizzato et al. 2019,
// Sec. 3.2.2 mode lattice and App. B, N_tri as the sum of the selection
// function Delta^(3)).
//
// Modes are integer vectors q != 0; bin b holds q with T_b <= |q|^2 < T_{b+1}.
// The triangle count of bins (b1, b2, b3) is the number of ordered pairs
// (q1, q2) with q1 in b1, q2 in b2 and q1 + q2 in b3.  A lattice row of a bin
// is a symmetric interval |x| <= B less a smaller one |x| <= A, so the pairs in
// rows y1 and y2 are eight signed terms
//   K(p, q, s) = #{(x1, x2) : |x1| <= p, |x2| <= q, |x1 + x2| <= s},
// and K has a closed form.  The count is a sum over pairs of rows, not over
// modes and rows.  The row half-widths are exact integer square roots.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"

namespace wlc {

// floor(sqrt(v)) for v >= 0, exact in 64-bit integers
__device__ __forceinline__ int64_t isqrt_floor(int64_t v) {
  if (v <= 0) return 0;
  int64_t r = (int64_t)sqrt((double)v);
  while (r * r > v) --r;
  while ((r + 1) * (r + 1) <= v) ++r;
  return r;
}

// x with lo <= x^2 + yy < hi, as up to two disjoint intervals [a0,b0], [a1,b1]
// (empty when a > b).  Returns the number of intervals written.
__device__ __forceinline__ int row_intervals(int64_t lo, int64_t hi, int64_t yy, int64_t *a, int64_t *b) {
  const int64_t top = hi - 1 - yy;  // x^2 <= top
  if (top < 0) return 0;
  const int64_t xmax = isqrt_floor(top);
  const int64_t need = lo - yy;  // x^2 >= need
  int64_t xmin = 0;
  if (need > 0) {
    xmin = isqrt_floor(need - 1) + 1;  // smallest x >= 0 with x^2 >= need
  }
  if (xmin > xmax) return 0;
  if (xmin == 0) {
    a[0] = -xmax; b[0] = xmax;
    return 1;
  }
  a[0] = -xmax; b[0] = -xmin;
  a[1] = xmin; b[1] = xmax;
  return 2;
}

// Largest x with x^2 + y^2 < t, or -1 where the row is empty.
__device__ __forceinline__ int64_t half_width(int64_t t, int64_t y) {
  const int64_t v = t - 1 - y * y;
  return v < 0 ? -1 : isqrt_floor(v);
}

// (u + 1) (u + 2) for u >= 0, else 0: twice the number of pairs i, j >= 0 with
// i + j <= u
__device__ __forceinline__ uint32_t pairs2(int32_t u) { return u >= 0 ? __umul24((uint32_t)u + 1u, (uint32_t)u + 2u) : 0u; }
__device__ __forceinline__ uint64_t pairs2(int64_t u) { return u >= 0 ? (uint64_t)(u + 1) * (uint64_t)(u + 2) : 0u; }
__device__ __forceinline__ uint32_t mul(uint32_t a, uint32_t b) { return __umul24(a, b); }
__device__ __forceinline__ uint64_t mul(uint64_t a, uint64_t b) { return a * b; }

// K(p, q, s), 0 where a half-width is negative: all pairs less twice those with
// x1 + x2 > s (the others have x1 + x2 < -s), i.e. with i + j <= p + q - s - 1 for
// i = p - x1 <= 2 p, j = q - x2 <= 2 q; at most one of i, j can pass its bound.
template <typename I, typename U>
__device__ __forceinline__ U row_pairs(I p, I q, I s) {
  const U k = mul((U)(2 * p + 1), (U)(2 * q + 1)) - pairs2((I)(p + q - s - 1)) + pairs2((I)(q - p - s - 2)) +
              pairs2((I)(p - q - s - 2));
  return (p | q | s) >= 0 ? k : (U)0;
}

// One triangle per blockIdx.y, LY1 rows y1 >= 0 of q1 by 256 rows y2 of q2 per
// workgroup: a thread holds its row y2, the half-widths of the rows y1 and
// y1 + y2 lie in LDS.  Rows y1 > 0 count twice (y -> -y).  With I = int32_t every
// intermediate fits (or wraps and comes back, mod 2^32) for radii to 16000.  The
// workgroups of a triangle are numbered from `base`, the first of this launch.
//
// Bound by integer arithmetic, about 120 instructions per pair of rows.  At
// 10 ell-bins to 3000 (64 triangles) the whole call takes 0.18 ms, against 13.8 ms with interval overlaps
// for every mode of q1 and row of q2.
constexpr int LY1 = 64;
template <typename I, typename U>
__global__ __launch_bounds__(256) void k_lattice_tris(const int64_t *__restrict__ thr, const int32_t *__restrict__ tri,
                                                      int64_t rmax, int64_t base, uint64_t *__restrict__ out) {
  __shared__ I w1[LY1][2], w3[LY1 + 256][2];
  __shared__ uint64_t part[256];
  const int t = blockIdx.y, tid = threadIdx.x;
  const int64_t n2 = (2 * rmax + 256) / 256, wg = base + blockIdx.x;
  const int64_t y1 = wg / n2 * LY1, y2 = wg % n2 * 256 - rmax;
  const int b1 = tri[3 * t], b2 = tri[3 * t + 1], b3 = tri[3 * t + 2];
  const int64_t lo1 = thr[b1], hi1 = thr[b1 + 1];
  const int64_t lo2 = thr[b2], hi2 = thr[b2 + 1], lo3 = thr[b3], hi3 = thr[b3 + 1];
  // the workgroup's nearest rows of q1 and q2 outside their bins: nothing here
  const int64_t near2 = y2 > 0 ? y2 : y2 + 255 < 0 ? y2 + 255 : 0;
  if (y1 * y1 >= hi1 || near2 * near2 >= hi2) return;
  for (int e = tid; e < LY1; e += 256) {
    w1[e][0] = (I)half_width(lo1, y1 + e);
    w1[e][1] = (I)half_width(hi1, y1 + e);
  }
  for (int e = tid; e < LY1 + 256; e += 256) {
    w3[e][0] = (I)half_width(lo3, y1 + y2 + e);
    w3[e][1] = (I)half_width(hi3, y1 + y2 + e);
  }
  const I a2 = (I)half_width(lo2, y2 + tid), c2 = (I)half_width(hi2, y2 + tid);
  __syncthreads();
  uint64_t c = 0;
  for (int e = 0; e < LY1; ++e) {
    const I a1 = w1[e][0], c1 = w1[e][1], a3 = w3[e + tid][0], c3 = w3[e + tid][1];
    if (c1 < 0) break;  // the rows beyond are empty too
    U k = row_pairs<I, U>(c1, c2, c3) - row_pairs<I, U>(c1, c2, a3);
    k -= row_pairs<I, U>(c1, a2, c3) - row_pairs<I, U>(c1, a2, a3);
    k -= row_pairs<I, U>(a1, c2, c3) - row_pairs<I, U>(a1, c2, a3);
    k += row_pairs<I, U>(a1, a2, c3) - row_pairs<I, U>(a1, a2, a3);
    c += (y1 + e == 0 ? (uint64_t)k : 2 * (uint64_t)k);
  }
  part[tid] = c;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) part[tid] += part[tid + w];
    __syncthreads();
  }
  if (tid == 0 && part[0]) atomicAdd((unsigned long long *)&out[t], (unsigned long long)part[0]);
}

__global__ void k_zero_u64(uint64_t *p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// modes per bin: one thread per (bin, row y)
__global__ void k_lattice_modes(const int64_t *__restrict__ thr, int n_ell, int64_t rmax, uint64_t *__restrict__ out) {
  const int b = blockIdx.y;
  const int64_t lo = thr[b], hi = thr[b + 1];
  uint64_t c = 0;
  for (int64_t y = -rmax + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; y <= rmax;
       y += (int64_t)gridDim.x * blockDim.x) {
    int64_t a[2], bb[2];
    const int n = row_intervals(lo, hi, y * y, a, bb);
    for (int p = 0; p < n; ++p) c += (uint64_t)(bb[p] - a[p] + 1);
  }
  if (c) atomicAdd((unsigned long long *)&out[b], (unsigned long long)c);
}

// Full launch helpers with the host-known radius bound.
void launch_lattice(const int64_t *thr_dev, int64_t thr_max, int n_ell, const int32_t *tri, int n_tri,
                    uint64_t *modes, uint64_t *tris, hipStream_t s) {
  const int64_t rmax = (int64_t)std::sqrt((double)thr_max) + 2;
  if (modes) {
    hipLaunchKernelGGL(k_zero_u64, dim3((n_ell + 255) / 256), dim3(256), 0, s, modes, n_ell);
    hipLaunchKernelGGL(k_lattice_modes, dim3(8, n_ell), dim3(256), 0, s, thr_dev, n_ell, rmax, modes);
  }
  if (tris && n_tri > 0) {
    hipLaunchKernelGGL(k_zero_u64, dim3((n_tri + 255) / 256), dim3(256), 0, s, tris, n_tri);
    // one launch up to a radius of 262000
    const int64_t wgs = (rmax / LY1 + 1) * ((2 * rmax + 256) / 256), most = LAUNCH_THREADS / 256;
    for (int64_t base = 0; base < wgs; base += most) {
      const dim3 grid((unsigned)std::min(most, wgs - base), (unsigned)n_tri);
      if (rmax <= 16000)
        hipLaunchKernelGGL((k_lattice_tris<int32_t, uint32_t>), grid, dim3(256), 0, s, thr_dev, tri, rmax, base, tris);
      else
        hipLaunchKernelGGL((k_lattice_tris<int64_t, uint64_t>), grid, dim3(256), 0, s, thr_dev, tri, rmax, base, tris);
    }
  }
}

}  // namespace wlc
