// (S/N)^2 = D^T C^-1 D (Rizzato et al. 2019, eq. SNprim) by an FP64 Cholesky
// factorisation of the bordered matrix
//     M = [ C~    d~ ]        C~ = 2^t C 2^t,  d~ = 2^t d,
//         [ d~^T   . ]
// Factoring the first n columns of M leaves y = L^-1 d~ in its last row, and
// (S/N)^2 = y^T y.
//
// Panels of 128 columns, two launches each: the rows below the factored diagonal
// block are solved against it (k_solve), then the trailing columns receive the
// update of the solved panels that is due, while the first workgroups of the
// same launch already update and factor the next diagonal block (k_trail), so
// that the serial chain runs beside the update.
//
// Measured, a call of wlc_snr2 (before: 64-wide diagonal blocks in launches of
// their own, left-looking over 256 columns; both on one card): n = 818 0.95 -> 0.24
// ms, 2420 3.1 -> 0.74 ms, 4550 6.0 -> 1.60 ms, 10000 15.1 -> 7.7 ms, 17059 42.7 ->
// 29.8 ms, 25044 106 -> 84 ms, 33165 219 -> 189 ms, 82575 2.85 -> 2.81 s.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dev.h"
#include "kernels.h"

namespace wlc {

constexpr int NB = 128;      // panel width
// While this many columns remain, the panels of a group of eight update only the
// group's own columns, and then the rest of the matrix together, so that it is
// read and written once per 1024 columns in launches of many tiles (k = 1024: 60
// TFLOP/s).  n = 10000 8.3 ms without groups, 7.8 with; 12768 15.1 and 14.0; 6550
// 3.17 either way; groups down to 4000 remaining columns cost 4550 3 %.
constexpr int64_t GROUP_MIN = 6000;
constexpr int GROUP = 8;
// Otherwise (and among a group's own columns) a column block is updated with
// GAP panels at a time, in every launch the blocks whose turn it is: a GAP-th of
// the reads and writes of the matrix, and each launch its share of the work.
// n = 2420 0.82 ms with every panel at once, 0.78 two, 0.76 four, 0.85 eight (one
// tile then outlasts the factorisation beside it); 4550 1.86, 1.74, 1.66, 1.90.
constexpr int GAP = 4;

// ------------------------------------------------------------- prepare
// Lower triangle of M from the scaled covariance (f32 or f64) and d: one
// block per row and PREP_COLS columns, blocks right of the row's end exit.
// M is written with non-temporal stores (it is far larger than the caches).
constexpr int PREP_COLS = 2048;
template <typename InT>
__global__ void k_chol_prep(const InT *__restrict__ C, const int32_t *__restrict__ t, const double *__restrict__ d,
                            const int32_t *__restrict__ perm, int64_t n, int64_t ld, int64_t row_off,
                            double *__restrict__ Wm) {
  const int64_t i = row_off + blockIdx.y;  // row of M, 0..n
  const int64_t jb = (int64_t)blockIdx.x * PREP_COLS;
  if (i > n || jb > i) return;  // the block lies right of the row's last entry
  const int64_t pi = perm && i < n ? perm[i] : i;
#pragma unroll
  for (int q = 0; q < PREP_COLS / 256; ++q) {
    const int64_t j = jb + q * 256 + threadIdx.x;
    if (j <= i && j < n) {
      const int64_t pj = perm ? perm[j] : j;
      __builtin_nontemporal_store(i < n ? (double)C[pi * n + pj] : ldexp(d[pj], t[pj]), &Wm[i * ld + j]);
    }
  }
}

void launch_chol_prep(const void *C, int c_f32, const int32_t *row_exp2, const double *d, int64_t n, int64_t ld,
                      double *Wm, hipStream_t s, const int32_t *perm) {
  for (int64_t r0 = 0; r0 <= n; r0 += 65535) {
    const int64_t rows = std::min<int64_t>(65535, n + 1 - r0);
    const dim3 grid((unsigned)((n + PREP_COLS - 1) / PREP_COLS), (unsigned)rows);
    if (c_f32)
      hipLaunchKernelGGL(k_chol_prep<float>, grid, dim3(256), 0, s, (const float *)C, row_exp2, d, perm, n, ld, r0,
                         Wm);
    else
      hipLaunchKernelGGL(k_chol_prep<double>, grid, dim3(256), 0, s, (const double *)C, row_exp2, d, perm, n, ld,
                         r0, Wm);
  }
}

// ------------------------------------------------------------- panels of 128
// Everything inside a panel works on 16 x 16 tiles held transposed in
// registers: T(w, j), row block w and column block j, has in lane l = 16 g + r
// and element v the entry of row 16 w + r, column 16 j + g + 4 v.  That is the
// accumulator of v_mfma_f64_16x16x4 for the product (columns of block j) x
// (rows of block w), and the same registers are, as they stand, its two
// operands: element v is what step v of a 16-deep product wants from either
// side.  So T(w, t) -= L(t, j) T(w, j) and T(w, j) <- L_jj^-1 T(w, j) chain from
// register to register, and a tile that other wavefronts need goes through
// memory as it stands, lane after lane ("packed": element pairs (0, 1) of the
// 64 lanes, then (2, 3)).
constexpr int RB = 16;          // rows of a tile
constexpr int NT = NB / RB;     // tiles across a panel
constexpr int TILE = RB * RB;   // doubles of a tile
constexpr int PACK_ROW = NT * TILE;                    // doubles of a packed row block: 16 rows x 128 columns
constexpr int PACK_DIAG = NT * (NT + 1) / 2 * TILE;    // packed diagonal block: L(t, j), t > j, and L_jj^-1

__device__ __forceinline__ int diag_at(int t, int j) { return (t * (t + 1) / 2 + j) * TILE; }

// tile <-> packed memory
__device__ __forceinline__ void put_tile(double *dst, int lane, const f64x4 &t) {
  *reinterpret_cast<double2 *>(dst + 2 * lane) = make_double2(t[0], t[1]);
  *reinterpret_cast<double2 *>(dst + 128 + 2 * lane) = make_double2(t[2], t[3]);
}
__device__ __forceinline__ f64x4 get_tile(const double *src, int lane) {
  const double2 a = *reinterpret_cast<const double2 *>(src + 2 * lane);
  const double2 b = *reinterpret_cast<const double2 *>(src + 128 + 2 * lane);
  return f64x4{a.x, a.y, b.x, b.y};
}

// acc +- A B over one 16-deep step of tiles
__device__ __forceinline__ f64x4 tile_fma(const f64x4 &a, const f64x4 &b, f64x4 acc) {
#pragma unroll
  for (int v = 0; v < 4; ++v) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[v], b[v], acc, 0, 0, 0);
  return acc;
}
__device__ __forceinline__ f64x4 tile_fms(const f64x4 &a, const f64x4 &b, f64x4 acc) {
#pragma unroll
  for (int v = 0; v < 4; ++v) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[v], b[v], acc, 0, 0, 0);
  return acc;
}

// lane K of each 16-lane row, to the whole row
template <int K>
__device__ __forceinline__ double row_bcast(double x) {
  return __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, __double_as_longlong(x), 0x150 + K, 0xf, 0xf, true));
}

// 1 / sqrt(d): the hardware estimate and one third-order step,
// y (1 + e/2 + 3 e^2 / 8) with e = 1 - d y^2.  An infinite d counts as the
// largest number, whose root is as good as infinite.
__device__ __forceinline__ double rsqrt_full(double d) {
  const double c = fmin(d, 1.7976931348623157e308);
  const double y = __builtin_amdgcn_rsq(c);
  const double e = fma(-c * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// acc[J + q] += (lane J + q of the 16-lane row of x) * m for q < N, one
// instruction each (the compiler would move the broadcast to a register first,
// which doubles the instructions).  A broadcast may not read a register within
// two issue slots of its write: a block opens with that wait, and leaves as
// much behind the first register that it writes, the next pivot's.
#define WLC_BCAST(q) "v_fmac_f64_dpp %[a" #q "], %[x], %[m] row_newbcast:%[j" #q "] row_mask:0xf bank_mask:0xf\n\t"
template <int J, int N>
__device__ __forceinline__ void fmac_cols(double *a, double x, double m) {
  if constexpr (N >= 8) {
    asm("s_nop 1\n\t" WLC_BCAST(0) WLC_BCAST(1) WLC_BCAST(2) WLC_BCAST(3) WLC_BCAST(4) WLC_BCAST(5) WLC_BCAST(6)
            WLC_BCAST(7)
        : [a0] "+v"(a[J]), [a1] "+v"(a[J + 1]), [a2] "+v"(a[J + 2]), [a3] "+v"(a[J + 3]), [a4] "+v"(a[J + 4]),
          [a5] "+v"(a[J + 5]), [a6] "+v"(a[J + 6]), [a7] "+v"(a[J + 7])
        : [x] "v"(x), [m] "v"(m), [j0] "n"(J), [j1] "n"(J + 1), [j2] "n"(J + 2), [j3] "n"(J + 3), [j4] "n"(J + 4),
          [j5] "n"(J + 5), [j6] "n"(J + 6), [j7] "n"(J + 7));
    fmac_cols<J + 8, N - 8>(a, x, m);
  } else if constexpr (N >= 4) {
    asm("s_nop 1\n\t" WLC_BCAST(0) WLC_BCAST(1) WLC_BCAST(2) WLC_BCAST(3)
        : [a0] "+v"(a[J]), [a1] "+v"(a[J + 1]), [a2] "+v"(a[J + 2]), [a3] "+v"(a[J + 3])
        : [x] "v"(x), [m] "v"(m), [j0] "n"(J), [j1] "n"(J + 1), [j2] "n"(J + 2), [j3] "n"(J + 3));
    fmac_cols<J + 4, N - 4>(a, x, m);
  } else if constexpr (N == 3) {
    asm("s_nop 1\n\t" WLC_BCAST(0) WLC_BCAST(1) WLC_BCAST(2)
        : [a0] "+v"(a[J]), [a1] "+v"(a[J + 1]), [a2] "+v"(a[J + 2])
        : [x] "v"(x), [m] "v"(m), [j0] "n"(J), [j1] "n"(J + 1), [j2] "n"(J + 2));
  } else if constexpr (N == 2) {
    asm("s_nop 1\n\t" WLC_BCAST(0) WLC_BCAST(1) "s_nop 0"
        : [a0] "+v"(a[J]), [a1] "+v"(a[J + 1])
        : [x] "v"(x), [m] "v"(m), [j0] "n"(J), [j1] "n"(J + 1));
  } else if constexpr (N == 1) {
    asm("s_nop 1\n\t" WLC_BCAST(0) "s_nop 1" : [a0] "+v"(a[J]) : [x] "v"(x), [m] "v"(m), [j0] "n"(J));
  }
}
#undef WLC_BCAST
// x[v] += (lane K of the row of x[v]) * m for v <= K / 4: row K of V is zero
// right of its diagonal
#define WLC_BCAST(v) "v_fmac_f64_dpp %[x" #v "], %[x" #v "], %[m] row_newbcast:%[k] row_mask:0xf bank_mask:0xf\n\t"
template <int K>
__device__ __forceinline__ void fmac_rows(double (&x)[4], double m) {
  if constexpr (K < 4)
    asm("s_nop 1\n\t" WLC_BCAST(0) "s_nop 1" : [x0] "+v"(x[0]) : [m] "v"(m), [k] "n"(K));
  else if constexpr (K < 8)
    asm("s_nop 1\n\t" WLC_BCAST(0) WLC_BCAST(1) "s_nop 1"
        : [x0] "+v"(x[0]), [x1] "+v"(x[1])
        : [m] "v"(m), [k] "n"(K));
  else if constexpr (K < 12)
    asm("s_nop 1\n\t" WLC_BCAST(0) WLC_BCAST(1) WLC_BCAST(2) "s_nop 1"
        : [x0] "+v"(x[0]), [x1] "+v"(x[1]), [x2] "+v"(x[2])
        : [m] "v"(m), [k] "n"(K));
  else
    asm("s_nop 1\n\t" WLC_BCAST(0) WLC_BCAST(1) WLC_BCAST(2) WLC_BCAST(3) "s_nop 1"
        : [x0] "+v"(x[0]), [x1] "+v"(x[1]), [x2] "+v"(x[2]), [x3] "+v"(x[3])
        : [m] "v"(m), [k] "n"(K));
}
#undef WLC_BCAST

// Column K of a 16 x 16 factorisation A = L L^T: lane 16 g + r of every group g
// holds row r (a[c] = A[r][c]; entries right of the diagonal take harmless
// updates that are never read) and the columns g + 4 v of row r of V, L^-1
// but for the scaling of its rows, by forward substitution in the same pass
// (V = I at the start); own collects row r's pivot.  The pivot and the column's
// entries reach the lanes by row broadcasts, so a column is one chain of
// registers: broadcast, 1 / sqrt, scale, update.  What follows from a pivot
// that is not positive is not used.
template <int K>
__device__ __forceinline__ void factor_col(double (&a)[RB], double (&x)[4], double &own, int r) {
  const double d = row_bcast<K>(a[K]);
  const double y = rsqrt_full(d);
  a[K] *= y;
  fmac_cols<K + 1, RB - 1 - K>(a, a[K], -a[K]);
  own = r == K ? d : own;
  if constexpr (K + 1 < RB) {
    fmac_rows<K>(x, (r > K ? -a[K] : 0.0) * y);
    factor_col<K + 1>(a, x, own, r);
  }
}

// Factor the diagonal tile t by one wavefront.  row[] = row r of L (junk right
// of the diagonal), the result L^-1 in tile layout.  sh: 16 x 18 doubles of
// this wavefront's own.
__device__ __forceinline__ f64x4 factor_tile(const f64x4 &t, double *sh, int lane, double (&row)[RB], bool &bad) {
  const int r = lane & 15, g = lane >> 4;
  constexpr int P = RB + 2;
#pragma unroll
  for (int v = 0; v < 4; ++v) sh[r * P + g + 4 * v] = t[v];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (int q = 0; q < RB / 2; ++q) {
    const double2 w = *reinterpret_cast<const double2 *>(&sh[r * P + 2 * q]);
    row[2 * q] = w.x;
    row[2 * q + 1] = w.y;
  }
  double x[4], own = 1.0;
#pragma unroll
  for (int v = 0; v < 4; ++v) x[v] = r == g + 4 * v ? 1.0 : 0.0;
  factor_col<0>(row, x, own, r);
  // the rows are complete here: later selections among them must not pull the
  // arithmetic that makes them behind branches of their own
#pragma unroll
  for (int c = 0; c < RB; ++c) asm volatile("" : "+v"(row[c]));
  bad |= !(own > 0.0);
  const double ys = rsqrt_full(own);
  return f64x4{x[0] * ys, x[1] * ys, x[2] * ys, x[3] * ys};
}

// A 128 x 128 diagonal block: the 36 tiles of its lower triangle at diag_at,
// first as the matrix has them and in the end as L (off the diagonal packed; on
// it rows with their 16-byte chunks exchanged by diag_row), the inverse of the
// current diagonal tile, and a scratch row block.
struct DiagLds {
  double tile[PACK_DIAG];
  double inv[TILE];
  double row[RB * (RB + 2)];
};
__device__ __forceinline__ int diag_row(int r, int c) { return r * RB + 2 * ((c >> 1) ^ (r & 7)) + (c & 1); }
// place of (row r, column c) of a tile in its packed form
__device__ __forceinline__ int packed_at(int r, int c) { return (c >> 3) * 128 + 2 * (16 * (c & 3) + r) + ((c >> 2) & 1); }

// The row blocks of wavefront W: 1 and 0 for the one that walks down the
// diagonal, (7, 2), (6, 3), (5, 4) for the others, which have the same number of
// tiles to update at every column (9, 7, 5, ... in all).
template <int W>
struct DiagRows {
  static constexpr int R0 = W == 0 ? 1 : NT - W, R1 = W == 0 ? 0 : W + 1;
  f64x4 a[R0 + 1], b[R1 + 1];
};

// Start the copies of row block rb (column blocks 0 .. rb) of the jb x jb block
// at j0 straight into LDS, eight rows of 128 B each, in the order of diag_row:
// lane l copies row l / 8 and the 16-byte chunk that belongs into its slot.
// The descriptor ends at the block's last row, and columns are clamped to it:
// rows and columns from jb on hold something or zero.
template <int RBK>
__device__ __forceinline__ void diag_copy(DiagLds &S, const double *__restrict__ Wm, int64_t ld, int64_t j0, int jb,
                                          int lane) {
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(Wm + j0 * ld + j0), 0, (int)(((jb - 1) * ld + ((jb + 1) & ~1)) * 8), 0x00020000);
#pragma unroll
  for (int t = 0; t <= RBK; ++t)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = 8 * h + (lane >> 3);
      const int c = min(t * RB + 2 * ((lane & 7) ^ (r & 7)), (jb - 1) & ~1);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, (__attribute__((address_space(3))) void *)(S.tile + diag_at(RBK, t) + h * 8 * RB), 16,
          (uint32_t)(((RBK * RB + r) * ld + c) * 8), 0, 0, 0);
    }
}

// The row block as diag_copy left it: the mirror image above the diagonal, the
// identity from jb on.
template <int RBK>
__device__ __forceinline__ void diag_get(const DiagLds &S, int jb, int lane, f64x4 (&acc)[RBK + 1]) {
  const int r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int t = 0; t <= RBK; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int c = g + 4 * v, i = RBK * RB + r, j = t * RB + c;
      const int hi = t == RBK ? max(r, c) : r, lo = t == RBK ? min(r, c) : c;
      const double x = S.tile[diag_at(RBK, t) + diag_row(hi, lo)];
      acc[t][v] = max(i, j) < jb ? x : i == j ? 1.0 : 0.0;
    }
}

// Barrier over LDS alone: global stores stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// A wavefront's row blocks of the diagonal block at r0.
template <int W>
__device__ __forceinline__ void diag_load(DiagLds &S, const double *__restrict__ Wm, int64_t ld, int64_t r0, int jb,
                                          int lane, DiagRows<W> &T) {
  constexpr int R0 = DiagRows<W>::R0, R1 = DiagRows<W>::R1;
  diag_copy<R0>(S, Wm, ld, r0, jb, lane);
  diag_copy<R1>(S, Wm, ld, r0, jb, lane);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's copies
  diag_get<R0>(S, jb, lane, T.a);
  diag_get<R1>(S, jb, lane, T.b);
}

// Factorisation of a diagonal block, right-looking over its eight column blocks.
// Wavefront 0 walks down the diagonal: it factors and inverts tile (j, j), then
// multiplies tile (j + 1, j) by the inverse and updates tile (j + 1, j + 1),
// while the others, their tiles in registers, apply column j - 1, hand tiles
// (j + 1, j) and (j + 1, j + 1) over, and multiply their tiles of column j by the
// inverse.  Two barriers per column.
//
// Bound by wavefront 0's chain of 128 pivots (broadcast, estimate and
// refinement of 1 / sqrt, scaling, the next column's update: 160 cycles each)
// and the eight hand-overs between tiles (1600 cycles each): 17 us, where a
// workgroup-wide 64 x 64 factorisation with one barrier per column took 28 us
// and had to run twice.  Its loop is not unrolled, so that one copy of the code,
// still in the instruction cache, runs all eight columns.  A narrow last panel
// stops after its last tile: 15 columns take
// 3 us, and the whole launch 10 instead of 32.
__device__ __forceinline__ void diag_walk(DiagLds &S, const DiagRows<0> &T, int jb, int lane, double *__restrict__ pack,
                                          int *__restrict__ flag) {
  const int r = lane & 15, g = lane >> 4;
  const f64x4 z = f64x4{0.0, 0.0, 0.0, 0.0};
  bool bad = false;
  put_tile(S.tile + diag_at(1, 0), lane, T.a[0]);
  put_tile(S.tile + diag_at(1, 1), lane, T.a[1]);
  f64x4 next = T.b[0];
#pragma unroll 1
  for (int j = 0; j * RB < jb; ++j) {
    double row[RB];
    const f64x4 inv = factor_tile(next, S.row, lane, row, bad);
    put_tile(S.inv, lane, inv);
    put_tile(pack + diag_at(j, j), lane, inv);
    lds_barrier();
    const int j1 = min(j + 1, NT - 1);
    double *dst = S.tile + diag_at(j1, j), *own = S.tile + diag_at(j, j);
    const f64x4 t = get_tile(S.tile + diag_at(j1, j1), lane), b = get_tile(dst, lane);
    const f64x4 x = tile_fma(inv, b, z);
    // the rows of the diagonal tile go to LDS under the products, four columns
    // from each lane group
    double o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double c0 = row[q], c1 = row[4 + q], c2 = row[8 + q], c3 = row[12 + q];
      const double lo = g & 1 ? c1 : c0, hi = g & 1 ? c3 : c2;
      o[q] = g & 2 ? hi : lo;
    }
    *reinterpret_cast<double2 *>(own + diag_row(r, 4 * g)) = make_double2(o[0], o[1]);
    *reinterpret_cast<double2 *>(own + diag_row(r, 4 * g + 2)) = make_double2(o[2], o[3]);
    if (j + 1 < NT) put_tile(dst, lane, x);
    next = tile_fms(x, x, t);
    lds_barrier();
  }
  if (bad) atomicOr(flag, 1);
}

template <int W>
__device__ __forceinline__ void diag_follow(DiagLds &S, DiagRows<W> &T, int jb, int lane) {
  constexpr int R0 = DiagRows<W>::R0, R1 = DiagRows<W>::R1;  // R0 > R1
  const f64x4 z = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    if (j * RB >= jb) break;
    if (j > 0) {
      // column j - 1, but for tile (j, j), which wavefront 0 has
#pragma unroll
      for (int t = j; t <= R0; ++t) {
        if (R0 > j) {
          const f64x4 l = t == R0 ? T.a[j - 1] : get_tile(S.tile + diag_at(t, j - 1), lane);
          T.a[t] = tile_fms(l, T.a[j - 1], T.a[t]);
          if (R1 > j && t <= R1) T.b[t] = tile_fms(l, T.b[j - 1 < R1 ? j - 1 : 0], T.b[t <= R1 ? t : 0]);
        }
      }
    }
    if (R0 == j + 1) {
      put_tile(S.tile + diag_at(R0, R0 - 1), lane, T.a[R0 - 1]);
      put_tile(S.tile + diag_at(R0, R0), lane, T.a[R0]);
    }
    if (R1 == j + 1) {
      put_tile(S.tile + diag_at(R1, R1 - 1), lane, T.b[R1 - 1]);
      put_tile(S.tile + diag_at(R1, R1), lane, T.b[R1]);
    }
    lds_barrier();
    if (R0 > j + 1) {
      const f64x4 inv = get_tile(S.inv, lane);
      T.a[j < R0 ? j : 0] = tile_fma(inv, T.a[j < R0 ? j : 0], z);
      put_tile(S.tile + diag_at(R0, j < R0 ? j : 0), lane, T.a[j < R0 ? j : 0]);
      if (R1 > j + 1) {
        T.b[j < R1 ? j : 0] = tile_fma(inv, T.b[j < R1 ? j : 0], z);
        put_tile(S.tile + diag_at(R1, j < R1 ? j : 0), lane, T.b[j < R1 ? j : 0]);
      }
    }
    lds_barrier();
  }
}

__device__ __forceinline__ void diag_block(DiagLds &S, double *__restrict__ Wm, int64_t ld, int64_t j0, int jb, int w,
                                           int lane, double *__restrict__ pack,
                                           int *__restrict__ flag) {
  if (w == 0) {
    DiagRows<0> T;
    diag_load<0>(S, Wm, ld, j0, jb, lane, T);
    diag_walk(S, T, jb, lane, pack, flag);
  } else if (w == 1) {
    DiagRows<1> T;
    diag_load<1>(S, Wm, ld, j0, jb, lane, T);
    diag_follow<1>(S, T, jb, lane);
  } else if (w == 2) {
    DiagRows<2> T;
    diag_load<2>(S, Wm, ld, j0, jb, lane, T);
    diag_follow<2>(S, T, jb, lane);
  } else {
    DiagRows<3> T;
    diag_load<3>(S, Wm, ld, j0, jb, lane, T);
    diag_follow<3>(S, T, jb, lane);
  }
  // L to the matrix, eight rows of 128 B per store, and its tiles off the
  // diagonal, packed, to pack: nine tiles per wavefront
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const int rb = q <= w ? w : NT - 1 - w, t = q <= w ? q : q - w - 1;
    const double *src = S.tile + diag_at(rb, t);
    if (t < rb) put_tile(pack + diag_at(rb, t), lane, get_tile(src, lane));
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = 8 * h + (lane >> 3), c = 2 * (lane & 7), i = rb * RB + r, j = t * RB + c;
      double2 o;
      if (t < rb) {
        o = make_double2(src[packed_at(r, c)], src[packed_at(r, c + 1)]);
      } else {
        o = *reinterpret_cast<const double2 *>(src + diag_row(r, c));
      }
      // a pair may reach one column past the diagonal or the block: that entry
      // of the row is above the diagonal and never read
      if (i < jb && j <= i) *reinterpret_cast<double2 *>(Wm + (j0 + i) * ld + j0 + j) = o;
    }
  }
}

__global__ __launch_bounds__(256) void k_diag(double *__restrict__ Wm, int64_t ld, int64_t j0, int jb,
                                              double *__restrict__ pack, int *__restrict__ flag) {
  __shared__ __attribute__((aligned(16))) DiagLds S;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  diag_block(S, Wm, ld, j0, jb, w, lane, pack, flag);
}

// Panel solve X = B L^-T of the rows below a diagonal block: 64 rows per
// workgroup, 16 per wavefront, forward substitution over the eight column
// blocks entirely in registers.  The packed diagonal block (72 KB) and the rows
// themselves (1 KB per row and load, 16 KB per wavefront) are copied straight
// into LDS, the 16-byte chunk c of row r at slot c ^ r, from where the tiles
// are read free of bank conflicts; X goes back the same way.  X goes to the
// matrix and, packed, to rows_pack for the trailing update.
//
// Bound at up to 256 workgroups by its start: launch, 136 KB into each CU's LDS
// and one wavefront's 144 products (4 us): 9.2 us at 800 rows, 9.6 at 4500 (15.8
// with 8-byte gathers of 16 rows a load; 10.1 and 10.9 with each column's tiles
// read when their turn comes and X's rows read one by one).  Tiles straight from
// the L2, eight ahead, took 10.8 and 11.3.
// FULL: the panel has all its 128 columns, and a column of tiles is read while
// the one before is multiplied.
template <bool FULL>
__global__ __launch_bounds__(256) void k_solve(double *__restrict__ Wm, int64_t ld, int64_t j0, int jb, int64_t rows,
                                               const double *__restrict__ pack, double *__restrict__ rows_pack) {
  __shared__ __attribute__((aligned(16))) double lp[PACK_DIAG];
  __shared__ __attribute__((aligned(16))) double lb[4 * RB * NB];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int64_t blk = (int64_t)blockIdx.x * 4 + w;  // 16-row block below the diagonal block
  const int64_t i0 = j0 + jb + blk * RB;
  double *B = Wm + i0 * ld + j0, *sb = lb + w * RB * NB;
  // rows past the matrix read as zero: the descriptor ends at the last one
  const int64_t nr = min((int64_t)RB, rows - i0);
  const __amdgpu_buffer_rsrc_t rb =
      __builtin_amdgcn_make_buffer_rsrc((void *)B, 0, nr > 0 ? (int)(((nr - 1) * ld + min((int64_t)NB, ld - j0)) * 8) : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void *)pack, 0, PACK_DIAG * 8, 0x00020000);
#pragma unroll
  for (int q = 0; q < RB; ++q)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (__attribute__((address_space(3))) void *)(sb + q * NB), 16,
                                             (uint32_t)(q * ld * 8 + 16 * (lane ^ q)), 0, 0, 0);
#pragma unroll
  for (int q = 0; q < PACK_DIAG / 512; ++q)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rp, (__attribute__((address_space(3))) void *)(lp + (q * 4 + w) * 128),
                                             16, (uint32_t)(((q * 4 + w) * 128 + 2 * lane) * 8), 0, 0, 0);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's copies into LDS
  __syncthreads();
  f64x4 T[NT];
  const int at = r * NB + (g & 1);
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double x = sb[at + 2 * ((8 * t + 2 * v + (g >> 1)) ^ r)];
      T[t][v] = FULL || t * RB + g + 4 * v < jb ? x : 0.0;
    }
  f64x4 L[2][NT];
  auto fetch = [&](int j) {
#pragma unroll
    for (int t = j; t < NT; ++t) L[j & 1][t] = get_tile(lp + diag_at(t, j), lane);
  };
  fetch(0);
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    if (!FULL && j * RB >= jb) break;
    if (j + 1 < NT) fetch(j + 1);
    __builtin_amdgcn_sched_barrier(0);
    T[j] = tile_fma(L[j & 1][j], T[j], f64x4{0.0, 0.0, 0.0, 0.0});
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int t = j + 1; t < NT; ++t)
        T[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-L[j & 1][t][v], T[j][v], T[t], 0, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
#pragma unroll
    for (int v = 0; v < 4; ++v) sb[at + 2 * ((8 * t + 2 * v + (g >> 1)) ^ r)] = T[t][v];
    if (rows_pack) put_tile(rows_pack + blk * PACK_ROW + t * TILE, lane, T[t]);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // an odd jb lets a pair reach one column past the block: the corner entry of
  // the bordered matrix, which nothing reads
  auto row = [&](int q) { return *reinterpret_cast<const double2 *>(sb + q * NB + 2 * (lane ^ q)); };
  if (FULL && nr == RB) {  // all reads in flight together
    double2 out[RB];
#pragma unroll
    for (int q = 0; q < RB; ++q) out[q] = row(q);
#pragma unroll
    for (int q = 0; q < RB; ++q) *reinterpret_cast<double2 *>(B + q * ld + 2 * lane) = out[q];
  } else {
#pragma unroll
    for (int q = 0; q < RB; ++q)
      if (q < nr && 2 * lane < jb) *reinterpret_cast<double2 *>(B + q * ld + 2 * lane) = row(q);
  }
}

// The packed rows of the solved panels: panel q (its first row below is
// 128 (q + 1)) in slot q % slots; panel `last` has just been solved.
struct Panels {
  const double *base;
  int64_t stride;
  int slots, last;
  // 16-row block ab of the matrix in panel q
  __device__ __forceinline__ const double *block(int q, int64_t ab) const {
    return base + (q % slots) * stride + (ab - (int64_t)NT * (q + 1)) * PACK_ROW;
  }
};

// Trailing update W[i][j] -= sum_k X[i][k] X[j][k], i >= j, after panel p has been
// solved, r0 its first row below:
//  - the diagonal block at r0 with panel p: the first nine workgroups, a 16 x 16
//    tile per wavefront; the one that is done last (none waits) factors it, so
//    that the factorisation's serial chain runs beside the rest;
//  - columns r0 + 128 (1 + m B), m = 0, 1, ..., 128 each, with panels
//    p - B + 1 .. p: each column block is read and written once per B
//    panels, a B-th of them in every launch, and has received every panel but the
//    last when its turn comes;
//  - the rest of columns r0 .. r0 + 127 with panel p.
// A workgroup takes a tile of 32 S rows and columns (four wavefronts, each S x S
// tiles of 16), operands straight from the L2 into registers (every load of a
// wavefront is 1 KB, half a 16-deep step ahead), no LDS and no barrier.
//
// While the update is small the chain sets the time (24 us, 17 of them the
// factorisation; with one workgroup for update and factorisation of the block
// 31); then the matrix cores, and the reads and writes of W (16 bytes per 256 B
// flops).
constexpr int DIAG_WG = NT * (NT + 1) / 2 / 4;
// the counter of the diagonal block's workgroups, in ints past the pivot flag
constexpr int DIAG_COUNT = 16;

// A wavefront's 16 x 16 tile (ib, jb0) of the diagonal block at r0, own rows.
__device__ __forceinline__ void trail_diag_tile(double *__restrict__ Wm, int64_t ld, int64_t r0, int own,
                                                const Panels &X, int first, int ib, int jb0, int lane) {
  const int r = lane & 15, g = lane >> 4;
  double *dst = Wm + r0 * ld + r0;
  f64x4 acc[2];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = min(ib * RB + g + 4 * v, own - 1), j = min(jb0 * RB + r, i);
    acc[0][v] = dst[i * ld + j];
    acc[1][v] = 0.0;
  }
#pragma unroll 1
  for (int k = first; k <= X.last; ++k) {
    const double *pa = X.block(k, r0 / RB + ib) + 2 * lane, *pb = X.block(k, r0 / RB + jb0) + 2 * lane;
    double2 a[2 * NT], b[2 * NT];  // a panel at once: the loads' latency is what this waits for
#pragma unroll
    for (int st = 0; st < 2 * NT; ++st) {
      a[st] = *reinterpret_cast<const double2 *>(pa + st * 128);
      b[st] = *reinterpret_cast<const double2 *>(pb + st * 128);
    }
#pragma unroll
    for (int st = 0; st < 2 * NT; ++st) {
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[st].x, b[st].x, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[st].y, b[st].y, acc[1], 0, 0, 0);
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = ib * RB + g + 4 * v, j = jb0 * RB + r;
    if (i < own && j <= i) dst[i * ld + j] = acc[0][v] + acc[1][v];
  }
}

// U.batch: tiles of the column blocks that are U.gap apart (t0 rows of tiles in
// the first of them), with panels U.first .. X.last; the diagonal block and the
// rest of its columns take panels U.now .. X.last
struct Update {
  int first, now, gap, batch, t0;
};
template <int S>
__global__ __launch_bounds__(256, 2) void k_trail(double *__restrict__ Wm, int64_t ld, int64_t r0, int64_t rows,
                                                  int64_t c1, Panels X, Update U, double *__restrict__ pack,
                                                  int *__restrict__ flag) {
  __shared__ __attribute__((aligned(16))) DiagLds D;
  __shared__ int done;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int64_t own = min((int64_t)NB, c1 - r0);  // rows of the next diagonal block
  if (blockIdx.x < DIAG_WG) {
    const int t = blockIdx.x * 4 + w;
    int ib = 0;
    while ((ib + 1) * (ib + 2) / 2 <= t) ++ib;
    if (ib * RB < own) trail_diag_tile(Wm, ld, r0, (int)own, X, U.now, ib, t - ib * (ib + 1) / 2, lane);
    // the tiles are visible to the device before the count says so
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if (threadIdx.x == 0) done = atomicAdd(flag + DIAG_COUNT, 1);
    __syncthreads();
    if (done != DIAG_WG - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (threadIdx.x == 0) flag[DIAG_COUNT] = 0;  // for the next launch
    diag_block(D, Wm, ld, r0, (int)own, w, lane, pack, flag);
    return;
  }
  constexpr int CT = NT / (2 * S);  // tiles across a column block
  int q = blockIdx.x - DIAG_WG;
  int64_t ib, jb0;  // the workgroup's first 16-blocks
  int first = U.now;
  if (q < U.batch) {  // column block m: CT tiles by t0 - m CT gap rows of them
    const int step = CT * U.gap, t0 = U.t0, k = q / CT;
    const double h = t0 + 0.5 * step;
    int m = (int)((h - sqrt(max(h * h - 2.0 * step * k, 0.0))) / step);
    while (m > 0 && m * t0 - step * (m * (m - 1) / 2) > k) --m;
    while ((m + 1) * t0 - step * ((m + 1) * m / 2) <= k) ++m;
    const int64_t c = r0 / RB + NT * (1 + (int64_t)m * U.gap);
    ib = c + (int64_t)(k - (m * t0 - step * (m * (m - 1) / 2))) * 2 * S;
    jb0 = c + (q % CT) * 2 * S;
    first = U.first;
  } else {
    q -= U.batch;
    ib = (r0 + own) / RB + (int64_t)(q / CT) * 2 * S;
    jb0 = r0 / RB + (q % CT) * 2 * S;
  }
  ib += (w >> 1) * S;
  jb0 += (w & 1) * S;
  const int64_t ilim = (rows + RB - 1) / RB;
  // whole wavefront outside the matrix or above the diagonal
  if (ib >= ilim || jb0 * RB >= c1 || jb0 > ib + S - 1) return;
  int64_t pa[S], pb[S];  // row blocks in a panel's packed rows
  const double *p = X.block(first, 0) + 2 * lane;
#pragma unroll
  for (int x = 0; x < S; ++x) {
    pa[x] = min(ib + x, ilim - 1) * PACK_ROW;
    pb[x] = min(jb0 + x, ilim - 1) * PACK_ROW;
  }
  // accumulator of rows x columns: element v of lane l is row g + 4 v, column
  // l % 16
  f64x4 acc[S][S];
#pragma unroll
  for (int x = 0; x < S; ++x)
#pragma unroll
    for (int y = 0; y < S; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t i = min((ib + x) * RB + g + 4 * v, rows - 1);
        const int64_t j = min((jb0 + y) * RB + r, c1 - 1);
        acc[x][y][v] = Wm[i * ld + min(i, j)];
      }
  double2 a[2][S], b[2][S];
  // half step st of the panel at p: two of the four products of a 16-deep step
  auto load = [&](int h, const double *p, int st) {
#pragma unroll
    for (int x = 0; x < S; ++x) {
      a[h][x] = *reinterpret_cast<const double2 *>(p + st * 128 + pa[x]);
      b[h][x] = *reinterpret_cast<const double2 *>(p + st * 128 + pb[x]);
    }
  };
  auto mul = [&](int h) {
#pragma unroll
    for (int x = 0; x < S; ++x)
#pragma unroll
      for (int y = 0; y < S; ++y)
        acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[h][x].x, b[h][y].x, acc[x][y], 0, 0, 0);
#pragma unroll
    for (int x = 0; x < S; ++x)
#pragma unroll
      for (int y = 0; y < S; ++y)
        acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[h][x].y, b[h][y].y, acc[x][y], 0, 0, 0);
  };
  load(0, p, 0);
#pragma unroll 1
  for (int k = first; k <= X.last; ++k) {
    const double *next = k < X.last ? X.block(k + 1, 0) + 2 * lane : p;
#pragma unroll
    for (int st = 0; st < 2 * NT; st += 2) {
      load(1, p, st + 1);
      mul(0);
      load(0, st + 2 < 2 * NT ? p : next, (st + 2) % (2 * NT));
      mul(1);
    }
    p = next;
  }
#pragma unroll
  for (int x = 0; x < S; ++x)
#pragma unroll
    for (int y = 0; y < S; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t i = (ib + x) * RB + g + 4 * v;
        const int64_t j = (jb0 + y) * RB + r;
        // (rows before r0 + own are the diagonal block's, or another column block's own)
        if (i < rows && j < c1 && i >= j && i >= r0 + own) Wm[i * ld + j] = acc[x][y][v];
      }
}

// The updates due after panel X.last, first row below r0, columns up to c1, and
// the factorisation of the next diagonal block.
static void launch_trail(double *Wm, int64_t ld, int64_t r0, int64_t rows, int64_t c1, const Panels &X, Update U,
                         double *pack, int *flag, hipStream_t s, KernelProbe *probe) {
  const bool timed = probe && probe->ev && probe->count < probe->cap;
  const int64_t own = std::min<int64_t>(NB, c1 - r0);
  if (probe) {
    auto entries = [&](int64_t c, int64_t cols) { return (double)cols * (double)(rows - c) - (double)cols * (cols - 1) / 2.0; };
    double f = (X.last - U.now + 1) * entries(r0, own);
    for (int64_t c = r0 + NB; c < c1; c += NB * U.gap)
      f += (X.last - U.first + 1) * entries(c, std::min<int64_t>(NB, c1 - c));
    probe->flops += 2.0 * NB * f;
    ++probe->launches;
  }
  // the batch in t x t tiles
  auto batch_of = [&](int64_t t) {
    int64_t k = c1 > r0 + NB ? (rows - r0 - NB + t - 1) / t : 0, n = 0;
    U.t0 = (int)k;
    for (int64_t c = r0 + NB; c < c1; c += NB * U.gap, k -= NB / t * U.gap) n += k * (NB / t);
    U.batch = (int)n;
    return n;
  };
  auto grid = [&](int64_t t) {
    return dim3((unsigned)(DIAG_WG + U.batch + (rows - (r0 + own) / RB * RB + t - 1) / t * (NB / t)));
  };
  if (timed) (void)hipEventRecord(probe->ev[2 * probe->count], s);
  // 64 x 64 tiles until 128 x 128 ones fill the chip one and a half times over
  // (two workgroups per CU): n = 10000 7.82 ms, from 400 tiles on 7.94
  if (batch_of(128) >= 768) {
    hipLaunchKernelGGL(k_trail<4>, grid(128), dim3(256), 0, s, Wm, ld, r0, rows, c1, X, U, pack, flag);
  } else {
    batch_of(64);
    hipLaunchKernelGGL(k_trail<2>, grid(64), dim3(256), 0, s, Wm, ld, r0, rows, c1, X, U, pack, flag);
  }
  if (timed) (void)hipEventRecord(probe->ev[2 * probe->count++ + 1], s);
}

// Panels whose packed rows lie in the scratch, of GROUP that can be used: one up to
// 1008 rows, three up to 1520, five to 2032, seven to 2544, then eight, and fewer
// again past 131000 rows (seven to 149726, one from 524205).  Column blocks wait
// for GAP panels at most, fewer where fewer fit, and groups need more than GAP.
static int chol_slots(int64_t n) {
  const int64_t fit = ((int64_t)(chol_scratch_bytes(n) / 8) - PACK_DIAG) / ((n + 64) * NB);
  return (int)std::max<int64_t>(1, std::min<int64_t>(GROUP, fit));
}

// Factor columns [0, n) of M (n + 1 rows).  scratch: the packed diagonal block,
// then the packed rows of chol_slots(n) solved panels.  The pivot flag is checked by
// the caller after synchronisation.
int chol_factor(double *Wm, int64_t n, int64_t ld, double *scratch, int *flag, hipStream_t s,
                KernelProbe *probe) {
  const int64_t rows = n + 1, pack_rows = (n + 64) * NB;  // doubles of a panel's packed rows
  double *pack = scratch, *part = scratch + PACK_DIAG;
  const int slots = chol_slots(n);
  hipLaunchKernelGGL(k_diag, dim3(1), dim3(256), 0, s, Wm, ld, 0, (int)std::min<int64_t>(NB, n), pack, flag);
  Panels X{part, pack_rows, slots, 0};
  int begin = 0;     // the panels before this one have reached every column
  int64_t gend = n;  // columns from here on wait for the end of the group
  for (int64_t j0 = 0; j0 < n; j0 += NB, ++X.last) {
    const int jb = (int)std::min<int64_t>(NB, n - j0);
    const int64_t r0 = j0 + jb;  // first row below
    if (begin == X.last && slots > GAP && n - j0 >= GROUP_MIN) gend = j0 + slots * NB;
    const dim3 grid((unsigned)((rows - r0 + 63) / 64));
    double *solved = r0 < n ? part + X.last % slots * pack_rows : nullptr;
    if (jb == NB)
      hipLaunchKernelGGL(k_solve<true>, grid, dim3(256), 0, s, Wm, ld, j0, jb, rows, pack, solved);
    else
      hipLaunchKernelGGL(k_solve<false>, grid, dim3(256), 0, s, Wm, ld, j0, jb, rows, pack, solved);
    if (r0 >= n) break;
    Update U{};
    U.now = X.last;
    U.gap = std::min(GAP, slots);
    U.first = std::max(begin, X.last - U.gap + 1);
    int64_t c1 = gend;
    if (r0 == gend) {  // the end of a group: its panels to all the columns it left
      U.now = U.first = begin;
      U.gap = 1;
      c1 = gend = n;
      begin = X.last + 1;
    }
    launch_trail(Wm, ld, r0, rows, c1, X, U, pack, flag, s, probe);
  }
  return 0;
}

// Scratch, the size that callers know from the workspace queries and that sets
// where wlc_snr2_noalloc ends (2424 rows at ten ell-bins): 32 KB, and 256 doubles
// for each of the n + 1 rows and each whole 512 rows of n, at least once and at
// most 64 times (1 GB in all); or one panel and the packed diagonal block, if
// that is more.  chol_slots takes what fits.
size_t chol_scratch_bytes(int64_t n) {
  const int64_t times = std::clamp<int64_t>((n + 15) / 16 / 32, 1, 64);
  const size_t rows = (size_t)64 * 64 * 8 + (size_t)std::min<int64_t>(524288, times * (n + 1)) * 256 * 8;
  const size_t panel = (size_t)PACK_DIAG * 8 + (n > NB ? (size_t)(n + 64) * NB * 8 : 0);
  return std::max(rows, panel);
}

// ------------------------------------------------------------- y^T y
__global__ void k_sumsq_row(const double *__restrict__ Wm, int64_t n, int64_t ld, double *__restrict__ out) {
  __shared__ double part[256];
  const double *y = Wm + n * ld;
  double s = 0.0;
  for (int64_t j = threadIdx.x; j < n; j += 256) s += y[j] * y[j];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = part[0];
}

void launch_sumsq_row(const double *Wm, int64_t n, int64_t ld, double *out, hipStream_t s) {
  hipLaunchKernelGGL(k_sumsq_row, dim3(1), dim3(256), 0, s, Wm, n, ld, out);
}

// Prefix sums of y^2 (the last row of the bordered factor) at the group ends
// ends[0] <= ... <= ends[ng-1] = n: one block sums each group, then one
// thread accumulates the groups in order.
__global__ void k_sumsq_groups(const double *__restrict__ Wm, int64_t n, int64_t ld, const int32_t *__restrict__ ends,
                               double *__restrict__ part) {
  __shared__ double red[256];
  const int g = blockIdx.x;
  const int64_t lo = g == 0 ? 0 : ends[g - 1], hi = ends[g];
  const double *y = Wm + n * ld;
  double s = 0.0;
  for (int64_t j = lo + threadIdx.x; j < hi; j += 256) s += y[j] * y[j];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[g] = red[0];
}

__global__ void k_prefix(const double *__restrict__ part, int ng, double *__restrict__ out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double s = 0.0;
  for (int g = 0; g < ng; ++g) {
    s += part[g];
    out[g] = s;
  }
}

void launch_sumsq_groups(const double *Wm, int64_t n, int64_t ld, const int32_t *ends, int ng, double *part,
                         double *out, hipStream_t s) {
  hipLaunchKernelGGL(k_sumsq_groups, dim3((unsigned)ng), dim3(256), 0, s, Wm, n, ld, ends, part);
  hipLaunchKernelGGL(k_prefix, dim3(1), dim3(64), 0, s, part, ng, out);
}

}  // namespace wlc
