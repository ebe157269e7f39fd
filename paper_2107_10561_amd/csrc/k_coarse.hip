// The direct coarse solve of a member whose spatial rows fall into uncoupled
// blocks and a border.  With spatial factors (time-decoupled) one time block of
// the coarse operator, without them the whole matrix of scalar rows, is
//   [ V  B ]   V = blockdiag(V_1 .. V_nc): the velocity components, each cut
//   [ C  D ]   into parts by separators; border: the separators and the rows
//              without a diagonal entry (the pressure).
// The V_c are eliminated as one batch by the complex-pivot chain (k_dense.hip),
// then the Schur complement S = D - C V^-1 B by a second chain, and the solve
// is applied in factored form,
//   p = S^-1 (g - Z f),  Z = C V^-1,   u = V^-1 f + G p,  G = -V^-1 B
// (three launches), or with P = S^-1 [-Z | I] formed, p = P (f, g) (two), or,
// small or transposed, as the whole inverse of each time block,
//   [ V^-1 0 ; 0 0 ] + [ G ; I ] P   (one).
// The chains are bound by their panels in sequence, 16 complex pivots each: in
// 3d (16x3x3 cells) 32 for nine blocks of order 506 and 55 for a border of 870
// instead of 340 for the whole matrix of order 5,427 (138 for the components
// uncut), with fewer operations and 178 instead of 471 MB per apply; in 3d
// without factors (8x2x2 cells, order 2806) 55 instead of 176.  All
// matrices here are complex, row-major, in the member's order (blocks one
// after the other, then the border); entry x of a real form is
// [[Re, -Im], [Im, Re]].
#include "stv_internal.h"

namespace stv {

typedef double stv_d4 __attribute__((ext_vector_type(4)));

// complex value of block q of the time block p: t (m) + a, t = al - i be
__device__ __forceinline__ double2 cc_value(const CompCoarse& M, int p, int64_t q) {
  const double2 f = reinterpret_cast<const double2*>(M.ma)[q];
  return make_double2(fma(M.al[p], f.x, f.y), -M.be[p] * f.x);
}

// Entry e of an array that the solve reads (V^-1, G, P): a real number per
// entry for a real eigenvalue's block, a complex one for a pair's.
__device__ __forceinline__ double2 cc_get(const double2* a, int64_t e, bool pair) {
  return pair ? a[e] : make_double2(reinterpret_cast<const double*>(a)[e], 0.0);
}

__device__ __forceinline__ void cc_put(double2* a, int64_t e, bool pair, double2 v) {
  if (pair) a[e] = v;
  else reinterpret_cast<double*>(a)[e] = v.x;
}

__device__ __forceinline__ unsigned long long atomic_max_bits(unsigned long long* at, double v) {
  // non-negative doubles order as their bit patterns (a NaN above infinity)
  return atomicMax(at, __builtin_bit_cast(unsigned long long, v));
}

// The dense V_c and D in real form (the matrices zeroed before): member row
// blockIdx.x, time block blockIdx.y, member blockIdx.z; one wavefront per row.
// Only couplings inside a block and inside the border are written here.
__global__ void __launch_bounds__(64) k_cc_fill(const CompCoarse* __restrict__ cc) {
  const CompCoarse& M = cc[blockIdx.z];
  const int p = blockIdx.y, e = blockIdx.x;
  if (p == 0 && e == 0 && threadIdx.x < kCcProbeWords) M.probe_max[threadIdx.x] = 0ull;
  if (p >= M.nblk || e >= M.n_v + M.n_p) return;
  int c = 0;
  while (c < M.nc && e >= M.off[c] + M.n[c]) ++c;
  const bool border = c == M.nc;
  const int o = border ? M.n_v : M.off[c], n = border ? M.n_p : M.n[c], i = e - o;
  double* A = M.A[p][border ? kCcMax : c];
  const int64_t ld = M.lda[border ? kCcMax : c];
  const int32_t row = M.row_off + M.order[e];
  for (int32_t q = M.rowptr[row] + (int)threadIdx.x; q < M.rowptr[row + 1]; q += 64) {
    const int j = M.where[M.col[q] - M.row_off] - o;
    if (j < 0 || j >= n) continue;
    const double2 v = cc_value(M, p, q);
    *reinterpret_cast<double2*>(&A[2 * (int64_t)i * ld + 2 * j]) = make_double2(v.x, -v.y);
    *reinterpret_cast<double2*>(&A[(2 * (int64_t)i + 1) * ld + 2 * j]) = make_double2(v.y, v.x);
  }
}

// Inverse rows out of the eliminated real form, in natural order: row i is S's
// row rpiv[2i], column 2t belongs to j = rpiv[2t] / 2.  Nothing is read where
// the pivot record is not a permutation (verdict).
__device__ __forceinline__ void cc_collect(const double* A, int64_t ld, const int* rpiv, int n,
                                           int i, bool pair, double2* out) {
  const double* row = A + (int64_t)rpiv[2 * i] * ld;
  for (int t = threadIdx.x; t < n; t += 256) {
    const double2 e = *reinterpret_cast<const double2*>(row + 2 * (int64_t)t);
    cc_put(out, (int64_t)i * n + (rpiv[2 * t] >> 1), pair, make_double2(e.x, -e.y));
  }
}

__global__ void __launch_bounds__(256) k_cc_collect_v(const CompCoarse* __restrict__ cc, int nc) {
  const CompCoarse& M = cc[blockIdx.z];
  const int p = blockIdx.y / nc, c = blockIdx.y % nc, i = blockIdx.x;
  if (p >= M.nblk || c >= M.nc || i >= M.n[c] || *M.verdict[p][c]) return;
  cc_collect(M.A[p][c], M.lda[c], M.rpiv[p][c], M.n[c], i, M.sz[p] == 2, M.Vi[p][c]);
}

__global__ void __launch_bounds__(256) k_cc_collect_s(const CompCoarse* __restrict__ cc) {
  const CompCoarse& M = cc[blockIdx.z];
  const int p = blockIdx.y, m = blockIdx.x;
  if (p >= M.nblk || m >= M.n_p || *M.verdict[p][kCcMax]) return;
  cc_collect(M.A[p][kCcMax], M.lda[kCcMax], M.rpiv[p][kCcMax], M.n_p, m, true, M.Si[p]);
}

// Z = C V^-1, row m: the border row's entries in block c (listed at cptr) times
// the rows of V_c^-1 (coalesced over the columns).
__global__ void __launch_bounds__(256) k_cc_z(const CompCoarse* __restrict__ cc, int nc) {
  const CompCoarse& M = cc[blockIdx.z];
  const int p = blockIdx.y / nc, c = blockIdx.y % nc, m = blockIdx.x;
  if (p >= M.nblk || c >= M.nc || m >= M.n_p) return;
  const int n = M.n[c];
  const bool pair = M.sz[p] == 2;
  const double2* Vi = M.Vi[p][c];
  const int32_t e0 = M.cptr[m * M.nc + c], e1 = M.cptr[m * M.nc + c + 1];
  double2* out = M.Z[p] + (int64_t)m * M.n_v + M.off[c];
  for (int j = threadIdx.x; j < n; j += 256) {
    double re = 0.0, im = 0.0;
#pragma unroll 4
    for (int32_t e = e0; e < e1; ++e) {
      const double2 a = cc_value(M, p, M.cq[e]), v = cc_get(Vi, (int64_t)M.ci[e] * n + j, pair);
      re = fma(a.x, v.x, fma(-a.y, v.y, re));
      im = fma(a.x, v.y, fma(a.y, v.x, im));
    }
    out[j] = make_double2(re, im);
  }
}

// acc[k] = sum over the listed entries e of B(., m) times x at row k of a
// kRows-row slice of a row-major matrix (column bi[e] - o): the entries' values
// are read once for the slice's rows.
constexpr int kRows = 8;
template <typename X>
__device__ __forceinline__ void cc_times_b(const CompCoarse& M, int p, int32_t e0, int32_t e1,
                                           X&& x, double2 (&acc)[kRows]) {
#pragma unroll
  for (int k = 0; k < kRows; ++k) acc[k] = make_double2(0.0, 0.0);
#pragma unroll 2
  for (int32_t e = e0; e < e1; ++e) {
    const double2 a = cc_value(M, p, M.bq[e]);
    const int j = M.bi[e];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      const double2 v = x(k, j);
      acc[k].x = fma(a.x, v.x, fma(-a.y, v.y, acc[k].x));
      acc[k].y = fma(a.x, v.y, fma(a.y, v.x, acc[k].y));
    }
  }
}

// G = -V^-1 B: rows i0 .. of block c, a border column per thread.
__global__ void __launch_bounds__(256) k_cc_g(const CompCoarse* __restrict__ cc, int nc, int blk) {
  const CompCoarse& M = cc[blockIdx.z / (nc * blk)];
  const int pc = blockIdx.z % (nc * blk), p = pc / nc, c = pc % nc;
  const int i0 = blockIdx.x * kRows, m = blockIdx.y * 256 + (int)threadIdx.x;
  if (p >= M.nblk || c >= M.nc || i0 >= M.n[c] || m >= M.n_p) return;
  const int n = M.n[c], o = M.off[c];
  const bool pair = M.sz[p] == 2;
  const double2* Vi = M.Vi[p][c];
  double2 acc[kRows];
  cc_times_b(M, p, M.bptr[m * M.nc + c], M.bptr[m * M.nc + c + 1],
             [&](int k, int j) { return cc_get(Vi, (int64_t)min(i0 + k, n - 1) * n + j - o, pair); },
             acc);
#pragma unroll
  for (int k = 0; k < kRows; ++k)
    if (i0 + k < n)
      cc_put(M.G[p], (int64_t)(o + i0 + k) * M.n_p + m, pair, make_double2(-acc[k].x, -acc[k].y));
}

// S = D - Z B, rows m0 .., a column per thread, onto D in the Schur block's
// matrix (real form).
__global__ void __launch_bounds__(256) k_cc_s(const CompCoarse* __restrict__ cc) {
  const CompCoarse& M = cc[blockIdx.z / 4];
  const int p = blockIdx.z % 4, m0 = blockIdx.x * kRows, col = blockIdx.y * 256 + (int)threadIdx.x;
  if (p >= M.nblk || m0 >= M.n_p) return;
  if (col >= M.n_p) return;
  double* A = M.A[p][kCcMax];
  const int64_t ld = M.lda[kCcMax];
  const double2* Z = M.Z[p];
  double2 acc[kRows];
  cc_times_b(M, p, M.bptr[col * M.nc], M.bptr[(col + 1) * M.nc],
             [&](int k, int j) { return Z[(int64_t)min(m0 + k, M.n_p - 1) * M.n_v + j]; }, acc);
#pragma unroll
  for (int k = 0; k < kRows; ++k) {
    if (m0 + k >= M.n_p) continue;
    double2* even = reinterpret_cast<double2*>(&A[2 * (int64_t)(m0 + k) * ld + 2 * col]);
    const double2 d = *even;
    const double re = d.x - acc[k].x, im = -d.y - acc[k].y;
    *even = make_double2(re, -im);
    *reinterpret_cast<double2*>(&A[(2 * (int64_t)(m0 + k) + 1) * ld + 2 * col]) =
        make_double2(im, re);
  }
}

// A 32 x 32 tile of a complex (real: pair false) matrix product on FP64 matrix
// cores: one instruction tile for each of four wavefronts, 16 columns of the
// left factor per step staged in LDS.  left(r, k) and right(k, c) read the
// factors (zero outside); element v of the result is row wr + 4 v + (lane >> 4),
// column wc + (lane & 15) of the tile.  Bound by the number of tiles: of 64 x 64
// there are 65 for P and 169 for X at order 786 (dG(1), 16x4 cells), for 256
// compute units (that build 1.25 -> 1.20 ms).
constexpr int kCcTile = 32, kCcK = 16;
struct CcLds { double2 a[kCcTile][kCcK + 1], b[kCcK][kCcTile + 1]; };
template <typename L, typename R>
__device__ __forceinline__ void cc_tile(CcLds& lds, int len, bool pair, L&& left, R&& right,
                                        stv_d4& re, stv_d4& im) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lr = lane >> 4, lc = lane & 15, wr = 16 * (w >> 1), wc = 16 * (w & 1);
  for (int k0 = 0; k0 < len; k0 += kCcK) {
    double2 a[2], b[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = tid + 256 * u;
      a[u] = left(e / kCcK, k0 + e % kCcK);
      b[u] = right(k0 + e / kCcTile, e % kCcTile);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = tid + 256 * u;
      lds.a[e / kCcK][e % kCcK] = a[u];
      lds.b[e / kCcTile][e % kCcTile] = b[u];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kCcK; k += 4) {
      const double2 x = lds.a[wr + lc][k + lr], y = lds.b[k + lr][wc + lc];
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.x, re, 0, 0, 0);
      if (!pair) continue;
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.y, y.y, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.y, im, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.x, im, 0, 0, 0);
    }
  }
}

// P = S^-1 [-Z | I].  Only where the product is small (CcDims::form_p): it
// saves one launch per solve.
__global__ void __launch_bounds__(256) k_cc_p(const CompCoarse* __restrict__ cc, int blocks) {
  __shared__ CcLds lds;
  const CompCoarse& M = cc[blockIdx.z / blocks];
  const int p = blockIdx.z % blocks;
  if (p >= M.nblk) return;
  if (!M.P[p]) return;
  const int n_p = M.n_p, n_v = M.n_v, n_s = n_v + n_p;
  const int m0 = blockIdx.y * kCcTile, e0 = blockIdx.x * kCcTile;
  if (m0 >= n_p || e0 >= n_s) return;
  const bool pair = M.sz[p] == 2;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lr = lane >> 4, lc = lane & 15, wr = 16 * (w >> 1), wc = 16 * (w & 1);
  const double2 *Si = M.Si[p], *Z = M.Z[p], zero = make_double2(0.0, 0.0);
  stv_d4 re = {}, im = {};
  if (e0 < n_v)
    cc_tile(lds, n_p, pair,
            [&](int r, int k) {
              return m0 + r < n_p && k < n_p ? Si[(int64_t)(m0 + r) * n_p + k] : zero;
            },
            [&](int k, int c) {
              return k < n_p && e0 + c < n_v ? Z[(int64_t)k * n_v + e0 + c] : zero;
            },
            re, im);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int m = m0 + wr + 4 * v + lr, e = e0 + wc + lc;
    if (m >= n_p || e >= n_s) continue;
    cc_put(M.P[p], (int64_t)m * n_s + e, pair,
           e < n_v ? make_double2(-re[v], -im[v]) : Si[(int64_t)m * n_p + e - n_v]);
  }
}

// A time block's whole inverse in the level's row order: block rows G P + V^-1,
// border rows P.  One time component (CcDims::form_x): real, into the coarse
// store, scaled by the block's V and W.  More (form_c): Xp, a complex or real
// entry per spatial pair, for k_cc_apply: 16 n^2 instead of the 32 n^2 bytes of
// the recombined inverse for a pair, 24 instead of 72 with a real block beside.
__global__ void __launch_bounds__(256) k_cc_x(const CompCoarse* __restrict__ cc, int blocks) {
  __shared__ CcLds lds;
  const CompCoarse& M = cc[blockIdx.z / blocks];
  const int p = blockIdx.z % blocks;
  const int n_p = M.n_p, n_v = M.n_v, n_s = n_v + n_p;
  const int e0 = blockIdx.y * kCcTile, f0 = blockIdx.x * kCcTile;
  if (p >= M.nblk || e0 >= n_s || f0 >= n_s) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lr = lane >> 4, lc = lane & 15, wr = 16 * (w >> 1), wc = 16 * (w & 1);
  const double2 zero = make_double2(0.0, 0.0);
  // the tile's rows: place in the level, block (kCcMax: border), its range;
  // columns: place in the level
  __shared__ int row_at[kCcTile], row_c[kCcTile], row_o[kCcTile], row_n[kCcTile], col_at[kCcTile];
  if (threadIdx.x < kCcTile) {
    const int e = min(e0 + (int)threadIdx.x, n_s - 1), f = min(f0 + (int)threadIdx.x, n_s - 1);
    int c = kCcMax, o = 0, n = 0;
    for (int t = 0; t < M.nc; ++t)
      if (e >= M.off[t] && e < M.off[t] + M.n[t]) { c = t; o = M.off[t]; n = M.n[t]; }
    row_at[threadIdx.x] = M.order[e];
    row_c[threadIdx.x] = c;
    row_o[threadIdx.x] = o;
    row_n[threadIdx.x] = n;
    col_at[threadIdx.x] = M.order[f];
  }
  __syncthreads();
  const int f = min(f0 + wc + lc, n_s - 1);
  const bool pair = M.sz[p] == 2;
  const double2 *G = M.G[p], *P = M.P[p];
  stv_d4 re = {}, im = {};
  if (e0 < n_v)
    cc_tile(lds, n_p, pair,
            [&](int r, int k) {
              return e0 + r < n_v && k < n_p ? cc_get(G, (int64_t)(e0 + r) * n_p + k, pair) : zero;
            },
            [&](int k, int c) {
              return k < n_p && f0 + c < n_s ? cc_get(P, (int64_t)k * n_s + f0 + c, pair) : zero;
            },
            re, im);
  // the rows' own entries; all reads stand before the writes, which they
  // could not pass
  double2 x[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int er = wr + 4 * v + lr, e = min(e0 + er, n_s - 1);
    const int c = row_c[er], o = row_o[er], n = row_n[er];
    const bool border = c == kCcMax, in = f >= o && f < o + n;
    const double2* from = border ? P : M.Vi[p][in ? c : 0];
    const int64_t at = border ? (int64_t)(e - n_v) * n_s + f
                              : in ? (int64_t)(e - o) * n + f - o : 0;
    const double2 q = cc_get(from, at, pair);
    x[v].x = (border ? 0.0 : re[v]) + (border || in ? q.x : 0.0);
    x[v].y = (border ? 0.0 : im[v]) + (border || in ? q.y : 0.0);
  }
  if (f0 + wc + lc >= n_s) return;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    if (e0 + wr + 4 * v + lr >= n_s) continue;
    const int64_t at = (int64_t)row_at[wr + 4 * v + lr] * n_s + col_at[wc + lc];
    if (M.X) M.X[at] = M.V[0] * (x[v].x * M.W[0]);
    else cc_put(M.Xp[p], at, pair, x[v]);
  }
}

// d = J^-1 r from the time blocks' whole inverses, a wavefront per spatial row:
// z = W r on the fly, y_p = x_p z_p, d = V y.  Bound by the latency of the
// descriptor, then of a row's loads: the former are all at fixed places, four of
// the latter in flight per lane (a workgroup per row: 63 members of 218 rows 34 ->
// 13 us, 72 of 458 77 -> 38 us, one of 786 5.2 -> 4.9 us, one of 1,438 9.2 -> 9.6).
template <int B>
__global__ void __launch_bounds__(256) k_cc_apply(const CompCoarse* __restrict__ cc,
                                                  const double* __restrict__ r,
                                                  double* __restrict__ d) {
  const CompCoarse& M = cc[blockIdx.z];
  const int lane = threadIdx.x & 63;
  const int n = M.n_v + M.n_p, s = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (s >= n) return;
  const double* rz = r + (int64_t)M.row_off * B;
  double2 acc[B];
#pragma unroll
  for (int p = 0; p < B; ++p) {
    acc[p] = make_double2(0.0, 0.0);
    if (p >= M.nblk) continue;
    const bool pair = M.sz[p] == 2;
    double w0[B], w1[B];
#pragma unroll
    for (int l = 0; l < B; ++l) {
      w0[l] = M.w[p][0][l];
      w1[l] = M.w[p][1][l];
    }
    constexpr int U = 4;
    for (int c0 = lane; c0 < n; c0 += 64 * U) {
      double2 x[U];
      double v[U][B];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = min(c0 + 64 * u, n - 1);
        x[u] = cc_get(M.Xp[p], (int64_t)s * n + c, pair);
#pragma unroll
        for (int l = 0; l < B; ++l) v[u][l] = rz[(int64_t)c * B + l];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        double z0 = 0.0, z1 = 0.0;
#pragma unroll
        for (int l = 0; l < B; ++l) {
          z0 = fma(w0[l], v[u][l], z0);
          z1 = fma(w1[l], v[u][l], z1);
        }
        const double re = fma(x[u].x, z0, fma(-x[u].y, z1, acc[p].x));
        const double im = fma(x[u].x, z1, fma(x[u].y, z0, acc[p].y));
        const bool in = c0 + 64 * u < n;
        acc[p].x = in ? re : acc[p].x;
        acc[p].y = in ? im : acc[p].y;
      }
    }
  }
  double out[B];
#pragma unroll
  for (int i = 0; i < B; ++i) out[i] = 0.0;
#pragma unroll
  for (int p = 0; p < B; ++p) {
    if (p >= M.nblk) continue;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      acc[p].x += __shfl_xor(acc[p].x, off, 64);
      acc[p].y += __shfl_xor(acc[p].y, off, 64);
    }
#pragma unroll
    for (int i = 0; i < B; ++i) {
      out[i] = fma(M.v[p][0][i], acc[p].x, out[i]);
      if (M.sz[p] == 2) out[i] = fma(M.v[p][1][i], acc[p].y, out[i]);
    }
  }
  double v = out[0];
#pragma unroll
  for (int i = 1; i < B; ++i) v = lane == i ? out[i] : v;
  if (lane < B) d[((int64_t)M.row_off + s) * B + lane] = v;
}

// d = J^-T r: per time block t = sum_s conj(u_s) x_p[s, .] with u = (V^T r) (its
// pair of columns), d_l = Re(t w_l).  16 columns per workgroup, 64 row groups of
// 16 threads each take the rows g, g + 64, ... and meet in LDS in a fixed order
// (as k_dense_gemv_t).
template <int B>
__global__ void __launch_bounds__(1024) k_cc_apply_t(const CompCoarse* __restrict__ cc,
                                                     const double* __restrict__ r,
                                                     double* __restrict__ d) {
  constexpr int NC = 16, NG = 64;
  __shared__ double2 red[NG][NC + 1];
  const CompCoarse& M = cc[blockIdx.z];
  const int n = M.n_v + M.n_p;
  if ((int)blockIdx.x * NC >= n) return;
  const int c = threadIdx.x % NC, g = threadIdx.x / NC;
  const int j = min((int)blockIdx.x * NC + c, n - 1);
  const double* rz = r + (int64_t)M.row_off * B;
  double out[B];
#pragma unroll
  for (int l = 0; l < B; ++l) out[l] = 0.0;
  for (int p = 0; p < M.nblk; ++p) {
    const bool pair = M.sz[p] == 2;
    double v0[B], v1[B];
#pragma unroll
    for (int i = 0; i < B; ++i) {
      v0[i] = M.v[p][0][i];
      v1[i] = M.v[p][1][i];
    }
    double2 t = make_double2(0.0, 0.0);
#pragma unroll 4
    for (int s = g; s < n; s += NG) {
      const double2 x = cc_get(M.Xp[p], (int64_t)s * n + j, pair);
      double u0 = 0.0, u1 = 0.0;
#pragma unroll
      for (int i = 0; i < B; ++i) {
        const double v = rz[(int64_t)s * B + i];
        u0 = fma(v0[i], v, u0);
        u1 = fma(v1[i], v, u1);
      }
      t.x = fma(x.x, u0, fma(x.y, u1, t.x));
      t.y = fma(x.y, u0, fma(-x.x, u1, t.y));
    }
    __syncthreads();   // the last block's sums have been read
    red[g][c] = t;
    __syncthreads();
    for (int h = NG / 2; h >= 1; h >>= 1) {
      if (g < h) {
        red[g][c].x += red[g + h][c].x;
        red[g][c].y += red[g + h][c].y;
      }
      __syncthreads();
    }
    t = red[0][c];
#pragma unroll
    for (int l = 0; l < B; ++l) {
      out[l] = fma(M.w[p][0][l], t.x, out[l]);
      if (pair) out[l] = fma(-M.w[p][1][l], t.y, out[l]);
    }
  }
  if (g != 0 || (int)blockIdx.x * NC + c >= n) return;
#pragma unroll
  for (int l = 0; l < B; ++l) d[((int64_t)M.row_off + j) * B + l] = out[l];
}

// ---------------------------------------------------------------------------
// Whether the parts give an inverse.  Each V_c takes its pivots in itself, so a
// velocity block that is nearly singular inside a well-conditioned matrix leaves
// V^-1 and S with entries that cancel in V^-1 + G P, and no bound on the blocks'
// own condition sees that (max |V| max |V^-1| of 3e7 and 1e6 for S with an error
// of 5e-9; 2e5 and 1e3 on a channel operator without any).  So the factors are
// tried: y = A^-1 z by them for kProbe pseudo-random right-hand sides, and a
// time block counts as inverted when, over the rows with a diagonal entry and
// over those without (of another scale: the pressure) separately,
//   max_i |z - A y|_i <= 2^-53 (4096 + 2 n) max_i (|A| |y| + |z|)_i.
// Measured over channel operators of order 210 to 9,204 (nu 1e-6 to 1e-1, tau
// 1e-4 to 10): 2 to 5e3 units of 2^-53 on the rows with a diagonal entry,
// within the bound for all 372; on the others 20 to 4.3e4 for these factors
// and 20 to 2e3 for a pivoted inverse of the whole matrix, although the
// solutions are about as accurate (errors 4e-14 to 8e-12 and 2e-13 to 7e-12):
// those rows' |A| |y| does not hold the border's part of y, G y_border, which
// cancels against V^-1 z (29 of the 372, on cells stretched by 3 to 1 and 5 to
// 1, are beyond the bound).  So a time block beyond it on those rows alone is
// looked at again: e = A^-1 (z - A y) by the factors is what the residual
// means for y, and w = A^-1 s, s_i = +-2^-53 (|A| |y| + |z|)_i, what one
// rounding per row does; it counts as inverted when max |e| <= 128 max |w|
// over the rows with a diagonal entry.  Measured 5 to 82 for the 29, 137 and
// more for operators with a velocity block close to singular that the bound
// refuses (5e2 and more where the solution has lost two digits).  Otherwise
// the build eliminates the whole coarse matrix.  Three launches (four without
// P), the second look two (three) where a member needs it; the right-hand
// sides share every load.
constexpr int kProbe = kCcProbe;
constexpr double kProbeNoise = 128.0;
constexpr int kProbeParts = 16, kProbeCount = 24;   // probe_max: residuals, second look, arrivals
static_assert(kProbeCount + 2 == kCcProbeWords);

// entry e of right-hand side j: parts in [-1, 1) from a multiplicative hash
__device__ __forceinline__ double2 cc_probe(int e, int j, bool pair) {
  auto part = [&](uint32_t k) {
    uint32_t h = ((uint32_t)e * kProbe * 2 + (uint32_t)j * 2 + k + 1u) * 2654435769u;
    h = (h ^ (h >> 15)) * 2246822519u;
    h = (h ^ (h >> 13)) * 3266489917u;
    return (double)(int32_t)(h ^ (h >> 16)) * 0x1p-31;
  };
  return make_double2(part(0), pair ? part(1) : 0.0);
}

__device__ __forceinline__ void cc_mad(double2& s, double2 a, double2 b) {
  s.x = fma(a.x, b.x, fma(-a.y, b.y, s.x));
  s.y = fma(a.x, b.y, fma(a.y, b.x, s.y));
}

__device__ __forceinline__ double cc_abs1(double2 a) { return fabs(a.x) + fabs(a.y); }

// the larger of the two; a NaN stays
__device__ __forceinline__ double cc_larger(double a, double b) { return (a != a || a > b) ? a : b; }

__device__ __forceinline__ void cc_wave_sum(double2 (&s)[kProbe]) {
#pragma unroll
  for (int j = 0; j < kProbe; ++j)
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      s[j].x += __shfl_xor(s[j].x, off, 64);
      s[j].y += __shfl_xor(s[j].y, off, 64);
    }
}

// The trial's input: the right-hand sides, or the columns that k_cc_probe_r left.
template <bool COLS>
__device__ __forceinline__ double2 cc_probe_in(const CompCoarse& M, const double2* z, int e, int j, bool pair) {
  return COLS ? z[(int64_t)j * (M.n_v + M.n_p) + e] : cc_probe(e, j, pair);
}

// A workgroup's N maxima into the member's words from `at`, in its first threads.
template <int N>
__device__ __forceinline__ void cc_probe_max(const CompCoarse& M, int at, const double (&red)[4][N]) {
  if (threadIdx.x >= N) return;
  double v = red[0][threadIdx.x];
  for (int k = 1; k < 4; ++k) v = cc_larger(red[k][threadIdx.x], v);
  const unsigned long long old = atomic_max_bits(&M.probe_max[at + threadIdx.x], v);
  // The maxima have been made where their old values are back; the arrival
  // comes after them, without a fence (which would write the L2 back, once per
  // workgroup: a batch of 136 members 137 us).
  asm volatile("" : : "v"(old) : "memory");
}

// Whether this is the last of the `all` workgroups counted in word `at`.
__device__ __forceinline__ bool cc_probe_last(const CompCoarse& M, int at, unsigned long long all) {
  return atomicAdd(&M.probe_max[at], 1ull) == all - 1;
}

__device__ __forceinline__ double cc_probe_word(const CompCoarse& M, int i) {
  return __builtin_bit_cast(double, __hip_atomic_load(&M.probe_max[i], __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT));
}

// On rows with a diagonal entry: the larger solution of the error columns and
// of the noise columns (lane 0 of a wavefront).
__device__ __forceinline__ void cc_probe_parts(const double2 (&s)[kProbe], bool diag, double (&red)[2]) {
  red[0] = diag ? cc_larger(cc_abs1(s[0]), cc_abs1(s[1])) : 0.0;
  red[1] = diag ? cc_larger(cc_abs1(s[2]), cc_abs1(s[3])) : 0.0;
}

// Border part, a wavefront per border row (the last row may come twice): y = P z,
// or without P first q = z_border - Z z (last false), then y = S^-1 q (last true).
template <bool COLS>
__global__ void __launch_bounds__(256) k_cc_probe_p(const CompCoarse* __restrict__ cc, bool last) {
  __shared__ double red[4][2];
  const CompCoarse& M = cc[blockIdx.z];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int p = blockIdx.y, m = min((int)blockIdx.x * 4 + wv, M.n_p - 1);
  if (p >= M.nblk || (int)blockIdx.x * 4 >= M.n_p) return;
  const bool pair = M.sz[p] == 2, form = M.P[p] != nullptr;
  const int n_s = M.n_v + M.n_p;
  double2* q = M.probe_q + (int64_t)p * kProbe * M.n_p;
  const double2* z = M.probe_z + (int64_t)p * (kProbe + 1) * n_s;
  double2 s[kProbe] = {};
  if (last) {
    const double2* row = M.Si[p] + (int64_t)m * M.n_p;
    for (int e = lane; e < M.n_p; e += 64) {
      const double2 a = row[e];
#pragma unroll
      for (int j = 0; j < kProbe; ++j) cc_mad(s[j], a, q[(int64_t)j * M.n_p + e]);
    }
  } else {
    const int len = form ? n_s : M.n_v;
    for (int e = lane; e < len; e += 64) {
      const double2 a = form ? cc_get(M.P[p], (int64_t)m * len + e, pair)
                             : M.Z[p][(int64_t)m * len + e];
#pragma unroll
      for (int j = 0; j < kProbe; ++j) cc_mad(s[j], a, cc_probe_in<COLS>(M, z, e, j, pair));
    }
  }
  cc_wave_sum(s);
  if (lane == 0) {
    double2* y = M.probe_y + (int64_t)p * kProbe * n_s + M.n_v + m;
#pragma unroll
    for (int j = 0; j < kProbe; ++j) {
      if (last || form) {
        y[(int64_t)j * n_s] = s[j];
      } else {
        const double2 v = cc_probe_in<COLS>(M, z, M.n_v + m, j, pair);
        q[(int64_t)j * M.n_p + m] = make_double2(v.x - s[j].x, v.y - s[j].y);
      }
    }
  }
  if (!COLS || !(last || form)) return;
  if (lane == 0) cc_probe_parts(s, z[(int64_t)kProbe * n_s + M.n_v + m].x != 0.0, red[wv]);
  __syncthreads();
  cc_probe_max(M, kProbeParts + 2 * p, red);
}

// Block part, a wavefront per row (the last row may come twice): y = V^-1 z + G y_border.
// With COLS the member's last workgroup (counted in the last word) gives the verdict.
template <bool COLS>
__global__ void __launch_bounds__(256) k_cc_probe_u(const CompCoarse* __restrict__ cc) {
  __shared__ double red[4][2];
  const CompCoarse& M = cc[blockIdx.z];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int p = blockIdx.y, e = min((int)blockIdx.x * 4 + wv, M.n_v - 1);
  if (p >= M.nblk || (int)blockIdx.x * 4 >= M.n_v) return;
  const bool pair = M.sz[p] == 2;
  int c = 0;
  while (c + 1 < M.nc && e >= M.off[c] + M.n[c]) ++c;
  const int n = M.n[c], o = M.off[c], n_s = M.n_v + M.n_p;
  double2* y = M.probe_y + (int64_t)p * kProbe * n_s;
  const double2* z = M.probe_z + (int64_t)p * (kProbe + 1) * n_s;
  double2 s[kProbe] = {};
  for (int k = lane; k < n; k += 64) {
    const double2 a = cc_get(M.Vi[p][c], (int64_t)(e - o) * n + k, pair);
#pragma unroll
    for (int j = 0; j < kProbe; ++j) cc_mad(s[j], a, cc_probe_in<COLS>(M, z, o + k, j, pair));
  }
  for (int m = lane; m < M.n_p; m += 64) {
    const double2 a = cc_get(M.G[p], (int64_t)e * M.n_p + m, pair);
#pragma unroll
    for (int j = 0; j < kProbe; ++j) cc_mad(s[j], a, y[(int64_t)j * n_s + M.n_v + m]);
  }
  cc_wave_sum(s);
  if (!COLS) {
    if (lane != 0) return;
#pragma unroll
    for (int j = 0; j < kProbe; ++j) y[(int64_t)j * n_s + e] = s[j];
    return;
  }
  if (lane == 0) cc_probe_parts(s, z[(int64_t)kProbe * n_s + e].x != 0.0, red[wv]);
  __syncthreads();
  cc_probe_max(M, kProbeParts + 2 * p, red);
  if (threadIdx.x != 0) return;
  if (!cc_probe_last(M, kProbeCount + 1, (unsigned long long)((M.n_v + 3) / 4) * M.nblk)) return;
  for (int q = 0; q < M.nblk; ++q) {
    int* verdict = M.verdict[q][kCcMax];
    if (*verdict != kCcBareRows) continue;
    const double err = cc_probe_word(M, kProbeParts + 2 * q), noise = cc_probe_word(M, kProbeParts + 2 * q + 1);
    *verdict = !(err <= kProbeNoise * noise && noise < INFINITY);
  }
}

// Residuals and their scale, a wavefront per row, and the columns of the second
// look; the member's last workgroup gives the verdict.
__global__ void __launch_bounds__(256) k_cc_probe_r(const CompCoarse* __restrict__ cc) {
  __shared__ double red[4][4];   // per wavefront: residual, scale; without a diagonal the last two
  const CompCoarse& M = cc[blockIdx.z];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int n_s = M.n_v + M.n_p;
  const int p = blockIdx.y, e = min((int)blockIdx.x * 4 + wv, n_s - 1);   // the last row twice
  if (p >= M.nblk || (int)blockIdx.x * 4 >= n_s) return;
  const bool pair = M.sz[p] == 2;
  const double2* y = M.probe_y + (int64_t)p * kProbe * n_s;
  double2* cols = M.probe_z + (int64_t)p * (kProbe + 1) * n_s;
  const int32_t row = M.row_off + M.order[e];
  double2 s[kProbe] = {}, w[kProbe] = {};
  bool diag = false;
  for (int32_t q = M.rowptr[row] + lane; q < M.rowptr[row + 1]; q += 64) {
    const double2 a = cc_value(M, p, q);
    const int at = M.where[M.col[q] - M.row_off];
    diag = diag || (at == e && (a.x != 0.0 || a.y != 0.0));
#pragma unroll
    for (int j = 0; j < kProbe; ++j) {
      const double2 v = y[(int64_t)j * n_s + at];
      cc_mad(s[j], a, v);
      w[j].x = fma(cc_abs1(a), cc_abs1(v), w[j].x);
    }
  }
  cc_wave_sum(s);
  cc_wave_sum(w);
  diag = __any(diag);
  if (lane == 0) {
    double r = 0.0, t = 0.0;
#pragma unroll
    for (int j = 0; j < kProbe; ++j) {
      const double2 z = cc_probe(e, j, pair), v = make_double2(z.x - s[j].x, z.y - s[j].y);
      const double scale = w[j].x + cc_abs1(z);
      r = cc_larger(cc_abs1(v), r);
      t = cc_larger(scale, t);
      if (j < 2) {
        cols[(int64_t)j * n_s + e] = v;
        cols[(int64_t)(j + 2) * n_s + e] = make_double2(copysign(0x1p-53 * scale, z.x), 0.0);
      }
    }
    cols[(int64_t)kProbe * n_s + e] = make_double2(diag ? 1.0 : 0.0, 0.0);
    red[wv][0] = diag ? r : 0.0;
    red[wv][1] = diag ? t : 0.0;
    red[wv][2] = diag ? 0.0 : r;
    red[wv][3] = diag ? 0.0 : t;
  }
  __syncthreads();
  cc_probe_max(M, 4 * p, red);
  if (threadIdx.x != 0) return;
  if (!cc_probe_last(M, kProbeCount, (unsigned long long)((n_s + 3) / 4) * M.nblk)) return;
  for (int q = 0; q < M.nblk; ++q) {
    auto within = [&](int k) {
      const double res = cc_probe_word(M, 4 * q + 2 * k), scale = cc_probe_word(M, 4 * q + 2 * k + 1);
      return res <= 0x1p-53 * (4096.0 + 2.0 * n_s) * scale && scale < INFINITY;
    };
    int* verdict = M.verdict[q][kCcMax];
    if (!within(0)) *verdict = 1;
    else if (!within(1) && *verdict == 0) *verdict = kCcBareRows;
  }
}

// z_e = (W r)_e of time block p at member position e (its complex pair)
template <int B>
__device__ __forceinline__ double2 cc_rhs(const CompCoarse& M, int p, int e,
                                          const double* __restrict__ r) {
  const int64_t s = (int64_t)(M.row_off + M.order[e]) * B;
  const int f = M.first[p];
  double z0 = 0.0, z1 = 0.0;
#pragma unroll
  for (int l = 0; l < B; ++l) z0 = fma(M.W[f * B + l], r[s + l], z0);
  if (M.sz[p] == 2) {
#pragma unroll
    for (int l = 0; l < B; ++l) z1 = fma(M.W[(f + 1) * B + l], r[s + l], z1);
  }
  return make_double2(z0, z1);
}

// The border vectors of one of the two sets.
__device__ __forceinline__ double2* cc_pw(const CompCoarse& M, int set) {
  return M.pw + (int64_t)set * 2 * M.nblk * M.n_p;
}

// Sum over a workgroup of 256 threads, in thread 0.
__device__ __forceinline__ double2 cc_block_sum(double re, double im, double2 (&red)[4]) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    re += __shfl_xor(re, off, 64);
    im += __shfl_xor(im, off, 64);
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = make_double2(re, im);
  __syncthreads();
  return make_double2((red[0].x + red[1].x) + (red[2].x + red[3].x),
                      (red[0].y + red[1].y) + (red[2].y + red[3].y));
}

// First half of the solve: p = P z, one workgroup per border row and time
// block; without P, q = z_border - Z z instead (k_cc_solve_s then forms
// p = S^-1 q).
template <int B>
__global__ void __launch_bounds__(256) k_cc_solve_p(const CompCoarse* __restrict__ cc, int set,
                                                    const double* __restrict__ r) {
  __shared__ double2 red[4];
  const CompCoarse& M = cc[blockIdx.z];
  const int p = blockIdx.y, m = blockIdx.x;
  if (p >= M.nblk || m >= M.n_p) return;
  const bool form = M.P[p] != nullptr;
  const int len = form ? M.n_v + M.n_p : M.n_v;
  double re = 0.0, im = 0.0;
  if (form && M.sz[p] == 1) {
    const double* row = reinterpret_cast<const double*>(M.P[p]) + (int64_t)m * len;
#pragma unroll 4
    for (int e = threadIdx.x; e < len; e += 256) re = fma(row[e], cc_rhs<B>(M, p, e, r).x, re);
  } else {
    const double2* row = (form ? M.P[p] : M.Z[p]) + (int64_t)m * len;
#pragma unroll 4
    for (int e = threadIdx.x; e < len; e += 256) {
      const double2 a = row[e], z = cc_rhs<B>(M, p, e, r);
      re = fma(a.x, z.x, fma(-a.y, z.y, re));
      im = fma(a.x, z.y, fma(a.y, z.x, im));
    }
  }
  const double2 v = cc_block_sum(re, im, red);
  if (threadIdx.x != 0) return;
  double2* pw = cc_pw(M, set);
  if (form) {
    pw[p * M.n_p + m] = v;
  } else {
    const double2 z = cc_rhs<B>(M, p, M.n_v + m, r);
    pw[(M.nblk + p) * M.n_p + m] = make_double2(z.x - v.x, z.y - v.y);
  }
}

// p = S^-1 q, one workgroup per border row and time block.
__global__ void __launch_bounds__(256) k_cc_solve_s(const CompCoarse* __restrict__ cc, int set) {
  __shared__ double2 red[4];
  const CompCoarse& M = cc[blockIdx.z];
  const int p = blockIdx.y, m = blockIdx.x;
  if (p >= M.nblk || m >= M.n_p || M.P[p]) return;
  const double2* row = M.Si[p] + (int64_t)m * M.n_p;
  double2* pw = cc_pw(M, set);
  const double2* q = pw + (M.nblk + p) * M.n_p;
  double re = 0.0, im = 0.0;
#pragma unroll 4
  for (int e = threadIdx.x; e < M.n_p; e += 256) {
    const double2 a = row[e], z = q[e];
    re = fma(a.x, z.x, fma(-a.y, z.y, re));
    im = fma(a.x, z.y, fma(a.y, z.x, im));
  }
  const double2 v = cc_block_sum(re, im, red);
  if (threadIdx.x == 0) pw[p * M.n_p + m] = v;
}

// Second half: u = V^-1 z + G p and the time recombination, one wavefront per
// spatial row (a border row only copies its p).
template <int B>
__global__ void __launch_bounds__(256) k_cc_solve_u(const CompCoarse* __restrict__ cc, int set,
                                                    const double* __restrict__ r,
                                                    double* __restrict__ d) {
  const CompCoarse& M = cc[blockIdx.z];
  const int lane = threadIdx.x & 63;
  const int e = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (e >= M.n_v + M.n_p) return;
  const double2* pw = cc_pw(M, set);
  int c = 0;
  while (c < M.nc && e >= M.off[c] + M.n[c]) ++c;
  double out[B];
#pragma unroll
  for (int i = 0; i < B; ++i) out[i] = 0.0;
  for (int p = 0; p < M.nblk; ++p) {
    double re = 0.0, im = 0.0;
    if (c < M.nc && M.sz[p] == 1) {
      const int n = M.n[c];
      const double* row = reinterpret_cast<const double*>(M.Vi[p][c]) + (int64_t)(e - M.off[c]) * n;
#pragma unroll 4
      for (int j = lane; j < n; j += 64) re = fma(row[j], cc_rhs<B>(M, p, M.off[c] + j, r).x, re);
      const double* g = reinterpret_cast<const double*>(M.G[p]) + (int64_t)e * M.n_p;
#pragma unroll 4
      for (int m = lane; m < M.n_p; m += 64) re = fma(g[m], pw[p * M.n_p + m].x, re);
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) re += __shfl_xor(re, off, 64);
    } else if (c < M.nc) {
      const int n = M.n[c];
      const double2* row = M.Vi[p][c] + (int64_t)(e - M.off[c]) * n;
#pragma unroll 4
      for (int j = lane; j < n; j += 64) {
        const double2 a = row[j], z = cc_rhs<B>(M, p, M.off[c] + j, r);
        re = fma(a.x, z.x, fma(-a.y, z.y, re));
        im = fma(a.x, z.y, fma(a.y, z.x, im));
      }
      const double2* g = M.G[p] + (int64_t)e * M.n_p;
#pragma unroll 4
      for (int m = lane; m < M.n_p; m += 64) {
        const double2 a = g[m], z = pw[p * M.n_p + m];
        re = fma(a.x, z.x, fma(-a.y, z.y, re));
        im = fma(a.x, z.y, fma(a.y, z.x, im));
      }
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) {
        re += __shfl_xor(re, off, 64);
        im += __shfl_xor(im, off, 64);
      }
    } else {
      const double2 v = pw[p * M.n_p + e - M.n_v];
      re = v.x;
      im = v.y;
    }
    const int f = M.first[p];
#pragma unroll
    for (int i = 0; i < B; ++i) {
      out[i] = fma(M.V[i * B + f], re, out[i]);
      if (M.sz[p] == 2) out[i] = fma(M.V[i * B + f + 1], im, out[i]);
    }
  }
  if (lane < B) {
    double v = out[0];
#pragma unroll
    for (int i = 1; i < B; ++i) v = lane == i ? out[i] : v;
    d[(int64_t)(M.row_off + M.order[e]) * B + lane] = v;
  }
}

__global__ void __launch_bounds__(256) k_block_nonzero(const double* __restrict__ val, int b2,
                                                       int64_t nnzb, uint8_t* __restrict__ nz) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= nnzb) return;
  bool any = false;
  for (int e = 0; e < b2; ++e) any |= val[q * b2 + e] != 0.0;   // a NaN counts
  nz[q] = any;
}

hipError_t launch_block_nonzero(hipStream_t s, int b, const double* val, int64_t nnzb, uint8_t* nz) {
  k_block_nonzero<<<(unsigned)((nnzb + 255) / 256), 256, 0, s>>>(val, b * b, nnzb, nz);
  return hipGetLastError();
}

__global__ void __launch_bounds__(64) k_expand_blocks(int b, int32_t n_s,
                                                      const int32_t* __restrict__ ptr,
                                                      const int32_t* __restrict__ bcol,
                                                      const int32_t* __restrict__ src,
                                                      const double* __restrict__ val,
                                                      int32_t* __restrict__ rowptr,
                                                      int32_t* __restrict__ col,
                                                      double2* __restrict__ ma) {
  const int32_t r = blockIdx.x, first = ptr[r];
  const int len = (ptr[r + 1] - first) * b;
  const int64_t base = (int64_t)first * b * b;
  for (int t = threadIdx.x; t < len * b; t += 64) {
    const int l = t / len, k = (t % len) / b, j = t % len % b;
    col[base + t] = bcol[first + k] * b + j;
    ma[base + t] = make_double2(0.0, val[(int64_t)src[first + k] * b * b + l * b + j]);
  }
  if ((int)threadIdx.x < b) rowptr[r * b + threadIdx.x] = (int32_t)(base + threadIdx.x * len);
  if (r == n_s - 1 && threadIdx.x == 0) rowptr[n_s * b] = (int32_t)(base + b * len);
}

hipError_t launch_expand_blocks(hipStream_t s, int b, int32_t n_s, const int32_t* ptr,
                                const int32_t* bcol, const int32_t* src, const double* val,
                                int32_t* rowptr, int32_t* col, double* ma) {
  k_expand_blocks<<<(unsigned)n_s, 64, 0, s>>>(b, n_s, ptr, bcol, src, val, rowptr, col,
                                               reinterpret_cast<double2*>(ma));
  return hipGetLastError();
}

// The members in slices whose grids stay within 65,535 in z (a batch has up to
// 65,535 members, and up to 48 blocks each).
template <typename F>
static hipError_t cc_slices(const CompCoarse* cc, const CcDims& D, F&& f) {
  constexpr unsigned kSlice = 1024;
  static_assert(kSlice * 4 * kCcMax <= 65535);
  for (unsigned at = 0; at < D.cnt; at += kSlice) {
    CcDims S = D;
    S.cnt = D.cnt - at < kSlice ? D.cnt - at : kSlice;
    const hipError_t e = f(cc + at, S);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_cc_fill(hipStream_t s, const CompCoarse* cc, const CcDims& D) {
  k_cc_fill<<<dim3(D.n_s, D.blk, D.cnt), 64, 0, s>>>(cc);
  return hipGetLastError();
}

// After the V chain: V^-1, Z, G and the Schur blocks.
static hipError_t cc_schur(hipStream_t s, const CompCoarse* cc, const CcDims& D) {
  const unsigned cols = (D.n_p + 255) / 256;
  k_cc_collect_v<<<dim3(D.n, D.blk * D.nc, D.cnt), 256, 0, s>>>(cc, D.nc);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_cc_z<<<dim3(D.n_p, D.blk * D.nc, D.cnt), 256, 0, s>>>(cc, D.nc);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_cc_s<<<dim3((D.n_p + kRows - 1) / kRows, cols, 4 * D.cnt), 256, 0, s>>>(cc);
  return hipGetLastError();
}

hipError_t launch_cc_schur(hipStream_t s, const CompCoarse* cc, const CcDims& D) {
  return cc_slices(cc, D, [&](const CompCoarse* c, const CcDims& S) { return cc_schur(s, c, S); });
}

// The factors applied to the trial's right-hand sides or columns.
static hipError_t cc_probe_solve(hipStream_t s, const CompCoarse* cc, const CcDims& D,
                                 void (*border)(const CompCoarse*, bool), void (*block)(const CompCoarse*)) {
  const dim3 gb((D.n_p + 3) / 4, D.blk, D.cnt), gv((D.n_s + 3) / 4, D.blk, D.cnt);
  for (int last = 0; last <= !D.form_p; ++last) {
    border<<<gb, 256, 0, s>>>(cc, last != 0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  block<<<gv, 256, 0, s>>>(cc);
  return hipGetLastError();
}

// After the Schur chain: S^-1, P, G and the verdicts.
static hipError_t cc_finish(hipStream_t s, const CompCoarse* cc, const CcDims& D) {
  const unsigned cols = (D.n_p + 255) / 256;
  k_cc_g<<<dim3((D.n + kRows - 1) / kRows, cols, D.cnt * D.blk * D.nc), 256, 0, s>>>(cc, D.nc,
                                                                                   D.blk);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_cc_collect_s<<<dim3(D.n_p, D.blk, D.cnt), 256, 0, s>>>(cc);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (D.form_p) {
    k_cc_p<<<dim3((D.n_s + kCcTile - 1) / kCcTile, (D.n_p + kCcTile - 1) / kCcTile, D.cnt * D.blk),
             256, 0, s>>>(cc, D.blk);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (D.form_x || D.form_c) {
    const unsigned tiles = (D.n_s + kCcTile - 1) / kCcTile;
    k_cc_x<<<dim3(tiles, tiles, D.cnt * D.blk), 256, 0, s>>>(cc, D.blk);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = cc_probe_solve(s, cc, D, k_cc_probe_p<false>, k_cc_probe_u<false>)) != hipSuccess) return e;
  k_cc_probe_r<<<dim3((D.n_s + 3) / 4, D.blk, D.cnt), 256, 0, s>>>(cc);
  return hipGetLastError();
}

hipError_t launch_cc_finish(hipStream_t s, const CompCoarse* cc, const CcDims& D) {
  return cc_slices(cc, D, [&](const CompCoarse* c, const CcDims& S) { return cc_finish(s, c, S); });
}

hipError_t launch_cc_second(hipStream_t s, const CompCoarse* cc, const CcDims& D) {
  return cc_slices(cc, D, [&](const CompCoarse* c, const CcDims& S) {
    return cc_probe_solve(s, c, S, k_cc_probe_p<true>, k_cc_probe_u<true>);
  });
}

hipError_t launch_cc_apply(hipStream_t s, const CompCoarse* cc, const CcDims& D, bool transposed,
                           const double* r, double* d) {
  if (!D.form_c) return hipErrorInvalidValue;
  const dim3 row((D.n_s + 3) / 4, 1, D.cnt), col((D.n_s + 15) / 16, 1, D.cnt);
#define STV_CC(B)                                                               \
  case B:                                                                       \
    if (transposed) launch(k_cc_apply_t<B>, col, dim3(1024), 0, s, cc, r, d);   \
    else launch(k_cc_apply<B>, row, dim3(256), 0, s, cc, r, d);                 \
    break;
  switch (D.b) {
    STV_CC(2) STV_CC(3) STV_CC(4)
    default: return hipErrorInvalidValue;
  }
#undef STV_CC
  return hipGetLastError();
}

hipError_t launch_cc_solve(hipStream_t s, const CompCoarse* cc, const CcDims& D, int set,
                           const double* r, double* d) {
  const dim3 gp(D.n_p, D.blk, D.cnt), gu((D.n_s + 3) / 4, 1, D.cnt), block(256);
#define STV_CC(B)                                                       \
  case B:                                                               \
    launch(k_cc_solve_p<B>, gp, block, 0, s, cc, set, r);                    \
    if (!D.form_p) launch(k_cc_solve_s, gp, block, 0, s, cc, set);           \
    launch(k_cc_solve_u<B>, gu, block, 0, s, cc, set, r, d);                 \
    break;
  switch (D.b) {
    STV_CC(1) STV_CC(2) STV_CC(3) STV_CC(4)
    default: return hipErrorInvalidValue;
  }
#undef STV_CC
  return hipGetLastError();
}

}  // namespace stv
