// Level kernels of the V-cycle: the block-sparse level residual, the Vanka
// cell sweep and the grid transfers.  Vectors are FP64 and time-inner
// (x[s*B + l], B = k+1 temporal DoFs per spatial DoF).
#include "stv_internal.h"
#include "wave.h"

namespace stv {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Partner value for lane ^ M inside a row of 16 lanes (M <= 8): DPP lane
// permutations (xor 1, xor 2 as quad permutations, xor 8 as a rotation of the
// row by 8) and, for xor 4, a swizzle in bit-mask mode.  Every source lane
// is inside the row, so the permutations need no old value.
template <int M>
__device__ __forceinline__ int xor_i32(int v) {
  static_assert(M == 1 || M == 2 || M == 4 || M == 8, "inside a row");
  if constexpr (M == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
  if constexpr (M == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
  if constexpr (M == 8) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true);  // row_ror:8
  return __builtin_amdgcn_ds_swizzle(v, 0x101F);                                   // xor 4
}

template <int M>
__device__ __forceinline__ double xor_lane(double v) {
  const int lo = xor_i32<M>(__double2loint(v));
  const int hi = xor_i32<M>(__double2hiint(v));
  return __hiloint2double(hi, lo);
}

template <int M>
__device__ __forceinline__ float xor_lane(float v) {
  return __int_as_float(xor_i32<M>(__float_as_int(v)));
}

// x, y <- the lanes with bit M clear keep x and receive y's values of the
// partner lanes (lane ^ M) in y, and vice versa: one v_permlane{16,32}_swap
// per 32-bit word (M = 16: odd rows of x with even rows of y; M = 32: upper
// half of x with lower half of y).  Afterwards x + y is, in every lane, its
// own kept value plus its partner's sent one.
template <int M>
__device__ __forceinline__ void swap_words(unsigned& x, unsigned& y) {
  static_assert(M == 16 || M == 32, "across rows");
  if constexpr (M == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    x = r[0];
    y = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    x = r[0];
    y = r[1];
  }
}

template <int M>
__device__ __forceinline__ void swap_halves(double& x, double& y) {
  unsigned xl = (unsigned)__double2loint(x), xh = (unsigned)__double2hiint(x);
  unsigned yl = (unsigned)__double2loint(y), yh = (unsigned)__double2hiint(y);
  swap_words<M>(xl, yl);
  swap_words<M>(xh, yh);
  x = __hiloint2double((int)xh, (int)xl);
  y = __hiloint2double((int)yh, (int)yl);
}

template <int M>
__device__ __forceinline__ void swap_halves(float& x, float& y) {
  unsigned xw = __float_as_uint(x), yw = __float_as_uint(y);
  swap_words<M>(xw, yw);
  x = __uint_as_float(xw);
  y = __uint_as_float(yw);
}

// Transpose-reduce (FP64 or FP32 values): NV (a power of two, 4..64) per-lane
// partial sums are summed over the wavefront; afterwards the lanes L with
// L / (64 / NV) == v hold the total of value v.  Each halving step exchanges
// half of the values with the partner lane, so the cost is about
// NV + log2(64 / NV) exchanges, done without LDS: across rows by lane-half
// swaps, inside a row by DPP and swizzle.  LIVE marks the values that can be
// nonzero (bit v for value v): a pair of slots that are both known to be zero
// is not exchanged, which saves the padding of outputs per row up to a power
// of two.
template <int M, unsigned long long NEXT, int T, int H, int NV, typename V>
__device__ __forceinline__ void fold_swap_pairs(V (&p)[NV], int lane) {
  if constexpr (T < H) {
    if constexpr (((NEXT >> T) & 1ull) == 0) {
      p[T] = V(0);
    } else if constexpr (M >= 16) {
      V x = p[T], y = p[T + H];
      swap_halves<M>(x, y);
      p[T] = x + y;
    } else {
      const bool hi = lane & M;
      const V keep = hi ? p[T + H] : p[T];
      const V send = hi ? p[T] : p[T + H];
      p[T] = keep + xor_lane<M>(send);
    }
    fold_swap_pairs<M, NEXT, T + 1, H, NV>(p, lane);
  }
}

template <int CNT, int M, int NV, unsigned long long LIVE, typename V>
__device__ __forceinline__ void fold_swap_level(V (&p)[NV], int lane) {
  if constexpr (CNT > 1) {
    constexpr int H = CNT / 2;
    constexpr unsigned long long NEXT = (LIVE | (LIVE >> H)) & ((1ull << H) - 1ull);
    fold_swap_pairs<M, NEXT, 0, H, NV>(p, lane);
    fold_swap_level<H, M / 2, NV, NEXT>(p, lane);
  }
}

template <int NV, unsigned long long LIVE = (NV >= 64 ? ~0ull : (1ull << NV) - 1ull),
          typename V>
__device__ __forceinline__ V fold_swap(V (&p)[NV], int lane) {
  static_assert(NV >= 4 && NV <= 64, "the final exchanges stay inside a row");
  fold_swap_level<NV, 32, NV, LIVE>(p, lane);
  V u = p[0];
  if constexpr (NV <= 4) u += xor_lane<8>(u);
  if constexpr (NV <= 8) u += xor_lane<4>(u);
  if constexpr (NV <= 16) u += xor_lane<2>(u);
  if constexpr (NV <= 32) u += xor_lane<1>(u);
  return u;
}

// Live-value mask of G groups of P slots of which the first U are used.
constexpr unsigned long long live_slots(int G, int P, int U) {
  unsigned long long m = 0;
  for (int g = 0; g < G; ++g)
    for (int o = 0; o < U; ++o) m |= 1ull << (g * P + o);
  return m;
}

// Level residual from the spatial factors of an operator whose blocks are
// C[i][l] M + delta_il tw[i] A (time-independent coefficients): per block only
// the two scalars m = M(s, s') and a = A(s, s') are streamed.  LPR lanes per
// block row (64 / LPR rows per wavefront): lane `sub` of a row takes the
// row's blocks sub, sub + LPR, ..., U of them per round, with every load of a
// round issued before the first is used (indices clamped into the list, the
// blocks past its end weighted by zero, instead of branches), and keeps only
// the B partial sums of its own row; the row's lanes then add their sums
// (butterfly over the LPR lanes).  LPR x U slots per round are matched to
// the typical row length by the autotuner.
struct KronCoef { double C[16]; double tw[4]; };

// Sum of acc[0 .. NV) over the LPR lanes of a row, in every lane of the row.
template <int LPR, int NV>
__device__ __forceinline__ void row_sum(double (&acc)[NV]) {
#pragma unroll
  for (int off = LPR / 2; off >= 1; off >>= 1)
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] += __shfl_xor(acc[i], off, 64);
}

// The first nv of NV entries y[o0 ..] = r + sx acc, entry e from lane e % LPR.
template <int LPR, int NV, int E0 = 0>
__device__ __forceinline__ void row_store(const double (&acc)[NV], int nv, int sub, int64_t o0,
                                          const double* __restrict__ r, double* __restrict__ y,
                                          double sx) {
  constexpr int CNT = NV - E0 < LPR ? NV - E0 : LPR;
  // values first, then the choice: a conditional read of acc would be turned
  // into one read at a run-time index, which moves acc out of registers
  double v[CNT];
#pragma unroll
  for (int e = 0; e < CNT; ++e) v[e] = acc[E0 + e];
  double s = v[0];
#pragma unroll
  for (int e = 1; e < CNT; ++e) s = (sub == e) ? v[e] : s;
  if (sub < CNT && E0 + sub < nv) {
    const int64_t o = o0 + E0 + sub;
    y[o] = r ? fma(sx, s, r[o]) : sx * s;
  }
  if constexpr (E0 + LPR < NV) row_store<LPR, NV, E0 + LPR>(acc, nv, sub, o0, r, y, sx);
}

// Level residual y = r + sx J x  (sx = -1: r - J x; r == nullptr: sx J x) from
// the blocks.  LPR lanes per block row, a block per H lanes (B / H of its rows
// each), U blocks per lane and round, every load of a round issued before the
// first is used (as in k_spmv_kron).  Bound by HBM, given that: the rows of a
// 2d operator have 12 to 62 blocks, and a loop over them with a block column
// per lane spent two dependent latencies per round of 64 / B blocks (untuned
// shapes: 2d 256x64 dG(1), 148 MB, 41.7 -> 24.3 us, partly from the last-level
// cache; 2d 128x64 dG(2), 154 MB, 30.8 -> 24.6; 3d 32x8x8 dG(1), 168 MB, 28.9
// -> 26.7; 3d 32x16x8 dG(0), 112 MB, 30.6 -> 22.6).
template <int B, int H, int LPR, int U>
__global__ void __launch_bounds__(256) k_spmv_rows(const int32_t* __restrict__ rowptr,
                                                   const int32_t* __restrict__ col,
                                                   const double* __restrict__ val,
                                                   const double* __restrict__ r,
                                                   const double* __restrict__ x,
                                                   double* __restrict__ y, int32_t n_rows,
                                                   double sx) {
  constexpr int RPWV = 64 / LPR, BH = B / H, NQ = LPR / H;
  static_assert(B % H == 0 && (H & (H - 1)) == 0 && NQ >= BH);
  const int lane = threadIdx.x & 63, sub = lane % LPR, part = sub % H, slot = sub / H;
  const int row = (blockIdx.x * 4 + (threadIdx.x >> 6)) * RPWV + lane / LPR;
  const bool live = row < n_rows;
  const int rr = live ? row : n_rows - 1;
  double acc[BH];
#pragma unroll
  for (int i = 0; i < BH; ++i) acc[i] = 0.0;
  const int32_t q1 = rowptr[rr + 1];
  for (int32_t q0 = rowptr[rr]; q0 < q1; q0 += U * NQ) {
    int64_t c[U];
    double f[U][BH * B];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t q = min(q0 + slot + u * NQ, q1 - 1);
      c[u] = col[q];
      const double* vb = val + (int64_t)q * (B * B) + part * (BH * B);
#pragma unroll
      for (int e = 0; e < BH * B; ++e) f[u][e] = vb[e];
    }
    double xl[U][B];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int l = 0; l < B; ++l) xl[u][l] = x[c[u] * B + l];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < BH; ++i) {
        double s = acc[i];
#pragma unroll
        for (int l = 0; l < B; ++l) s = fma(f[u][i * B + l], xl[u][l], s);
        acc[i] = q0 + slot + u * NQ < q1 ? s : acc[i];
      }
  }
#pragma unroll
  for (int off = LPR / 2; off >= H; off >>= 1)
#pragma unroll
    for (int i = 0; i < BH; ++i) acc[i] += __shfl_xor(acc[i], off, 64);
  // entry part * BH + slot from the lane of that part and slot
  double s = acc[0];
#pragma unroll
  for (int i = 1; i < BH; ++i) s = slot == i ? acc[i] : s;
  if (live && slot < BH) {
    const int64_t o = (int64_t)row * B + part * BH + slot;
    y[o] = r ? fma(sx, s, r[o]) : sx * s;
  }
}

template <int B>
static hipError_t spmv_b(hipStream_t s, const DevLevel& L, bool tr, const double* r,
                         const double* x, double* y, double sx) {
  const int32_t* rp = tr ? L.rowptr_t : L.rowptr;
  const int32_t* cl = tr ? L.col_t : L.col;
  const double* vl = tr ? L.val_t : L.val;
  if (!rp || !cl || !vl) return hipErrorInvalidValue;
#define STV_SPMV(H, LPR, U)                                                                       \
  launch(k_spmv_rows<B, H, LPR, U>, dim3((L.n_s + 256 / LPR - 1) / (256 / LPR)), dim3(256), 0, s, \
         rp, cl, vl, r, x, y, L.n_s, sx)
  // shapes 1 to 4 (more act as 4).  A block of order 4 is two lines, which four
  // lanes read together (2d 128x32 dG(3): 21 us, one lane per block 28 us).
  // Shape 2 is what is used without tuning: two rounds of 16 lanes take most 2d
  // rows at once; rows of over 48 blocks on average (3d) have 32 lanes
  // (168 MB of dG(1) 27.6 -> 26.7 us, 177 MB of dG(2) 31.6 -> 29.9 us; dG(0),
  // of an eighth of the bytes per block, 22.6 -> 27.4 us and so does not).
  int shape = L.spmv_rpw;
  if (B > 1 && shape <= 2 && L.nnzb > 48 * (int64_t)L.n_s) shape = 3 - shape;
  if constexpr (B == 4) {
    switch (shape) {
      case 1: STV_SPMV(4, 64, 2); break;
      case 2: STV_SPMV(4, 32, 2); break;
      case 3: STV_SPMV(2, 32, 1); break;
      default: STV_SPMV(2, 16, 2); break;
    }
  } else {
    switch (shape) {
      case 1: STV_SPMV(1, 32, 2); break;
      case 2: STV_SPMV(1, 16, 2); break;
      case 3: STV_SPMV(1, 32, 1); break;
      default: STV_SPMV(1, 8, 4); break;
    }
  }
#undef STV_SPMV
  return hipGetLastError();
}

hipError_t launch_spmv(hipStream_t s, int b, const DevLevel& L, const double* r, const double* x,
                       double* y, double sx, bool transposed) {
  switch (b) {
    case 1: return spmv_b<1>(s, L, transposed, r, x, y, sx);
    case 2: return spmv_b<2>(s, L, transposed, r, x, y, sx);
    case 3: return spmv_b<3>(s, L, transposed, r, x, y, sx);
    case 4: return spmv_b<4>(s, L, transposed, r, x, y, sx);
  }
  return hipErrorInvalidValue;
}

// acc += the (m, a) blocks [q0, q1) of one row (list position in ma and col).
template <int B, int LPR, int U, int NV>
__device__ __forceinline__ void row_pairs(int32_t q0, int32_t q1, int sub,
                                          const int32_t* __restrict__ col,
                                          const double2* __restrict__ ma,
                                          const double* __restrict__ x, const KronCoef& K,
                                          double (&acc)[NV]) {
  const int nit = (q1 - q0 + U * LPR - 1) / (U * LPR);
  for (int it = 0; it < nit; ++it) {
    const int32_t qb = q0 + it * U * LPR + sub;
    int64_t c[U];
    double m[U], a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t q = qb + u * LPR;
      const bool v = q < q1;
      const int32_t qc = v ? q : q1 - 1;
      c[u] = col[qc];
      const double2 f = ma[qc];
      m[u] = v ? f.x : 0.0;
      a[u] = v ? f.y : 0.0;
    }
    double xl[U][B];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int l = 0; l < B; ++l) xl[u][l] = x[c[u] * B + l];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < B; ++i) {
        double ci = 0.0;
#pragma unroll
        for (int l = 0; l < B; ++l) ci = fma(K.C[i * B + l], xl[u][l], ci);
        acc[i] = fma(m[u], ci, fma(a[u] * K.tw[i], xl[u][i], acc[i]));
      }
  }
}

template <int B, int LPR, int U>
__global__ void __launch_bounds__(256) k_spmv_kron(const int32_t* __restrict__ rowptr,
                                                   const int32_t* __restrict__ col,
                                                   const double2* __restrict__ ma,
                                                   const double* __restrict__ r,
                                                   const double* __restrict__ x,
                                                   double* __restrict__ y, int32_t n_rows,
                                                   double sx, KronCoef K) {
  constexpr int RPWV = 64 / LPR;
  const int lane = threadIdx.x & 63, sub = lane % LPR;
  const int row = (blockIdx.x * 4 + (threadIdx.x >> 6)) * RPWV + lane / LPR;
  const bool live = row < n_rows;
  const int rr = live ? row : n_rows - 1;
  double acc[B];
#pragma unroll
  for (int i = 0; i < B; ++i) acc[i] = 0.0;
  row_pairs<B, LPR, U>(rowptr[rr], rowptr[rr + 1], sub, col, ma, x, K, acc);
  row_sum<LPR>(acc);
  if (live) row_store<LPR>(acc, B, sub, (int64_t)row * B, r, y, sx);
}

// The same residual from row groups (DevLevel::kg).  The velocity rows of
// one node repeat each other: D consecutive rows whose (m, a) values are
// equal and whose columns differ by the component only are read once for all
// D; their coupling blocks (m = 0, the same columns in every row) carry D
// values per column, and the D + 1 consecutive pressure rows of a cell one
// column per node and (D + 1) D values.  Rows that fit neither (nodes on a
// wall, whose normal component has its own boundary terms; operators of
// another structure) are read singly, their blocks with m != 0 as (m, a),
// the others as a.  The kernel streams its lists once and is bound by HBM:
// per node pair 20 bytes instead of 20 D (3d: 1.3 instead of 3.0 GB on the
// 128x24x24 level), and per pair of loads D rows of work instead of one.
// The D B sums of a velocity group are M x and A x apart, combined with C and
// tw once per row instead of once per block.  Blocks of the grid are split
// over the three kinds; lanes and rounds as in k_spmv_kron.  Measured on one
// MI355X, best shape, rows read singly -> groups: 3d 128x24x24 dG(1)
// 648 -> 355 us, 2d 512x128 dG(2) 77 -> 45 us, 2d 256x64 dG(1) 15.4 -> 11.6
// us; levels under about 10,000 rows are at the launch latency either way.
template <int B, int D, int LPR, int U>
__global__ void __launch_bounds__(256) k_spmv_group(KronGroups G, const double* __restrict__ r,
                                                    const double* __restrict__ x,
                                                    double* __restrict__ y, double sx,
                                                    KronCoef K) {
  constexpr int RPWV = 64 / LPR;
  const int lane = threadIdx.x & 63, sub = lane % LPR;
  const int wrow = (threadIdx.x >> 6) * RPWV + lane / LPR;
  const int blk = blockIdx.x;
  constexpr int NV = (D + 1) * B;   // entries of the largest group
  double acc[NV];
#pragma unroll
  for (int e = 0; e < NV; ++e) acc[e] = 0.0;
  int64_t row;
  int nv;
  bool live;
  if (blk < G.nb_v) {
    const int g = blk * 4 * RPWV + wrow;
    live = g < G.n_v;
    const int gg = live ? g : G.n_v - 1;
    double am[D * B], aa[D * B];
#pragma unroll
    for (int e = 0; e < D * B; ++e) am[e] = aa[e] = 0.0;
    {
      const int32_t q0 = G.vp1[gg], q1 = G.vp1[gg + 1];
      const int nit = (q1 - q0 + U * LPR - 1) / (U * LPR);
      for (int it = 0; it < nit; ++it) {
        const int32_t qb = q0 + it * U * LPR + sub;
        int64_t c[U];
        double2 f[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int32_t q = qb + u * LPR;
          const bool v = q < q1;
          const int32_t qc = v ? q : q1 - 1;
          c[u] = G.vc1[qc];
          const double2 w = G.vma[qc];
          f[u].x = v ? w.x : 0.0;
          f[u].y = v ? w.y : 0.0;
        }
        double xl[U][D * B];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int e = 0; e < D * B; ++e) xl[u][e] = x[c[u] * B + e];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int e = 0; e < D * B; ++e) {
            am[e] = fma(f[u].x, xl[u][e], am[e]);
            aa[e] = fma(f[u].y, xl[u][e], aa[e]);
          }
      }
    }
    {
      const int32_t q0 = G.vp2[gg], q1 = G.vp2[gg + 1];
      const int nit = (q1 - q0 + U * LPR - 1) / (U * LPR);
      for (int it = 0; it < nit; ++it) {
        const int32_t qb = q0 + it * U * LPR + sub;
        int64_t c[U];
        double f[U][D];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int32_t q = qb + u * LPR;
          const bool v = q < q1;
          const int32_t qc = v ? q : q1 - 1;
          c[u] = G.vc2[qc];
#pragma unroll
          for (int e = 0; e < D; ++e) {
            const double w = G.va2[(int64_t)qc * D + e];
            f[u][e] = v ? w : 0.0;
          }
        }
        double xl[U][B];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int l = 0; l < B; ++l) xl[u][l] = x[c[u] * B + l];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int e = 0; e < D; ++e)
#pragma unroll
            for (int l = 0; l < B; ++l) aa[e * B + l] = fma(f[u][e], xl[u][l], aa[e * B + l]);
      }
    }
#pragma unroll
    for (int e = 0; e < D; ++e)
#pragma unroll
      for (int i = 0; i < B; ++i) {
        double s = K.tw[i] * aa[e * B + i];
#pragma unroll
        for (int l = 0; l < B; ++l) s = fma(K.C[i * B + l], am[e * B + l], s);
        acc[e * B + i] = s;
      }
    row = G.vrow[gg];
    nv = D * B;
  } else if (blk < G.nb_v + G.nb_p) {
    const int g = (blk - G.nb_v) * 4 * RPWV + wrow;
    live = g < G.n_p;
    const int gg = live ? g : G.n_p - 1;
    const int32_t q0 = G.pp[gg], q1 = G.pp[gg + 1];
    for (int32_t q = q0 + sub; q < q1; q += LPR) {
      const int64_t c = G.pc[q];
      double f[(D + 1) * D], xl[D * B];
#pragma unroll
      for (int e = 0; e < (D + 1) * D; ++e) f[e] = G.pa[(int64_t)q * ((D + 1) * D) + e];
#pragma unroll
      for (int e = 0; e < D * B; ++e) xl[e] = x[c * B + e];
#pragma unroll
      for (int m = 0; m <= D; ++m)
#pragma unroll
        for (int e = 0; e < D; ++e)
#pragma unroll
          for (int l = 0; l < B; ++l)
            acc[m * B + l] = fma(f[m * D + e], xl[e * B + l], acc[m * B + l]);
    }
#pragma unroll
    for (int m = 0; m <= D; ++m)
#pragma unroll
      for (int i = 0; i < B; ++i) acc[m * B + i] *= K.tw[i];
    row = G.prow[gg];
    nv = NV;
  } else {
    const int g = (blk - G.nb_v - G.nb_p) * 4 * RPWV + wrow;
    live = g < G.n_s;
    const int gg = live ? g : G.n_s - 1;
    row_pairs<B, LPR, U>(G.sp1[gg], G.sp1[gg + 1], sub, G.sc1, G.sma, x, K, acc);
    // blocks without a mass entry: a only
    const int32_t q0 = G.sp2[gg], q1 = G.sp2[gg + 1];
    const int nit = (q1 - q0 + U * LPR - 1) / (U * LPR);
    for (int it = 0; it < nit; ++it) {
      const int32_t qb = q0 + it * U * LPR + sub;
      int64_t c[U];
      double a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int32_t q = qb + u * LPR;
        const bool v = q < q1;
        const int32_t qc = v ? q : q1 - 1;
        c[u] = G.sc2[qc];
        const double f = G.sa2[qc];
        a[u] = v ? f : 0.0;
      }
      double xl[U][B];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int l = 0; l < B; ++l) xl[u][l] = x[c[u] * B + l];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < B; ++i) acc[i] = fma(a[u] * K.tw[i], xl[u][i], acc[i]);
    }
    row = G.srow[gg];
    nv = B;
  }
  row_sum<LPR>(acc);
  if (live) row_store<LPR>(acc, nv, sub, row * B, r, y, sx);
}

// residual shapes from the factors: (lanes per block row, blocks per lane and
// round), 1-6 on the plain rows, 7-12 the same on the row groups
static constexpr int kKronShapes = 12;
static constexpr int kKronLpr[kKronShapes] = {4, 8, 8, 16, 16, 32, 4, 8, 8, 16, 16, 32};

int residual_shapes(const DevLevel& L) { return L.kron_ma ? kKronShapes : 4; }

template <int B>
static hipError_t spmv_kron_b(hipStream_t s, const DevLevel& L, const double* r, const double* x,
                              double* y, double sx) {
  KronCoef K{};
  for (int e = 0; e < B * B; ++e) K.C[e] = L.kron_C[e];
  for (int e = 0; e < B; ++e) K.tw[e] = L.kron_tw[e];
  const int sh = L.spmv_rpw - 1;
  if (sh < 0 || sh >= kKronShapes) return hipErrorInvalidValue;
  const int rows_per_wg = 4 * (64 / kKronLpr[sh]);
  const double2* ma = (const double2*)L.kron_ma;
  if (sh < kKronShapes / 2) {
    const dim3 grid((L.n_s + rows_per_wg - 1) / rows_per_wg), block(256);
#define STV_KRON(S, LP, UU)                                                                  \
  case S:                                                                                   \
    launch(k_spmv_kron<B, LP, UU>, grid, block, 0, s, L.rowptr, L.col, ma, r, x, y, L.n_s,  \
           sx, K);                                                                          \
    break;
    switch (sh) {
      STV_KRON(0, 4, 4) STV_KRON(1, 8, 3) STV_KRON(2, 8, 4)
      STV_KRON(3, 16, 2) STV_KRON(4, 16, 4) STV_KRON(5, 32, 2)
    }
#undef STV_KRON
    return hipGetLastError();
  }
  KronGroups G = L.kg;
  if (!G.vp1) return hipErrorInvalidValue;
  G.nb_v = (G.n_v + rows_per_wg - 1) / rows_per_wg;
  G.nb_p = (G.n_p + rows_per_wg - 1) / rows_per_wg;
  const dim3 grid(G.nb_v + G.nb_p + (G.n_s + rows_per_wg - 1) / rows_per_wg), block(256);
#define STV_GROUP(S, LP, UU)                                                                 \
  case S:                                                                                   \
    if (L.n_ls == 21)                                                                       \
      launch(k_spmv_group<B, 2, LP, UU>, grid, block, 0, s, G, r, x, y, sx, K);             \
    else                                                                                    \
      launch(k_spmv_group<B, 3, LP, UU>, grid, block, 0, s, G, r, x, y, sx, K);             \
    break;
  switch (sh) {
    STV_GROUP(6, 4, 4) STV_GROUP(7, 8, 3) STV_GROUP(8, 8, 4)
    STV_GROUP(9, 16, 2) STV_GROUP(10, 16, 4) STV_GROUP(11, 32, 2)
  }
#undef STV_GROUP
  return hipGetLastError();
}

hipError_t launch_spmv_kron(hipStream_t s, int b, const DevLevel& L, const double* r,
                            const double* x, double* y, double sx) {
  switch (b) {
    case 1: return spmv_kron_b<1>(s, L, r, x, y, sx);
    case 2: return spmv_kron_b<2>(s, L, r, x, y, sx);
    case 3: return spmv_kron_b<3>(s, L, r, x, y, sx);
    case 4: return spmv_kron_b<4>(s, L, r, x, y, sx);
  }
  return hipErrorInvalidValue;
}

// ma[q] = (m[q], a[q])
__global__ void k_interleave(const double* __restrict__ m, const double* __restrict__ a,
                             double2* __restrict__ ma, int64_t n) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
       q += (int64_t)gridDim.x * blockDim.x)
    ma[q] = make_double2(m[q], a[q]);
}

hipError_t launch_interleave(hipStream_t s, const double* m, const double* a, double* ma,
                             int64_t n) {
  k_interleave<<<2048, 256, 0, s>>>(m, a, (double2*)ma, n);
  return hipGetLastError();
}

// What rows i .. of a level can be grouped as, one wavefront per row i:
// kind bit 0: rows i .. i + D - 1 are a velocity group; bit 1: rows i .. i + D
// a pressure group (k_spmv_group); n1[i] = row i's blocks with m != 0.  The
// conditions are exact (equal values, equal lengths), so a group's rows give
// the sums that the single rows give, to rounding: C and tw are applied once
// per row to a group's sums, once per block to a single row's.
template <int D>
__global__ void __launch_bounds__(256) k_group_classify(const int32_t* __restrict__ rowptr,
                                                        const int32_t* __restrict__ col,
                                                        const double2* __restrict__ ma,
                                                        int32_t n_rows,
                                                        uint8_t* __restrict__ kind,
                                                        int32_t* __restrict__ n1) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const int32_t q0 = rowptr[row], len = rowptr[row + 1] - q0;
  int cnt = 0;
  for (int32_t e = lane; e < len; e += 64) cnt += ma[q0 + e].x != 0.0;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
  bool v = cnt > 0 && row + D <= n_rows;
  for (int c = 1; c < D && v; ++c) {
    const int32_t qc = rowptr[row + c];
    bool ok = rowptr[row + c + 1] - qc == len;
    for (int32_t e = lane; ok && e < len; e += 64) {
      const double2 f = ma[q0 + e], g = ma[qc + e];
      if (f.x != 0.0) ok = col[qc + e] == col[q0 + e] + c && g.x == f.x && g.y == f.y;
      else ok = col[qc + e] == col[q0 + e] && g.x == 0.0;
    }
    v = __all(ok);
  }
  bool p = cnt == 0 && row + D + 1 <= n_rows && len % D == 0;
  for (int c = 0; c <= D && p; ++c) {
    const int32_t qc = rowptr[row + c];
    bool ok = rowptr[row + c + 1] - qc == len;
    for (int32_t e = lane; ok && e < len; e += 64)
      ok = ma[qc + e].x == 0.0 && col[qc + e] == col[q0 + e] &&
           col[q0 + e] == col[q0 + e / D * D] + e % D;
    p = __all(ok);
  }
  if (lane == 0) {
    kind[row] = (uint8_t)((v ? 1 : 0) | (p ? 2 : 0));
    n1[row] = cnt;
  }
}

// Fills the lists of the groups whose rows and pointers are in G, one
// wavefront per group (velocity groups first, then pressure groups, then
// single rows); list order is block order.
template <int D>
__global__ void __launch_bounds__(256) k_group_fill(const int32_t* __restrict__ rowptr,
                                                    const int32_t* __restrict__ col,
                                                    const double2* __restrict__ ma,
                                                    KronGroups G) {
  const int lane = threadIdx.x & 63;
  int g = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (g >= G.n_v + G.n_p + G.n_s) return;
  if (g >= G.n_v && g < G.n_v + G.n_p) {
    g -= G.n_v;
    const int32_t row = G.prow[g], q0 = rowptr[row], len = rowptr[row + 1] - q0, o = G.pp[g];
    for (int32_t e = lane; e < len; e += 64) {
      if (e % D == 0) const_cast<int32_t*>(G.pc)[o + e / D] = col[q0 + e];
      for (int m = 0; m <= D; ++m)
        const_cast<double*>(G.pa)[((int64_t)o + e / D) * ((D + 1) * D) + m * D + e % D] =
            ma[rowptr[row + m] + e].y;
    }
    return;
  }
  const bool vel = g < G.n_v;
  if (!vel) g -= G.n_v + G.n_p;
  const int32_t row = vel ? G.vrow[g] : G.srow[g];
  int32_t o1 = vel ? G.vp1[g] : G.sp1[g], o2 = vel ? G.vp2[g] : G.sp2[g];
  int32_t* c1 = const_cast<int32_t*>(vel ? G.vc1 : G.sc1);
  int32_t* c2 = const_cast<int32_t*>(vel ? G.vc2 : G.sc2);
  double2* m1 = const_cast<double2*>(vel ? G.vma : G.sma);
  double* a2 = const_cast<double*>(vel ? G.va2 : G.sa2);
  const int nv = vel ? D : 1;
  const int32_t q0 = rowptr[row], len = rowptr[row + 1] - q0;
  for (int32_t e0 = 0; e0 < len; e0 += 64) {
    const int32_t e = e0 + lane;
    const bool in = e < len;
    const double2 f = in ? ma[q0 + e] : make_double2(0.0, 0.0);
    const bool one = in && f.x != 0.0, two = in && f.x == 0.0;
    const uint64_t b1 = __builtin_amdgcn_ballot_w64(one), b2 = __builtin_amdgcn_ballot_w64(two);
    const uint64_t below = (1ull << lane) - 1ull;
    if (one) {
      const int32_t q = o1 + __popcll(b1 & below);
      c1[q] = col[q0 + e];
      m1[q] = f;
    }
    if (two) {
      const int32_t q = o2 + __popcll(b2 & below);
      c2[q] = col[q0 + e];
      for (int c = 0; c < nv; ++c) a2[(int64_t)q * nv + c] = ma[rowptr[row + c] + e].y;
    }
    o1 += __popcll(b1);
    o2 += __popcll(b2);
  }
}

hipError_t launch_group_classify(hipStream_t s, const DevLevel& L, const double* ma,
                                 uint8_t* kind, int32_t* n1) {
  const dim3 grid((L.n_s + 3) / 4), block(256);
  if (L.n_ls == 21)
    k_group_classify<2><<<grid, block, 0, s>>>(L.rowptr, L.col, (const double2*)ma, L.n_s, kind, n1);
  else
    k_group_classify<3><<<grid, block, 0, s>>>(L.rowptr, L.col, (const double2*)ma, L.n_s, kind, n1);
  return hipGetLastError();
}

hipError_t launch_group_fill(hipStream_t s, const DevLevel& L, const double* ma,
                             const KronGroups& G) {
  const dim3 grid((G.n_v + G.n_p + G.n_s + 3) / 4), block(256);
  if (L.n_ls == 21)
    k_group_fill<2><<<grid, block, 0, s>>>(L.rowptr, L.col, (const double2*)ma, G);
  else
    k_group_fill<3><<<grid, block, 0, s>>>(L.rowptr, L.col, (const double2*)ma, G);
  return hipGetLastError();
}

// Largest deviation of the stored blocks from C m + delta tw a, and the
// largest block entry: one (deviation, magnitude) pair per workgroup.
template <int B>
__global__ void __launch_bounds__(256) k_kron_check(const double* __restrict__ val,
                                                    const double2* __restrict__ ma,
                                                    int64_t nnzb, KronCoef K,
                                                    double* __restrict__ partial) {
  __shared__ double sd[4], sm[4];
  double dev = 0.0, mag = 0.0;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nnzb;
       q += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
    for (int i = 0; i < B; ++i)
#pragma unroll
      for (int l = 0; l < B; ++l) {
        const double v = val[q * B * B + i * B + l];
        const double2 f = ma[q];
        const double rec = K.C[i * B + l] * f.x + (i == l ? K.tw[i] * f.y : 0.0);
        dev = fmax(dev, fabs(v - rec));
        mag = fmax(mag, fabs(v));
      }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    dev = fmax(dev, __shfl_xor(dev, off, 64));
    mag = fmax(mag, __shfl_xor(mag, off, 64));
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) { sd[wv] = dev; sm[wv] = mag; }
  __syncthreads();
  if (threadIdx.x == 0) {
    partial[2 * blockIdx.x] = fmax(fmax(sd[0], sd[1]), fmax(sd[2], sd[3]));
    partial[2 * blockIdx.x + 1] = fmax(fmax(sm[0], sm[1]), fmax(sm[2], sm[3]));
  }
}

hipError_t launch_kron_check(hipStream_t s, int b, const DevLevel& L, const double* ma_,
                             const double* C, const double* tw, double* partial, int nblk) {
  const double2* ma = (const double2*)ma_;
  KronCoef K{};
  for (int e = 0; e < b * b; ++e) K.C[e] = C[e];
  for (int e = 0; e < b; ++e) K.tw[e] = tw[e];
  switch (b) {
    case 1: k_kron_check<1><<<nblk, 256, 0, s>>>(L.val, ma, L.nnzb, K, partial); break;
    case 2: k_kron_check<2><<<nblk, 256, 0, s>>>(L.val, ma, L.nnzb, K, partial); break;
    case 3: k_kron_check<3><<<nblk, 256, 0, s>>>(L.val, ma, L.nnzb, K, partial); break;
    case 4: k_kron_check<4><<<nblk, 256, 0, s>>>(L.val, ma, L.nnzb, K, partial); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Values of the transposed level matrix: block qt of J^T is the transpose of
// block src[qt] of J (the pattern of J^T is built on the host).
template <int B>
__global__ void k_bsr_transpose_vals(const double* __restrict__ val,
                                     const int32_t* __restrict__ src, double* __restrict__ val_t,
                                     int64_t nnzb) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nnzb * B * B) return;
  const int64_t qt = e / (B * B);
  const int ij = (int)(e - qt * (B * B));
  const int i = ij / B, l = ij - i * B;
  val_t[e] = val[(int64_t)src[qt] * (B * B) + l * B + i];
}

hipError_t launch_bsr_transpose_vals(hipStream_t s, int b, const double* val, const int32_t* src,
                                     double* val_t, int64_t nnzb) {
  const int64_t n = nnzb * b * b;
  const unsigned grid = (unsigned)((n + 255) / 256);
  switch (b) {
    case 1: k_bsr_transpose_vals<1><<<grid, 256, 0, s>>>(val, src, val_t, nnzb); break;
    case 2: k_bsr_transpose_vals<2><<<grid, 256, 0, s>>>(val, src, val_t, nnzb); break;
    case 3: k_bsr_transpose_vals<3><<<grid, 256, 0, s>>>(val, src, val_t, nnzb); break;
    case 4: k_bsr_transpose_vals<4><<<grid, 256, 0, s>>>(val, src, val_t, nnzb); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Vanka cell sweep.  One 64-lane wavefront per cell T (four cells per
// workgroup, no LDS, no barriers): lane j holds rho_T[j] for the columns
// j = lane + 64c of the cell-local order (alpha, l) -> alpha*B + l, gathered
// straight from the level residual.  The stored inverse rows are row-major,
// so each row is one contiguous, fully coalesced read.  Rows are taken G at
// a time with every load of a group issued before the first is used
// (indices clamped into the cell's block instead of branches, so that the
// loads do not serialise), and the G partial sums are folded by one
// transpose-reduce.  Last-writer form: only the rows of the DoFs the cell
// owns are computed; row r of the cell ends in lane r % 64, which also
// fetched the old iterate of that DoF at the start, and the cell's rows are
// stored in one pass (d_j += omega c_j, or = omega c_j for a zero initial
// iterate).  Every DoF has exactly one owner, so the stores are disjoint (no
// atomics, deterministic).  FULL: the store keeps every row of J_T^-1 and the
// owned ones are picked by their local index.  The row products and the
// transpose-reduce are in the precision of the store (FP32 products of an
// FP32 store and the residual rounded to FP32, summed in FP32), the update
// of the iterate in FP64.
template <int B, int NLS, typename TS, bool FULL>
__global__ void __launch_bounds__(256) k_vanka(const double* __restrict__ rho,
                                              double* __restrict__ d,
                                              const int32_t* __restrict__ csd,
                                              const int32_t* __restrict__ own_ptr,
                                              const uint8_t* __restrict__ own_loc,
                                              const int64_t* __restrict__ inv_off, int ld,
                                              const TS* __restrict__ store, double omega,
                                              int zero_init, int n_cells) {
  constexpr int N = B * NLS;
  constexpr int NC = (N + 63) / 64;        // 64-column chunks of a row
  constexpr int NOC = (NLS + 63) / 64;     // 64-lane chunks of the owned DoFs
  constexpr int RC = NC;                   // 64-lane chunks of the owned rows (R <= N)
  constexpr int G = NC == 1 ? 16 : 8;      // rows per group
  const int lane = threadIdx.x & 63;
  // one cell per wavefront and step; a grid smaller than the cell count makes
  // the launch persistent (each wavefront strides over the cells)
  // (the cell index is wave-uniform: its per-cell data sits in scalar registers)
  const int T0 = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  for (int T = T0; T < n_cells; T += gridDim.x * 4) {
    const int32_t* sd = csd + (int64_t)T * NLS;
    const int o0 = own_ptr[T];
    const int no = own_ptr[T + 1] - o0;
    if (no <= 0) continue;
    const int R = no * B;
    const TS* A = store + inv_off[T];
    double x[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = lane + 64 * c;
      const int jc = j < N ? j : N - 1;
      const int be = jc / B;
      const double v = rho[(int64_t)sd[be] * B + (jc - be * B)];
      x[c] = j < N ? v : 0.0;
    }
    // the row products are in the precision of the store (see k_vanka_dec)
    TS xs[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) xs[c] = (TS)x[c];
    // owned DoFs, lane = owned index: local index and spatial DoF
    int ol[NOC], gs[NOC];
#pragma unroll
    for (int c = 0; c < NOC; ++c) {
      const int k = lane + 64 * c;
      ol[c] = own_loc[o0 + (k < no ? k : no - 1)];
      gs[c] = sd[ol[c]];
    }
    // the rows this lane stores (r = lane + 64 rc): DoF index and old value
    int64_t gi[RC];
    double dold[RC], res[RC];
#pragma unroll
    for (int rc = 0; rc < RC; ++rc) {
      const int r = lane + 64 * rc;
      const int rcl = r < R ? r : R - 1;
      const int os = rcl / B;
      int g = __shfl(gs[0], os & 63, 64);
      if constexpr (NOC > 1) {
        const int g1 = __shfl(gs[NOC - 1], os & 63, 64);
        g = os < 64 ? g : g1;
      }
      gi[rc] = (int64_t)g * B + (rcl - os * B);
      dold[rc] = zero_init ? 0.0 : d[gi[rc]];
      res[rc] = 0.0;
    }
    for (int r0 = 0; r0 < R; r0 += G) {
      TS a[G][NC];
#pragma unroll
      for (int t = 0; t < G; ++t) {
        const int row = min(r0 + t, R - 1);
        int srow = row;
        if constexpr (FULL) {
          const int os = row / B;
          int l = __builtin_amdgcn_readlane(ol[0], os & 63);
          if constexpr (NOC > 1) {
            const int l1 = __builtin_amdgcn_readlane(ol[NOC - 1], os & 63);
            l = os < 64 ? l : l1;
          }
          srow = l * B + (row - os * B);
        }
        // offsets inside the cell's block fit 32 bits: the loads address
        // from the block's (wave-uniform) base
        const unsigned ro = (unsigned)(srow * ld);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int j = lane + 64 * c;
          a[t][c] = A[ro + (unsigned)(j < N ? j : N - 1)];
        }
      }
      TS p[G];
#pragma unroll
      for (int t = 0; t < G; ++t) {
        TS acc = TS(0);
#pragma unroll
        for (int c = 0; c < NC; ++c) acc = fma(a[t][c], xs[c], acc);
        p[t] = acc;
      }
      const TS sum = fold_swap<G>(p, lane);   // row r0 + t in lanes t * (64 / G) ..
      // row r0 + t goes to lane (r0 + t) % 64 of chunk r0 / 64 (a group never
      // straddles two chunks: G divides 64)
      const int t = lane - (r0 & 63);
      const double v = (double)__shfl(sum, (t & (G - 1)) * (64 / G), 64);
      const int rcg = r0 >> 6;
#pragma unroll
      for (int rc = 0; rc < RC; ++rc)
        if (rc == rcg && t >= 0 && t < G) res[rc] = v;
    }
#pragma unroll
    for (int rc = 0; rc < RC; ++rc) {
      const int r = lane + 64 * rc;
      if (r < R) d[gi[rc]] = zero_init ? omega * res[rc] : fma(omega, res[rc], dold[rc]);
    }
  }
}

// ---------------------------------------------------------------------------
// Vanka cell sweep on time-decoupled inverses (CellSplit, last-writer form):
//   d_T <- d_T + omega (I (x) V) Q^-1 (I (x) W) rho_T   on the owned rows.
// One 64-lane wavefront per cell (B * NLS <= 64).  Lane j gathers rho_T[j]
// (local order alpha * B + l) and forms u = (I (x) W) rho_T in the same
// order (the B values of a spatial DoF by shuffles).  Lane j then takes the
// multipliers of stored column j: in block p (first time component f) at
// spatial DoF s, column j multiplies u[s, f] into output f; in the second
// half of a pair block (the imaginary part of the complex inverse) it
// multiplies -u[s, f + 1] into output f and u[s, f] into output f + 1, and
// in the first half u[s, f + 1] into output f + 1 as well: the real form of
// the complex product (the lane's constants come from the level's table,
// made with the store).  Each stored row (one owned spatial DoF) is one
// coalesced read and gives B per-lane products; 16 / BP rows at a time are
// folded by one transpose-reduce (slots of the padding outputs skipped),
// and the lane of DoF (k, i) combines the B outputs of row k with row i of
// V in FP64.  The products and the transpose-reduce are in the precision of
// the store: an FP32 store multiplies its values by the multipliers rounded
// to FP32 and sums in FP32, which halves the exchanges; the error this adds
// is of the order of the rounding of the stored values themselves.  Stores
// as in k_vanka.
// Occupancy the register allocation must leave room for (waves per SIMD):
// the sweep hides its load latency with waves; without spills the FP32 form
// fits 8, the FP64 form 6 (B = 1, 3) or 5 (B = 2).
template <int B, typename TS>
constexpr int dec_waves() {
  return sizeof(TS) == 4 ? 8 : (B == 2 ? 5 : 6);
}

template <int B, int NLS, typename TS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(dec_waves<B, TS>())))
k_vanka_dec(const double* __restrict__ rho,
                                                  double* __restrict__ d,
                                                  const int32_t* __restrict__ csd,
                                                  const int32_t* __restrict__ own_ptr,
                                                  const uint8_t* __restrict__ own_loc,
                                                  const int64_t* __restrict__ inv_off, int ld,
                                                  const TS* __restrict__ store, double omega,
                                                  int zero_init, int n_cells,
                                                  const double* __restrict__ tab,
                                                  const int32_t* __restrict__ code) {
  constexpr int N = B * NLS;
  static_assert(N <= 64 && NLS <= 64, "one wavefront per cell");
  constexpr int BP = B <= 2 ? 2 : 4;       // outputs per stored row, padded to a power of two
  constexpr int GN = 16 / BP;              // stored rows per transpose-reduce
  constexpr unsigned long long LIVE = live_slots(GN, BP, B);
  // stored rows loaded together: an interior cell owns about n_loc / 2
  // spatial DoFs, so one round of loads usually covers the cell (every load
  // in flight at once; each transpose-reduce waits only for its own rows)
  constexpr int GL = (B == 2 ? 2 : 3) * GN;
  const int lane = threadIdx.x & 63;
  const int jl = lane < N ? lane : N - 1;
  const int al = jl / B, cl = jl - al * B;   // spatial DoF and time component of lane j
  // per-lane constants of the level: W[cl][.], V[lane % B][.], the source
  // lanes of u and the multipliers of stored column j = lane
  double wl[B], vl[B];
#pragma unroll
  for (int l = 0; l < B; ++l) {
    wl[l] = tab[l * 64 + lane];
    vl[l] = tab[(B + l) * 64 + lane];
  }
  const int cd = code[lane];
  const int srca = cd & 63, srcb = (cd >> 6) & 63;
  // the multipliers 0, +1 or -1 of the two sources (2 bits each in the code
  // word): kept as constants for B <= 2, decoded per cell for B = 3, where
  // the registers they would hold cost a wavefront per SIMD
  constexpr bool DECODE = B == 3;
  double ca[DECODE ? 1 : B], cb[DECODE ? 1 : B];
#pragma unroll
  for (int o = 0; o < (DECODE ? 1 : B); ++o) {
    const int ea = (cd >> (12 + 2 * o)) & 3, eb = (cd >> (12 + 2 * B + 2 * o)) & 3;
    ca[o] = ea == 1 ? 1.0 : (ea == 3 ? -1.0 : 0.0);
    cb[o] = eb == 1 ? 1.0 : (eb == 3 ? -1.0 : 0.0);
  }
  // byte offset of the lane's column in a stored row, and of one row
  const unsigned jb = (unsigned)(jl * sizeof(TS)), rb = (unsigned)(ld * sizeof(TS));
  // the cell's offsets and its DoF list are fetched one cell ahead (a
  // persistent grid strides over the cells), so that a cell starts with its
  // row loads and its gather instead of a chain of dependent loads
  const int stride = gridDim.x * 4;
  int T = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  int o0n = 0, nxn = 0, sdn = 0;
  int64_t offn = 0;
  if (T < n_cells) {
    o0n = own_ptr[T];
    nxn = own_ptr[T + 1];
    offn = inv_off[T];
    sdn = csd[(int64_t)T * NLS + al];
  }
  for (; T < n_cells; T += stride) {
    const int o0 = o0n, no = nxn - o0n, sdv = sdn;
    const char* A = reinterpret_cast<const char*>(store + offn);
    const int Tn = T + stride;
    if (Tn < n_cells) {
      o0n = own_ptr[Tn];
      nxn = own_ptr[Tn + 1];
      offn = inv_off[Tn];
      sdn = csd[(int64_t)Tn * NLS + al];
    }
    if (no <= 0) continue;
    const int R = no * B;
    const double xv = rho[(int64_t)sdv * B + cl];
    const double x = lane < N ? xv : 0.0;
    double u = 0.0;
#pragma unroll
    for (int l = 0; l < B; ++l) u = fma(wl[l], __shfl(x, al * B + l, 64), u);
    const double ua = __shfl(u, srca, 64), ub = __shfl(u, srcb, 64);
    TS m[B];
#pragma unroll
    for (int o = 0; o < B; ++o) {
      if constexpr (DECODE) {
        const int ea = (cd >> (12 + 2 * o)) & 3, eb = (cd >> (12 + 2 * B + 2 * o)) & 3;
        const double ta = ea == 1 ? ua : (ea == 3 ? -ua : 0.0);
        const double tb = eb == 1 ? ub : (eb == 3 ? -ub : 0.0);
        m[o] = (TS)(ta + tb);
      } else {
        m[o] = (TS)fma(ca[o], ua, cb[o] * ub);
      }
    }
    // the owned DoF of each stored row (lane = owned index; its spatial
    // index from the lanes of its local DoF), the row this lane stores
    // (r = lane = k * B + i), its global index and old value
    const int ok = lane < no ? lane : no - 1;
    const int gs = __shfl(sdv, own_loc[o0 + ok] * B, 64);
    const int rl = lane < R ? lane : R - 1;
    const int kl = rl / B;
    const int64_t gi = (int64_t)__shfl(gs, kl, 64) * B + (rl - kl * B);
    const double dold = zero_init ? 0.0 : d[gi];
    double res = 0.0;
    for (int k0 = 0; k0 < no; k0 += GL) {
      TS a[GL];
#pragma unroll
      for (int t = 0; t < GL; ++t) {
        const unsigned row = (unsigned)min(k0 + t, no - 1);
        a[t] = *reinterpret_cast<const TS*>(A + (row * rb + jb));
      }
#pragma unroll
      for (int h = 0; h < GL / GN; ++h) {
        TS pp[16];
#pragma unroll
        for (int t = 0; t < GN; ++t)
#pragma unroll
          for (int o = 0; o < BP; ++o) pp[t * BP + o] = o < B ? a[h * GN + t] * m[o] : TS(0);
        // value t * BP + o in lanes 4 (t * BP + o) .. + 3
        const TS sum = fold_swap<16, LIVE>(pp, lane);
        const int kb = k0 + h * GN;
        const int kk = kl - kb;                  // this lane's row within the group
        const int kc = kk < 0 ? 0 : (kk >= GN ? GN - 1 : kk);
        double val = 0.0;
#pragma unroll
        for (int o = 0; o < B; ++o)
          val = fma(vl[o], (double)__shfl(sum, 4 * (kc * BP + o), 64), val);
        if (kk >= 0 && kk < GN) res = val;
      }
    }
    if (lane < R) d[gi] = zero_init ? omega * res : fma(omega, res, dold);
  }
}

// ---------------------------------------------------------------------------
// Vanka cell sweep on the complex time-decoupled store of a dG(1) level with
// one complex pair (built by k_inverse_cx): the stored row of owned spatial
// DoF a is Y_a. = (X^-1)_a. as [Re Y_a0 .. Re Y_a,n-1, Im Y_a0 .. Im Y_a,n-1],
// and with u = (I (x) W) rho_T (u_0 + i u_1 per spatial DoF c)
//   y_a = sum_c Y_ac (u_0c + i u_1c),  c_(a, i) = V_i0 Re y_a + V_i1 Im y_a:
// the same J_T^-1 rho_T = (I (x) V) Q^-1 (I (x) W) rho_T as the two plain rows
// of a, from half the stored values.  One wavefront per cell.  A stored row
// is read as one flat run of 2 NLS values, NF = 2 NLS / 64 (rounded up)
// coalesced loads: value v = 64 k + lane is Re Y_ac (v < NLS, c = v) or
// Im Y_ac (c = v - NLS), and the lane holds, per load, the two multipliers
// that put it into Re y_a and Im y_a (u_0c and u_1c for a real part, -u_1c
// and u_0c for an imaginary one), formed once per cell from its own
// 16-byte load of the time-inner pair rho_(c, 0..1).  G rows at a time give
// 2G sums (real and imaginary parts) folded by one transpose-reduce.  Output
// r = 2 os + i of the os-th owned DoF lands in lane r % 64, which fetched the
// DoF's old value at the start; stores as in k_vanka.  The complex products
// and the transpose-reduce are in the precision of the store, the
// recombination with V and the update in FP64.
template <int NLS, typename TS, int G>
__global__ void __launch_bounds__(256) k_vanka_cx(const double* __restrict__ rho,
                                                 double* __restrict__ d,
                                                 const int32_t* __restrict__ csd,
                                                 const int32_t* __restrict__ own_ptr,
                                                 const uint8_t* __restrict__ own_loc,
                                                 const int64_t* __restrict__ inv_off, int ld,
                                                 const TS* __restrict__ store, double omega,
                                                 int zero_init, int n_cells, CellSplit sp) {
  constexpr int B = 2;
  constexpr int NF = (2 * NLS + 63) / 64;    // flat 64-lane loads of a stored row
  constexpr int NOC = (NLS + 63) / 64;       // 64-lane chunks of the owned DoFs
  constexpr int RC = (B * NLS + 63) / 64;    // 64-lane chunks of the outputs
  const int lane = threadIdx.x & 63;
  const double w00 = sp.W[0], w01 = sp.W[1], w10 = sp.W[2], w11 = sp.W[3];
  const double v00 = sp.V[0], v01 = sp.V[1], v10 = sp.V[2], v11 = sp.V[3];
  // byte offsets of the lane's values in a stored row
  unsigned vb[NF];
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    const int v = 64 * k + lane;
    vb[k] = (unsigned)((v < 2 * NLS ? v : 2 * NLS - 1) * sizeof(TS));
  }
  const unsigned rb = (unsigned)(ld * sizeof(TS));
  const int T0 = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  for (int T = T0; T < n_cells; T += gridDim.x * 4) {
    const int32_t* sd = csd + (int64_t)T * NLS;
    const int o0 = own_ptr[T];
    const int no = own_ptr[T + 1] - o0;
    if (no <= 0) continue;
    const int R = no * B;
    const char* A = reinterpret_cast<const char*>(store + inv_off[T]);
    // the multipliers of the lane's values: (into Re y, into Im y)
    TS mre[NF], mim[NF];
#pragma unroll
    for (int k = 0; k < NF; ++k) {
      const int v = 64 * k + lane;
      const bool ok = v < 2 * NLS;
      const bool im = v >= NLS;
      const int c = ok ? (im ? v - NLS : v) : 0;
      const double2 rr = *reinterpret_cast<const double2*>(&rho[(int64_t)sd[c] * B]);
      const double u0 = fma(w00, rr.x, w01 * rr.y), u1 = fma(w10, rr.x, w11 * rr.y);
      mre[k] = (TS)(ok ? (im ? -u1 : u0) : 0.0);
      mim[k] = (TS)(ok ? (im ? u0 : u1) : 0.0);
    }
    int gs[NOC];
#pragma unroll
    for (int c = 0; c < NOC; ++c) {
      const int k = lane + 64 * c;
      gs[c] = sd[own_loc[o0 + (k < no ? k : no - 1)]];
    }
    int64_t gi[RC];
    double dold[RC], res[RC];
#pragma unroll
    for (int rc = 0; rc < RC; ++rc) {
      const int r = lane + 64 * rc;
      const int rcl = r < R ? r : R - 1;
      const int os = rcl / B;
      int g = __shfl(gs[0], os & 63, 64);
      if constexpr (NOC > 1) {
        const int g1 = __shfl(gs[NOC - 1], os & 63, 64);
        g = os < 64 ? g : g1;
      }
      gi[rc] = (int64_t)g * B + (rcl - os * B);
      dold[rc] = zero_init ? 0.0 : d[gi[rc]];
      res[rc] = 0.0;
    }
    for (int k0 = 0; k0 < no; k0 += G) {
      TS a[G][NF];
#pragma unroll
      for (int t = 0; t < G; ++t) {
        const unsigned ro = (unsigned)min(k0 + t, no - 1) * rb;
#pragma unroll
        for (int k = 0; k < NF; ++k) a[t][k] = *reinterpret_cast<const TS*>(A + (ro + vb[k]));
      }
      TS p[2 * G];
#pragma unroll
      for (int t = 0; t < G; ++t) {
        TS re = TS(0), im = TS(0);
#pragma unroll
        for (int k = 0; k < NF; ++k) {
          re = fma(a[t][k], mre[k], re);
          im = fma(a[t][k], mim[k], im);
        }
        p[2 * t] = re;
        p[2 * t + 1] = im;
      }
      const TS sum = fold_swap<2 * G>(p, lane);   // value e in lanes e (64 / 2G) ..
#pragma unroll
      for (int rc = 0; rc < RC; ++rc) {
        const int r = lane + 64 * rc;
        const int t = (r >> 1) - k0;
        const int tc = t < 0 ? 0 : (t >= G ? G - 1 : t);
        const double re = (double)__shfl(sum, (64 / (2 * G)) * (2 * tc), 64);
        const double im = (double)__shfl(sum, (64 / (2 * G)) * (2 * tc + 1), 64);
        const double val = (r & 1) ? fma(v10, re, v11 * im) : fma(v00, re, v01 * im);
        if (t >= 0 && t < G) res[rc] = val;
      }
    }
#pragma unroll
    for (int rc = 0; rc < RC; ++rc) {
      const int r = lane + 64 * rc;
      if (r < R) d[gi[rc]] = zero_init ? omega * res[rc] : fma(omega, res[rc], dold[rc]);
    }
  }
}

// rows per transpose-reduce of the complex sweep: 8 in FP64 (115 registers,
// four wavefronts per SIMD), 16 in FP32 (twice the rows in flight in about
// the same registers)
template <typename TS>
constexpr int cx_group() { return sizeof(TS) == 4 ? 16 : 8; }

template <int B, int NLS>
static hipError_t vanka_bn(hipStream_t s, const DevLevel& L, const double* rho, double* d,
                           double omega, int zero_init, int fp32, int full) {
  unsigned grid = (unsigned)((L.n_cells + 3) / 4);
  if (L.sweep_wgs > 0 && (unsigned)L.sweep_wgs < grid) grid = (unsigned)L.sweep_wgs;
  if constexpr (B * NLS <= 64) {
    if (L.dec) {
      if (full || L.split.b != B || !L.dec_tab || !L.dec_code) return hipErrorInvalidValue;
      if (fp32)
        launch(k_vanka_dec<B, NLS, float>, dim3(grid), dim3(256), 0, s, rho, d, L.cell_sdofs,
               L.own_ptr, L.own_loc, L.inv_off, L.inv_ld, (const float*)L.inv_store, omega,
               zero_init, L.n_cells, (const double*)L.dec_tab, (const int32_t*)L.dec_code);
      else
        launch(k_vanka_dec<B, NLS, double>, dim3(grid), dim3(256), 0, s, rho, d, L.cell_sdofs,
               L.own_ptr, L.own_loc, L.inv_off, L.inv_ld, (const double*)L.inv_store, omega,
               zero_init, L.n_cells, (const double*)L.dec_tab, (const int32_t*)L.dec_code);
      return hipGetLastError();
    }
  }
  if constexpr (B == 2 && NLS == 85) {
    if (L.dec && L.cx) {
      if (full) return hipErrorInvalidValue;
      if (L.comp) return launch_vanka_comp(s, L, rho, d, omega, zero_init, fp32, grid);
      if (fp32)
        launch(k_vanka_cx<NLS, float, cx_group<float>()>, dim3(grid), dim3(256), 0, s, rho, d,
               L.cell_sdofs, L.own_ptr, L.own_loc, L.inv_off, L.inv_ld,
               (const float*)L.inv_store, omega, zero_init, L.n_cells, L.split);
      else
        launch(k_vanka_cx<NLS, double, cx_group<double>()>, dim3(grid), dim3(256), 0, s, rho, d,
               L.cell_sdofs, L.own_ptr, L.own_loc, L.inv_off, L.inv_ld,
               (const double*)L.inv_store, omega, zero_init, L.n_cells, L.split);
      return hipGetLastError();
    }
  }
  if (L.dec) return hipErrorInvalidValue;
#define STV_VANKA(TS, F)                                                                     \
  launch(k_vanka<B, NLS, TS, F>, dim3(grid), dim3(256), 0, s, rho, d, L.cell_sdofs, L.own_ptr, L.own_loc,  \
                                              L.inv_off, L.inv_ld, (const TS*)L.inv_store, \
                                              omega, zero_init, L.n_cells)
  if (fp32) {
    if (full) STV_VANKA(float, true);
    else STV_VANKA(float, false);
  } else {
    if (full) STV_VANKA(double, true);
    else STV_VANKA(double, false);
  }
#undef STV_VANKA
  return hipGetLastError();
}

template <int B>
static hipError_t vanka_b(hipStream_t s, const DevLevel& L, const double* rho, double* d,
                          double omega, int zero_init, int fp32, int full) {
  if (L.n_ls == 21) return vanka_bn<B, 21>(s, L, rho, d, omega, zero_init, fp32, full);
  if (L.n_ls == 85) return vanka_bn<B, 85>(s, L, rho, d, omega, zero_init, fp32, full);
  return hipErrorInvalidValue;
}

hipError_t launch_vanka_cells(hipStream_t s, int b, const DevLevel& L, const double* rho,
                              double* d, double omega, int zero_init, int fp32, int full) {
  switch (b) {
    case 1: return vanka_b<1>(s, L, rho, d, omega, zero_init, fp32, full);
    case 2: return vanka_b<2>(s, L, rho, d, omega, zero_init, fp32, full);
    case 3: return vanka_b<3>(s, L, rho, d, omega, zero_init, fp32, full);
    case 4: return vanka_b<4>(s, L, rho, d, omega, zero_init, fp32, full);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Vanka sweep of the transposed operator J^T.  Its local inverse is
// (J_T^T)^-1 = (J_T^-1)^T, the stored full inverse read transposed: with the
// residual rho_T of J^T in lane j = lane + 64c, the correction
// c_o = sum_j (J_T^-1)[j][o] rho_j of local DoF o = lane + 64c accumulates in
// lane o, stored row j after row j (each row one coalesced read, rho_j
// broadcast by readlane), 8 rows per round with all their loads in flight.
// The owner rule and the update are those of the forward sweep: lane o
// learns whether the cell owns its DoF from the cell's owned list, fetches
// the DoF's old value at the start and stores once.  Needs every stored row.
template <int B, int NLS, typename TS>
__global__ void __launch_bounds__(256) k_vanka_t(const double* __restrict__ rho,
                                                double* __restrict__ d,
                                                const int32_t* __restrict__ csd,
                                                const int32_t* __restrict__ own_ptr,
                                                const uint8_t* __restrict__ own_loc,
                                                const int64_t* __restrict__ inv_off, int ld,
                                                const TS* __restrict__ store, double omega,
                                                int zero_init, int n_cells) {
  constexpr int N = B * NLS;
  constexpr int NC = (N + 63) / 64;
  constexpr int NOC = (NLS + 63) / 64;
  constexpr int U = 8;
  const int lane = threadIdx.x & 63;
  const int T0 = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  for (int T = T0; T < n_cells; T += gridDim.x * 4) {
    const int32_t* sd = csd + (int64_t)T * NLS;
    const int o0 = own_ptr[T];
    const int no = own_ptr[T + 1] - o0;
    if (no <= 0) continue;
    const TS* A = store + inv_off[T];
    double x[NC], acc[NC], dold[NC];
    int64_t gi[NC];
    bool own[NC];
    int ol[NOC];
#pragma unroll
    for (int c = 0; c < NOC; ++c) {
      const int k = lane + 64 * c;
      ol[c] = own_loc[o0 + (k < no ? k : no - 1)];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = lane + 64 * c;
      const int jc = j < N ? j : N - 1;
      const int be = jc / B;
      const int64_t g = (int64_t)sd[be] * B + (jc - be * B);
      const double v = rho[g];
      x[c] = j < N ? v : 0.0;
      acc[c] = 0.0;
      gi[c] = g;
      own[c] = false;
    }
    // ownership of this lane's DoFs: compare their spatial index with the
    // cell's owned list (broadcast entry by entry)
    for (int k = 0; k < no; ++k) {
      int a = __builtin_amdgcn_readlane(ol[0], k & 63);
      if constexpr (NOC > 1) {
        const int a1 = __builtin_amdgcn_readlane(ol[NOC - 1], k & 63);
        a = k < 64 ? a : a1;
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int o = lane + 64 * c;
        own[c] = own[c] || (o < N && o / B == a);
      }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double v = d[gi[c]];
      dold[c] = zero_init ? 0.0 : v;
    }
#pragma unroll 1
    for (int j0 = 0; j0 < N; j0 += U) {
      TS a[U][NC];
      double rj[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = j0 + u;
        const int jr = j < N ? j : N - 1;
        const unsigned ro = (unsigned)(jr * ld);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int o = lane + 64 * c;
          a[u][c] = A[ro + (unsigned)(o < N ? o : N - 1)];
        }
        // rho_j from its lane (chunk j / 64, uniform)
        double r = readlane_f64(x[0], jr & 63);
#pragma unroll
        for (int c = 1; c < NC; ++c) {
          const double rc = readlane_f64(x[c], jr & 63);
          r = (jr >> 6) == c ? rc : r;
        }
        rj[u] = j < N ? r : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = fma((double)a[u][c], rj[u], acc[c]);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (own[c]) d[gi[c]] = zero_init ? omega * acc[c] : fma(omega, acc[c], dold[c]);
  }
}

template <int B, int NLS>
static hipError_t vanka_t_bn(hipStream_t s, const DevLevel& L, const double* rho, double* d,
                             double omega, int zero_init, int fp32) {
  unsigned grid = (unsigned)((L.n_cells + 3) / 4);
  if (L.sweep_wgs > 0 && (unsigned)L.sweep_wgs < grid) grid = (unsigned)L.sweep_wgs;
  if (fp32)
    launch(k_vanka_t<B, NLS, float>, dim3(grid), dim3(256), 0, s, rho, d, L.cell_sdofs, L.own_ptr, L.own_loc,
                                                  L.inv_off, L.inv_ld, (const float*)L.inv_store,
                                                  omega, zero_init, L.n_cells);
  else
    launch(k_vanka_t<B, NLS, double>, dim3(grid), dim3(256), 0, s, rho, d, L.cell_sdofs, L.own_ptr, L.own_loc,
                                                   L.inv_off, L.inv_ld,
                                                   (const double*)L.inv_store, omega, zero_init,
                                                   L.n_cells);
  return hipGetLastError();
}

template <int B>
static hipError_t vanka_t_b(hipStream_t s, const DevLevel& L, const double* rho, double* d,
                            double omega, int zero_init, int fp32) {
  if (L.n_ls == 21) return vanka_t_bn<B, 21>(s, L, rho, d, omega, zero_init, fp32);
  if (L.n_ls == 85) return vanka_t_bn<B, 85>(s, L, rho, d, omega, zero_init, fp32);
  return hipErrorInvalidValue;
}

hipError_t launch_vanka_cells_t(hipStream_t s, int b, const DevLevel& L, const double* rho,
                                double* d, double omega, int zero_init, int fp32) {
  switch (b) {
    case 1: return vanka_t_b<1>(s, L, rho, d, omega, zero_init, fp32);
    case 2: return vanka_t_b<2>(s, L, rho, d, omega, zero_init, fp32);
    case 3: return vanka_t_b<3>(s, L, rho, d, omega, zero_init, fp32);
    case 4: return vanka_t_b<4>(s, L, rho, d, omega, zero_init, fp32);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Cellwise bilinear forms of two level vectors.  out[T] = sum_l tw[l]
// sum_{alpha, beta} lam[alpha, l] K_T[alpha][beta] x[beta, l] with
// K_T = sum_e kw[e] Kref[kidx[e]] (e in [kptr[T], kptr[T+1]); n_ls x n_ls
// spatial reference matrices): one wavefront per cell, lane j = alpha*B + l
// forms (K_T x)_j with x broadcast from its lane, then a wavefront sum.
// With fidx (per cell: the row k of f that belongs to it, or -1) the cell's
// right-hand-side term is added in the same pass:
//   out[T] = sc * (the form above) + sf * sum_j lam[T's DoF j] f[k][j],
// f in the cell-local order alpha*B + l (the gradient of an outflow loss
// with respect to cell viscosities and an inflow amplitude).
template <int B, int NLS>
__global__ void __launch_bounds__(256) k_cell_contract(
    const double* __restrict__ lam, const double* __restrict__ x,
    const int32_t* __restrict__ csd, int n_cells, const double* __restrict__ Kref,
    const int32_t* __restrict__ kptr, const int32_t* __restrict__ kidx,
    const double* __restrict__ kw, const double* __restrict__ tw, double sc,
    const int32_t* __restrict__ fidx, const double* __restrict__ f, double sf,
    double* __restrict__ out) {
  constexpr int N = B * NLS;
  constexpr int NC = (N + 63) / 64;
  const int lane = threadIdx.x & 63;
  const int T = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (T >= n_cells) return;  // uniform per wavefront
  const int32_t* sd = csd + (int64_t)T * NLS;
  double xv[NC], lv[NC], y[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int j = lane + 64 * c;
    xv[c] = lv[c] = y[c] = 0.0;
    if (j < N) {
      const int be = j / B;
      const int64_t g = (int64_t)sd[be] * B + (j - be * B);
      xv[c] = x[g];
      lv[c] = lam[g];
    }
  }
  for (int e = kptr[T]; e < kptr[T + 1]; ++e) {
    const double* K = Kref + (int64_t)kidx[e] * NLS * NLS;
    const double w = kw[e];
#pragma unroll
    for (int cj = 0; cj < NC; ++cj) {
      const int jn = (N - 64 * cj) < 64 ? (N - 64 * cj) : 64;
      for (int jl = 0; jl < jn; ++jl) {
        const int j = 64 * cj + jl;
        const int beta = j / B, lj = j - beta * B;
        const double xj = w * __shfl(xv[cj], jl, 64);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int o = lane + 64 * c;
          if (o < N && (o - (o / B) * B) == lj) y[c] = fma(K[(o / B) * NLS + beta], xj, y[c]);
        }
      }
    }
  }
  double sacc = 0.0;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int o = lane + 64 * c;
    if (o < N) sacc = fma(tw[o - (o / B) * B] * lv[c], y[c], sacc);
  }
  sacc = wave_sum(sacc);
  double facc = 0.0;
  const int fk = fidx ? fidx[T] : -1;
  if (fk >= 0) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int o = lane + 64 * c;
      if (o < N) facc = fma(lv[c], f[(int64_t)fk * N + o], facc);
    }
    facc = wave_sum(facc);
  }
  if (lane == 0) out[T] = fk >= 0 ? fma(sc, sacc, sf * facc) : sc * sacc;
}

// out[k] = sum_j lam[cell k's DoF j] f[k*N + j] (f in the cell-local order
// alpha*B + l) for the listed cells.
template <int B, int NLS>
__global__ void __launch_bounds__(256) k_cell_dot(const double* __restrict__ lam,
                                                  const int32_t* __restrict__ csd,
                                                  const int32_t* __restrict__ cells, int n,
                                                  const double* __restrict__ f,
                                                  double* __restrict__ out) {
  constexpr int N = B * NLS;
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (k >= n) return;
  const int32_t* sd = csd + (int64_t)cells[k] * NLS;
  double acc = 0.0;
  for (int j = lane; j < N; j += 64) {
    const int be = j / B;
    acc = fma(lam[(int64_t)sd[be] * B + (j - be * B)], f[(int64_t)k * N + j], acc);
  }
  acc = wave_sum(acc);
  if (lane == 0) out[k] = acc;
}

hipError_t launch_cell_contract(hipStream_t s, int b, const DevLevel& L, const double* lam,
                                const double* x, const double* Kref, const int32_t* kptr,
                                const int32_t* kidx, const double* kw, const double* tw,
                                double sc, const int32_t* fidx, const double* f, double sf,
                                double* out) {
  const unsigned grid = (unsigned)((L.n_cells + 3) / 4);
#define STV_CC(BB, NN)                                                                    \
  k_cell_contract<BB, NN><<<grid, 256, 0, s>>>(lam, x, L.cell_sdofs, L.n_cells, Kref, kptr, \
                                               kidx, kw, tw, sc, fidx, f, sf, out)
  if (L.n_ls == 21) {
    switch (b) { case 1: STV_CC(1, 21); break; case 2: STV_CC(2, 21); break;
                 case 3: STV_CC(3, 21); break; case 4: STV_CC(4, 21); break;
                 default: return hipErrorInvalidValue; }
  } else if (L.n_ls == 85) {
    switch (b) { case 1: STV_CC(1, 85); break; case 2: STV_CC(2, 85); break;
                 case 3: STV_CC(3, 85); break; case 4: STV_CC(4, 85); break;
                 default: return hipErrorInvalidValue; }
  } else {
    return hipErrorInvalidValue;
  }
#undef STV_CC
  return hipGetLastError();
}

hipError_t launch_cell_dot(hipStream_t s, int b, const DevLevel& L, const double* lam,
                           const int32_t* cells, int n, const double* f, double* out) {
  if (n <= 0) return hipSuccess;
  const unsigned grid = (unsigned)((n + 3) / 4);
#define STV_CD(BB, NN) k_cell_dot<BB, NN><<<grid, 256, 0, s>>>(lam, L.cell_sdofs, cells, n, f, out)
  if (L.n_ls == 21) {
    switch (b) { case 1: STV_CD(1, 21); break; case 2: STV_CD(2, 21); break;
                 case 3: STV_CD(3, 21); break; case 4: STV_CD(4, 21); break;
                 default: return hipErrorInvalidValue; }
  } else if (L.n_ls == 85) {
    switch (b) { case 1: STV_CD(1, 85); break; case 2: STV_CD(2, 85); break;
                 case 3: STV_CD(3, 85); break; case 4: STV_CD(4, 85); break;
                 default: return hipErrorInvalidValue; }
  } else {
    return hipErrorInvalidValue;
  }
#undef STV_CD
  return hipGetLastError();
}

// y[dof[i]] += sum_{e = ptr[i]}^{ptr[i+1]-1} coef[ck[e]] * f[fi[e]]: cellwise
// terms added into a vector by gathering, one thread per touched DoF, the
// terms of a DoF in the order of its list (deterministic, no atomics).
__global__ void k_cell_scatter(const int64_t* __restrict__ dof, const int32_t* __restrict__ ptr,
                               const int32_t* __restrict__ ck, const int64_t* __restrict__ fi,
                               const double* __restrict__ coef, const double* __restrict__ f,
                               int n_dof, double* __restrict__ y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_dof) return;
  double acc = y[dof[i]];
  for (int e = ptr[i]; e < ptr[i + 1]; ++e) acc = fma(coef[ck[e]], f[fi[e]], acc);
  y[dof[i]] = acc;
}

hipError_t launch_cell_scatter(hipStream_t s, const int64_t* dof, const int32_t* ptr,
                               const int32_t* ck, const int64_t* fi, const double* coef,
                               const double* f, int n_dof, double* y) {
  if (n_dof <= 0) return hipSuccess;
  k_cell_scatter<<<(unsigned)((n_dof + 255) / 256), 256, 0, s>>>(dof, ptr, ck, fi, coef, f,
                                                                 n_dof, y);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Averaged / additive forms: every cell writes its full damped correction
// omega J_T^-1 rho_T to corr[T*n_loc + (alpha*B + l)] (needs every stored
// row); a second kernel sums, per DoF and in cell order, the corrections of
// the cells containing it.
template <int B, typename TS>
__global__ void __launch_bounds__(64) k_vanka_corr(const double* __restrict__ rho,
                                                  double* __restrict__ corr,
                                                  const int32_t* __restrict__ csd, int n_ls,
                                                  const int64_t* __restrict__ inv_off, int ld,
                                                  const TS* __restrict__ store, double omega) {
  extern __shared__ double sm[];
  const int n_loc = n_ls * B;
  const int T = blockIdx.x;
  const int lane = threadIdx.x;
  const int32_t* sd = csd + (int64_t)T * n_ls;
  for (int e = lane; e < n_loc; e += 64) {
    const int be = e / B;
    sm[e] = rho[(int64_t)sd[be] * B + (e - be * B)];
  }
  __syncthreads();
  const TS* A = store + inv_off[T];
  for (int i = lane; i < n_loc; i += 64) {
    double acc = 0.0;
    for (int j = 0; j < n_loc; ++j) acc = fma((double)A[(int64_t)i * ld + j], sm[j], acc);
    corr[(int64_t)T * n_loc + i] = omega * acc;
  }
}

template <int B>
__global__ void k_vanka_combine(const double* __restrict__ corr, double* __restrict__ d,
                                const int32_t* __restrict__ inc_ptr,
                                const int32_t* __restrict__ inc_cell,
                                const uint8_t* __restrict__ inc_loc, int n_s, int n_loc, int pou) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)n_s * B) return;
  const int s = (int)(idx / B);
  const int l = (int)(idx - (int64_t)s * B);
  const int e0 = inc_ptr[s], e1 = inc_ptr[s + 1];
  double acc = 0.0;
  for (int e = e0; e < e1; ++e) acc += corr[(int64_t)inc_cell[e] * n_loc + inc_loc[e] * B + l];
  if (pou && e1 > e0) acc /= (double)(e1 - e0);   // rows of directly solved members have no cell
  d[idx] += acc;
}

hipError_t launch_vanka_cells_corr(hipStream_t s, int b, const DevLevel& L, const double* rho,
                                   double omega, int fp32) {
  const size_t shm = sizeof(double) * (size_t)(L.n_ls * b);
#define STV_CORR(BB)                                                                        \
  if (fp32)                                                                                 \
    k_vanka_corr<BB, float><<<L.n_cells, 64, shm, s>>>(rho, L.corr, L.cell_sdofs, L.n_ls,   \
                                                       L.inv_off, L.inv_ld,                 \
                                                       (const float*)L.inv_store, omega);   \
  else                                                                                      \
    k_vanka_corr<BB, double><<<L.n_cells, 64, shm, s>>>(rho, L.corr, L.cell_sdofs, L.n_ls,  \
                                                        L.inv_off, L.inv_ld,                \
                                                        (const double*)L.inv_store, omega);
  switch (b) {
    case 1: STV_CORR(1) break;
    case 2: STV_CORR(2) break;
    case 3: STV_CORR(3) break;
    case 4: STV_CORR(4) break;
    default: return hipErrorInvalidValue;
  }
#undef STV_CORR
  return hipGetLastError();
}

hipError_t launch_vanka_combine(hipStream_t s, int b, const DevLevel& L, double* d, int pou) {
  const int64_t n = (int64_t)L.n_s * b;
  dim3 grid((unsigned)((n + 255) / 256)), block(256);
  const int n_loc = L.n_ls * b;
  switch (b) {
    case 1: k_vanka_combine<1><<<grid, block, 0, s>>>(L.corr, d, L.inc_ptr, L.inc_cell, L.inc_loc, L.n_s, n_loc, pou); break;
    case 2: k_vanka_combine<2><<<grid, block, 0, s>>>(L.corr, d, L.inc_ptr, L.inc_cell, L.inc_loc, L.n_s, n_loc, pou); break;
    case 3: k_vanka_combine<3><<<grid, block, 0, s>>>(L.corr, d, L.inc_ptr, L.inc_cell, L.inc_loc, L.n_s, n_loc, pou); break;
    case 4: k_vanka_combine<4><<<grid, block, 0, s>>>(L.corr, d, L.inc_ptr, L.inc_cell, L.inc_loc, L.n_s, n_loc, pou); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

__global__ void k_fill(double* __restrict__ x, int64_t n, double v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = v;
}

__global__ void k_copy(const double* __restrict__ x, double* __restrict__ y, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = x[i];
}

hipError_t launch_fill(hipStream_t s, double* x, int64_t n, double v) {
  if (n <= 0) return hipSuccess;
  k_fill<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(x, n, v);
  return hipGetLastError();
}

hipError_t launch_copy(hipStream_t s, const double* x, double* y, int64_t n) {
  if (n <= 0) return hipSuccess;
  k_copy<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(x, y, n);
  return hipGetLastError();
}

}  // namespace stv
