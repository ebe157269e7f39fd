// Cell problems whose velocity components do not couple (levels with spatial
// factors, time-decoupled): the cell matrix of one time block is
//   [ V_1           B_1 ]      V_c (n x n, n = 3^D) the block of component c,
//   [     ..        ..  ]      B_c (n x m), C_c (m x n), m = D + 1 pressure
//   [          V_D  B_D ]      modes, no pressure-pressure block; V_c the same
//   [ C_1 ..   C_D   0  ]      for every c in cells away from the walls.
// Its inverse comes from the V_c^-1 and the m x m Schur complement
// S = -sum_c C_c V_c^-1 B_c:  with P = S^-1 [-C V^-1 | I] (the pressure rows),
// row (c, i) is [V_c^-1_i. | 0] + G_c,i P,  G_c = -V_c^-1 B_c.  That is D or
// one elimination of order n instead of one of order D n + m (3d: 27 against
// 85), and 31 instead of 85 values per velocity row in the store.
// Block elimination takes its pivots inside V_c first, then in S; a cell with a
// pivot below kPivotTol of its block's largest entry is flagged, and the build
// then eliminates the whole cell matrices of the level instead.  So is a cell
// where V^-1 is nearly singular although the cell's matrix is not: V^-1 and G P
// then cancel.  With
//   g = max_c max |V_c^-1| / max_i |(V_c^-1 + G_c P)_i . s|  (signs s), and
//   kappa = m max(|S|, |C V^-1 B|) max |S^-1|,
// the error of the velocity rows is below 2^-53 g kappa apart from V^-1's own
// (cell matrices of channel operators with one to four velocity directions
// scaled down to 1e-1 .. 1e-7: errors of 1e-5 to 0.5 of that), so g kappa is held to
// kCancelTol.  Channel operators, nu 1e-6 to 1e-1, tau 1e-4 to 10, have 9 to
// 470; errors at the limit are 2e-14 of the largest entry and less.  The check
// costs 3d 6,912 cells 0.72 -> 0.78 ms, 2d nothing measurable.
#include "stv_internal.h"
#include "wave.h"

#include <algorithm>

namespace stv {

static constexpr double kPivotTol = 1e-7;
static constexpr double kCancelTol = 4096.0;
static constexpr unsigned kSigns = 0x59a7c36;   // s of the check, bit j: the sign of node j

typedef double stv_d4 __attribute__((ext_vector_type(4)));

// Per cell: bit 0 = V_c equal for every component (exactly), bit 1 = the zero
// blocks are zero.  One wavefront per cell.
template <int D>
__global__ void __launch_bounds__(256) k_comp_flags(const int32_t* __restrict__ posmap,
                                                    const double2* __restrict__ ma,
                                                    uint8_t* __restrict__ flags, int n_cells) {
  constexpr int NV = D == 2 ? 9 : 27, NM = D + 1, NLS = D * NV + NM;
  const int lane = threadIdx.x & 63;
  const int T = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (T >= n_cells) return;
  const int32_t* pos = posmap + (int64_t)T * (NLS * NLS);
  bool same = true, ok = true;
  for (int e = lane; e < NLS * NLS; e += 64) {
    const int a = e / NLS, b = e - a * NLS;
    const int ca = a / NV, cb = b / NV;   // D: pressure
    const int32_t q = pos[e];
    const double2 f = q >= 0 ? ma[q] : make_double2(0.0, 0.0);
    if (ca != cb ? (ca < D && cb < D) : ca == D) {
      ok = ok && f.x == 0.0 && f.y == 0.0;
    } else if (ca == cb && ca > 0) {
      const int32_t q0 = pos[(a - ca * NV) * NLS + b - ca * NV];
      const double2 f0 = q0 >= 0 ? ma[q0] : make_double2(0.0, 0.0);
      same = same && f.x == f0.x && f.y == f0.y;
    }
  }
  same = __all(same);
  ok = __all(ok);
  if (lane == 0) flags[T] = (uint8_t)((same ? 1 : 0) | (ok ? 2 : 0));
}

hipError_t launch_comp_flags(hipStream_t s, const DevLevel& L, uint8_t* flags) {
  const dim3 grid((L.n_cells + 3) / 4), block(256);
  if (L.n_ls == 21)
    k_comp_flags<2><<<grid, block, 0, s>>>(L.posmap, (const double2*)L.kron_ma, flags, L.n_cells);
  else
    k_comp_flags<3><<<grid, block, 0, s>>>(L.posmap, (const double2*)L.kron_ma, flags, L.n_cells);
  return hipGetLastError();
}

// In-place Gauss-Jordan on one row of NC entries per lane (lanes >= NC / the
// rows hold zeros): pivots from columns 0 .. NV - 1 and rows 0 .. NV - 1, one
// step per column, the other rows and columns only updated.  Each step reads
// column 0 and writes entry j to j - 1, so the loop is rolled (one register
// name per entry, 300 instructions) and the eliminated column ends last;
// after NV steps the array is [columns NV .. NC - 1 | columns 0 .. NV - 1].
// A pivot row is left as it is (its other lanes' multiplier is formed with
// the pivot's reciprocal) and scaled by that reciprocal once at the end.
// var = the column this lane's row was the pivot of (-1: none), piv = in lane
// q the pivot row of column q.  Entry (row, q) then belongs to row var and
// column piv[q] of the inverse.
template <int NV, int NC, bool CX>
__device__ __forceinline__ void gj_rows(double (&re)[NC], double (&im)[CX ? NC : 1], int lane,
                                        double tol, int& var, int& piv, bool& sing) {
  double sr = 1.0, si = 0.0;
  var = -1;
  piv = 0;
#pragma unroll 1
  for (int p = 0; p < NV; ++p) {
    const bool cand = lane < NV && var < 0;
    double mag = fabs(re[0]);
    if constexpr (CX) mag += fabs(im[0]);
    const double b = (cand && mag == mag) ? mag : -1.0;
    const double mx = wave_max_f64(b);
    const uint64_t at = __builtin_amdgcn_ballot_w64(mx > 0.0 ? b == mx : cand);
    const int r = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(at));
    if (!(mx > tol)) sing = true;
    const double xr = readlane_f64(re[0], r);
    double xi = 0.0;
    if constexpr (CX) xi = readlane_f64(im[0], r);
    const double den = CX ? fma(xr, xr, xi * xi) : xr;
    const bool good = CX ? (den > 0.0 && den < INFINITY) : (fabs(den) > 0.0 && fabs(den) < INFINITY);
    if (!good) sing = true;
    const double id = good ? recip_f64(den) : 0.0;
    const double ir = CX ? xr * id : id, ii = CX ? -xi * id : 0.0;
    const bool me = lane == r;
    double gr, gi = 0.0;
    if constexpr (CX) {
      gr = me ? 0.0 : fma(re[0], ir, -im[0] * ii);
      gi = me ? 0.0 : fma(re[0], ii, im[0] * ir);
    } else {
      gr = me ? 0.0 : re[0] * ir;
    }
#pragma unroll
    for (int j = 1; j < NC; ++j) {
      const double pr = readlane_f64(re[j], r);
      if constexpr (CX) {
        const double pi = readlane_f64(im[j], r);
        re[j - 1] = fma(gi, pi, fma(-gr, pr, re[j]));
        im[j - 1] = fma(-gi, pr, fma(-gr, pi, im[j]));
      } else {
        re[j - 1] = fma(-gr, pr, re[j]);
      }
    }
    re[NC - 1] = me ? 1.0 : -gr;
    if constexpr (CX) im[NC - 1] = -gi;
    if (me) {
      var = p;
      sr = ir;
      si = ii;
    }
    if (lane == p) piv = r;
  }
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    if constexpr (CX) {
      const double t = re[j];
      re[j] = fma(t, sr, -im[j] * si);
      im[j] = fma(t, si, im[j] * sr);
    } else {
      re[j] *= sr;
    }
  }
}

// Inverses of one time block of every cell, one wavefront per cell (four
// independent ones per workgroup, so that a workgroup that ends leaves a whole
// slot on every SIMD of its compute unit for the coarse chain's workgroups that
// run beside; single wavefronts left the chain waiting and needed a cap): X_c =
// (t00 M + A) + i t10 M (real blocks: t00 M + A) of component c, bordered by
// the B columns and C rows of the components that share it (all of them where
// V_c is the same, else its own): lane = row (n velocity rows, D m border
// rows), its n + D m entries in registers, so an elimination step is one
// broadcast of the pivot row by readlane and one multiply-add per entry, with
// no LDS and no barrier.  The border ends as G, C V^-1 and the Schur sum.  Bound by
// VALU issue (a step is about 76 double readlanes and 152 multiply-adds in 3d).
// COMP (3d): written as the component store of k_vanka_comp; else as the
// time-decoupled rows of k_vanka_dec.
template <int D, bool CX, bool COMP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_inverse_comp(const int32_t* __restrict__ posmap, const double2* __restrict__ ma,
               const uint8_t* __restrict__ flags, const int32_t* __restrict__ own_ptr,
               const uint8_t* __restrict__ own_loc, const int64_t* __restrict__ inv_off, int ld,
               const int4* __restrict__ cinfo, const uint16_t* __restrict__ own_node, void* store,
               int fp32, uint8_t* __restrict__ status, int n_cells, double t00, double t10,
               int col_off, int accumulate) {
  constexpr int NV = D == 2 ? 9 : 27, NM = D + 1, NLS = D * NV + NM;
  constexpr int NB = D * NM, NC = NV + NB;
  static_assert(NC <= 64, "one row per lane");
  struct Wave {
    double2 zb[NB][NV];          // border rows: -C_c V_c^-1
    double2 corner[NB][NM];      // -C_c V_c^-1 B_c
    double2 sinv[NM][NM];
    int rowof[NV];               // stored node row of each node (COMP)
    double2 vs[D][NV];           // (V_c^-1 s)_i
    double2 ps[NB];              // C_c's rows of -C V^-1 s, then (P s_c)_m
    double2 gneg[NV][NB];        // G
    double2 vinv[COMP ? 1 : D][COMP ? 1 : NV][COMP ? 1 : NV];
    double2 prow[COMP ? 1 : NM][COMP ? 1 : NLS];
  };
  __shared__ Wave waves[4];
  const int lane = threadIdx.x & 63;
  Wave& sh = waves[threadIdx.x >> 6];
  auto& zb = sh.zb;
  auto& corner = sh.corner;
  auto& sinv = sh.sinv;
  auto& rowof = sh.rowof;
  auto& vinv = sh.vinv;
  auto& gneg = sh.gneg;
  auto& prow = sh.prow;
  auto put = [&](int64_t e, double v) {
    if (fp32) ((float*)store)[e] = (float)v;
    else ((double*)store)[e] = v;
  };
  const int T0 = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  for (int T = T0; T < n_cells; T += gridDim.x * 4) {
    const int32_t* pos = posmap + (int64_t)T * (NLS * NLS);
    const bool same = flags[T] & 1;
    bool sing = false;
    int R = 0, nptr = 0;
    int64_t base = 0;
    if constexpr (COMP) {
      const int4 ci = cinfo[T];
      base = ((int64_t)ci.y << 32) | (uint32_t)ci.x;
      nptr = ci.z;
      R = ci.w & 255;
      if (lane < NV) rowof[lane] = -1;
      wave_lds_sync();
      if (lane < R) rowof[own_node[nptr + lane] & 255] = lane;
      wave_lds_sync();
    }
    const int nvb = same ? 1 : D;
    double vmax[D];
#pragma unroll
    for (int c = 0; c < D; ++c) vmax[c] = 0.0;
    for (int c0 = 0; c0 < nvb; ++c0) {
      // border row (bc, bm) of lanes NV ..
      const int bb = lane - NV, bc = bb / NM, bm = bb - bc * NM;
      const bool vel = lane < NV, bor = lane >= NV && lane < NC && (same || bc == c0);
      double re[NC], im[CX ? NC : 1];
      // the row's entries, a sixth of them in flight at a time: the block
      // positions (those of no entry of this row replaced by the first), then
      // the values, chosen afterwards (the empty asm statements keep the
      // compiler from turning each choice into a branch around its load)
      constexpr int NG = 6, GC = (NC + NG - 1) / NG;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        int32_t q[GC];
        unsigned hv = 0;
#pragma unroll
        for (int k = 0; k < GC; ++k) {
          const int j = g * GC + k;
          if (j >= NC) continue;
          int at;
          bool have;
          if (j < NV) {
            at = vel ? (c0 * NV + lane) * NLS + c0 * NV + j : (D * NV + bm) * NLS + bc * NV + j;
            have = vel || bor;
          } else {
            const int jc = (j - NV) / NM, jm = (j - NV) - jc * NM;
            at = (jc * NV + lane) * NLS + D * NV + jm;
            have = vel && (same || jc == c0);
          }
          q[k] = pos[have ? at : 0];
          hv |= have ? 1u << k : 0u;
        }
        double2 f[GC];
#pragma unroll
        for (int k = 0; k < GC; ++k) {
          if (g * GC + k >= NC) continue;
          asm volatile("" : "+v"(q[k]));
          if (!((hv >> k) & 1u)) q[k] = -1;
          f[k] = ma[max(q[k], 0)];
        }
#pragma unroll
        for (int k = 0; k < GC; ++k) {
          const int j = g * GC + k;
          if (j >= NC) continue;
          asm volatile("" : "+v"(f[k].x), "+v"(f[k].y));
          re[j] = q[k] >= 0 ? fma(t00, f[k].x, f[k].y) : 0.0;
          if constexpr (CX) im[j] = q[k] >= 0 ? t10 * f[k].x : 0.0;
        }
      }
      double big = 0.0;
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        double m = fabs(re[j]);
        if constexpr (CX) m += fabs(im[j]);
        big = vel ? fmax(big, m) : 0.0;
      }
      int var, piv;
      gj_rows<NV, NC, CX>(re, im, lane, kPivotTol * wave_max_f64(big), var, piv, sing);
      // entry j of a row: border column j (j < NB), else column j - NB
      auto val = [&](int j) { return make_double2(re[j], CX ? im[CX ? j : 0] : 0.0); };
      if (lane >= NV && lane < NC && bor) {
#pragma unroll
        for (int jc = 0; jc < D; ++jc)
          if (jc == bc) {
#pragma unroll
            for (int m = 0; m < NM; ++m) corner[bb][m] = val(jc * NM + m);
          }
      }
      double2 rs = make_double2(0.0, 0.0);   // the row times s
      double rmax = 0.0;
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const int j = __builtin_amdgcn_readlane(piv, q);
        if (bor) zb[bb][j] = val(NB + q);
        if constexpr (!COMP) {
          if (vel) vinv[c0][var][j] = val(NB + q);
        }
        const double2 e = val(NB + q);
        const double sj = (kSigns >> j) & 1u ? -1.0 : 1.0;
        rs.x = fma(sj, e.x, rs.x);
        rs.y = fma(sj, e.y, rs.y);
        rmax = fmax(rmax, fabs(e.x) + fabs(e.y));
      }
      rmax = wave_max_f64(vel ? rmax : 0.0);
#pragma unroll
      for (int c = 0; c < D; ++c)
        if (same || c == c0) vmax[c] = rmax;
      if (bor) sh.ps[bb] = rs;
      if (vel) {
#pragma unroll
        for (int c = 0; c < D; ++c)
          if (same || c == c0) sh.vs[c][var] = rs;
#pragma unroll
        for (int b = 0; b < NB; ++b)
          if (same || b / NM == c0) {
            const double2 v = val(b);
            gneg[var][b] = make_double2(-v.x, -v.y);
          }
      }
      if constexpr (COMP) {
        // V part k-major: entry ((2 j + s) R + row), one block per distinct V_c
        const int o = vel ? rowof[var] : -1;
        if (o >= 0) {
          const int64_t vb = base + (int64_t)c0 * (2 * NV * R) + o;
#pragma unroll
          for (int q = 0; q < NV; ++q) {
            const int j = __builtin_amdgcn_readlane(piv, q);
            put(vb + (int64_t)(2 * j) * R, re[NB + q]);
            put(vb + (int64_t)(2 * j + 1) * R, CX ? im[CX ? NB + q : 0] : 0.0);
          }
          const int64_t gb = base + (int64_t)nvb * (2 * NV * R) + o;
#pragma unroll
          for (int b = 0; b < NB; ++b)
            if (same || b / NM == c0) {
              put(gb + (int64_t)(2 * b) * R, -re[b]);
              put(gb + (int64_t)(2 * b + 1) * R, CX ? -im[CX ? b : 0] : 0.0);
            }
        }
      }
    }
    wave_lds_sync();
    // S^-1, one row per lane
    double kappa;
    {
      double re[NM], im[CX ? NM : 1];
      double big = 0.0, part = 0.0;
      if (lane < NB) {
#pragma unroll
        for (int j = 0; j < NM; ++j)
          part = fmax(part, fabs(corner[lane][j].x) + fabs(corner[lane][j].y));
      }
#pragma unroll
      for (int j = 0; j < NM; ++j) {
        double2 f = make_double2(0.0, 0.0);
        if (lane < NM) {
#pragma unroll
          for (int c = 0; c < D; ++c) {
            const double2 g = corner[c * NM + lane][j];
            f.x += g.x;
            f.y += g.y;
          }
        }
        re[j] = f.x;
        if constexpr (CX) im[j] = f.y;
        big = fmax(big, fabs(f.x) + fabs(f.y));
      }
      int var, piv;
      const double bigs = wave_max_f64(big);
      gj_rows<NM, NM, CX>(re, im, lane, kPivotTol * bigs, var, piv, sing);
      double imax = 0.0;
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        const int j = __builtin_amdgcn_readlane(piv, q);
        const double2 e = make_double2(re[q], CX ? im[CX ? q : 0] : 0.0);
        if (lane < NM) {
          sinv[var][j] = e;
          imax = fmax(imax, fabs(e.x) + fabs(e.y));
        }
      }
      kappa = NM * fmax(bigs, wave_max_f64(part)) * wave_max_f64(imax);
    }
    wave_lds_sync();
    // cancellation between V^-1 and G P
    {
      double2 ps = make_double2(0.0, 0.0);
      if (lane < NB) {
        const int c = lane / NM, m = lane - c * NM;
#pragma unroll
        for (int k = 0; k < NM; ++k) {
          const double2 a = sinv[m][k], b = sh.ps[c * NM + k];
          ps.x += a.x * b.x - a.y * b.y;
          ps.y += a.x * b.y + a.y * b.x;
        }
      }
      wave_lds_sync();
      if (lane < NB) sh.ps[lane] = ps;
      wave_lds_sync();
#pragma unroll
      for (int c = 0; c < D; ++c) {
        double x = 0.0;
        if (lane < NV) {
          double2 v = sh.vs[c][lane];
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            const double2 g = gneg[lane][c * NM + m], q = sh.ps[c * NM + m];
            v.x += g.x * q.x - g.y * q.y;
            v.y += g.x * q.y + g.y * q.x;
          }
          x = fabs(v.x) + fabs(v.y);
        }
        if (!(kappa * vmax[c] <= kCancelTol * wave_max_f64(x))) sing = true;
      }
    }
    // pressure rows P = S^-1 [-C V^-1 | I], column e per lane
    for (int e = lane; e < (COMP ? 88 : NLS); e += 64) {
      const int c = e / NV, j = e - c * NV;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        double2 v = make_double2(0.0, 0.0);
        if (e < D * NV) {
#pragma unroll
          for (int k = 0; k < NM; ++k) {
            const double2 a = sinv[m][k], b = zb[c * NM + k][j];
            v.x += a.x * b.x - a.y * b.y;
            v.y += a.x * b.y + a.y * b.x;
          }
        } else if (e < NLS) {
          v = sinv[m][e - D * NV];
        }
        if constexpr (COMP) {
          const int ch = e / 22, k = e - ch * 22;
          const int64_t pb = base + (int64_t)(2 * NV * nvb + 2 * NB) * R;
          put(pb + (2 * k) * 16 + m * 4 + ch, v.x);
          put(pb + (2 * k + 1) * 16 + m * 4 + ch, v.y);
        } else {
          prow[m][e] = v;
        }
      }
    }
    if constexpr (!COMP) {
      wave_lds_sync();
      const int o0 = own_ptr[T], no = own_ptr[T + 1] - o0;
      const int64_t off = inv_off[T] + col_off;
      for (int e = lane; e < no * NLS; e += 64) {
        const int o = e / NLS, b = e - o * NLS;
        const int a = own_loc[o0 + o], c = a / NV, i = a - c * NV;
        double2 v;
        if (c == D) {
          v = prow[i][b];
        } else {
          v = b / NV == c ? vinv[same ? 0 : c][i][b - c * NV] : make_double2(0.0, 0.0);
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            const double2 g = gneg[i][c * NM + m], w = prow[m][b];
            v.x += g.x * w.x - g.y * w.y;
            v.y += g.x * w.y + g.y * w.x;
          }
        }
        put(off + (int64_t)o * ld + b, v.x);
        if constexpr (CX) put(off + (int64_t)o * ld + NLS + b, v.y);
      }
    }
    if (lane == 0) status[T] = (uint8_t)((sing ? 1 : 0) | (accumulate ? status[T] : 0));
    wave_lds_sync();
  }
}

// cap > 0: at most that many resident workgroups in 3d, striding over the cells
// (the caller leaves the other compute units to the coarse chain beside).
hipError_t launch_inverse_comp(hipStream_t s, const DevLevel& L, int fp32, uint8_t* status, int cap) {
  const double2* ma = (const double2*)L.kron_ma;
  int grid = (L.n_cells + 3) / 4;
  if (L.n_ls == 85 && cap > 0) grid = std::min(grid, cap);
#define STV_COMP(DD, CXX, ST, t0, t1, off, acc)                                               \
  {                                                                                          \
    k_inverse_comp<DD, CXX, ST><<<grid, 256, 0, s>>>(                                        \
        L.posmap, ma, L.comp_flags, L.own_ptr, L.own_loc, L.inv_off, L.inv_ld, L.comp_cell,  \
        L.comp_node, L.inv_store, fp32, status, L.n_cells, t0, t1, off, acc);                \
  }
  const CellSplit& S = L.split;
  if (L.n_ls == 85) {
    if (S.nblk != 1 || S.sz[0] != 2 || !L.comp_cell) return hipErrorInvalidValue;
    STV_COMP(3, true, true, S.T[0], S.T[2], 0, 0)
    return hipGetLastError();
  }
  const int B = S.b;
  for (int p = 0; p < S.nblk; ++p) {
    const int f = S.first[p];
    const double t0 = S.T[f * B + f];
    if (S.sz[p] == 1) STV_COMP(2, false, false, t0, 0.0, S.off[p], p > 0)
    else STV_COMP(2, true, false, t0, S.T[(f + 1) * B + f], S.off[p], p > 0)
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
#undef STV_COMP
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// Vanka cell sweep on the component store of a 3d dG(1) level (one complex
// pair), one wavefront per cell: with u = (I (x) W) rho_T (one complex number
// per spatial DoF),
//   p = P u (4 pressure modes),  y_(c, i) = (V_c^-1)_i. u_c + G_(c, i) p,
// and the update c_(a, i) = V_i0 Re y_a + V_i1 Im y_a of the owned DoFs.  The
// store per cell (R = owned nodes):
//   V part  [2 x 27][R]   re, im of V^-1 (node j, stored row) per distinct V_c
//   G part  [3 x 4 x 2][R]
//   P part  [2 x 22][16]  entry (2 k + s, 4 m + ch) = re/im of P[m][22 ch + k]
// The products are v_mfma_f64_16x16x4f64 (row = stored node, column = component
// and real/imaginary part; the complex product as a real one over (re, im) of
// the stored value): one load of the store per matrix instruction, V^-1 read
// once for the three components, and no lane reductions.  The P rows are cut
// into four chunks of 22 columns that use the instruction's row and column
// dimensions (row 4 m + ch against column 2 ch + part); the four diagonal
// chunks are added by readlane.  Bound by HBM: 10.6 kB per interior cell (8
// owned nodes) instead of 41 kB of whole complex rows.  A FP32 store is
// converted on load; all products are FP64.
template <typename TS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_vanka_comp(const double* __restrict__ rho,
                                                    double* __restrict__ d,
                                                    const int32_t* __restrict__ csd,
                                                    const int4* __restrict__ cinfo,
                                                    const int32_t* __restrict__ own_dof,
                                                    const TS* __restrict__ store, double omega,
                                                    int zero_init, int n_cells, CellSplit sp) {
  constexpr int NV = 27, NLS = 85, KV = 2 * NV, TV = 14, TG = 6, TP = 11, CH = 22;
  __shared__ double2 us[4][4 * CH];
  const int w = threadIdx.x >> 6;
  const double w00 = sp.W[0], w01 = sp.W[1], w10 = sp.W[2], w11 = sp.W[3];
  double2* u = us[w];
  const double* ud = reinterpret_cast<const double*>(u);
  const int T0 = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + w);
  for (int T = T0; T < n_cells; T += gridDim.x * 4) {
    // the per-lane index arithmetic stays inside the loop (hoisted, its
    // registers would cost the wavefronts that hide the loads)
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int lr = lane >> 4, lc = lane & 15;
    const int comp = lc >> 1, part = lc & 1, sreim = lr & 1, jhalf = lr >> 1;
    const bool act = lc < 6;
    // element of u (re or im) that a lane's operand takes, and its sign
    const int sel = sreim ^ part;
    const double sgn = (sreim && !part) ? -1.0 : 1.0;
    const double vr = part ? sp.V[2] : sp.V[0], vi = part ? sp.V[3] : sp.V[1];
    const int4 ci = cinfo[T];
    const TS* A = store + (((int64_t)ci.y << 32) | (uint32_t)ci.x);
    const int32_t* own = own_dof + 3 * ci.z;
    const int R = ci.w & 255, nvb = (ci.w >> 8) & 255, pmask = ci.w >> 16;
    const int32_t* sd = csd + (int64_t)T * NLS;
    const int s0 = sd[lane], s1 = sd[lane < NLS - 64 ? 64 + lane : NLS - 1];
    const double2 r0 = *reinterpret_cast<const double2*>(&rho[(int64_t)s0 * 2]);
    const double2 r1 = *reinterpret_cast<const double2*>(&rho[(int64_t)s1 * 2]);
    const TS* Ap = A + (KV * nvb + 24) * R;
    auto at = [](const TS* p, int e) {
      return *reinterpret_cast<const TS*>(reinterpret_cast<const char*>(p) + (unsigned)e * (unsigned)sizeof(TS));
    };
    TS ap[TP];
#pragma unroll
    for (int t = 0; t < TP; ++t) ap[t] = at(Ap + 64 * t, lane);
    // the first tile of the velocity rows, first V block
    TS av[TV], ag[TG];
    auto load_v = [&](int tile, int c) {
      const int row = min(tile + lc, R - 1);
      const TS* Av = A + c * (KV * R);
#pragma unroll
      for (int t = 0; t < TV; ++t)   // rows past KV: the last one (their operand is 0)
        av[t] = at(Av + 4 * t * R, (4 * t + 3 < KV ? lr : min(lr, KV - 1 - 4 * t)) * R + row);
    };
    auto load_g = [&](int tile) {
      const TS* Ag = A + nvb * (KV * R);
      const int row = min(tile + lc, R - 1);
#pragma unroll
      for (int t = 0; t < TG; ++t) ag[t] = at(Ag + 4 * t * R, lr * R + row);
    };
    if (R > 0) {
      load_v(0, 0);
      load_g(0);
    }
    // owned DoFs of the tile: outputs 4 v + lr of component comp (-1: not
    // this lane's or not owned); no branch between the loads
    int gi[4];
    double dold[4];
    auto load_d = [&](int tile) {
      int g[4];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        g[v] = own[3 * min(tile + 4 * v + lr, R - 1) + (act ? comp : 0)];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        dold[v] = 0.0;
        gi[v] = act && tile + 4 * v + lr < R && g[v] >= 0 ? 2 * g[v] + part : -1;
      }
      if (!zero_init) {
#pragma unroll
        for (int v = 0; v < 4; ++v) dold[v] = d[max(2 * g[v], 0) + part];
      }
    };
    if (R > 0) load_d(0);
    const int pm = (lane >> 1) & 3;
    const bool pown = lane < 8 && ((pmask >> pm) & 1);
    const int64_t pgi = (int64_t)sd[3 * NV + pm] * 2 + part;
    const double pold = zero_init ? 0.0 : d[pgi];
    u[lane] = make_double2(fma(w00, r0.x, w01 * r0.y), fma(w10, r0.x, w11 * r0.y));
    if (lane < 4 * CH - 64)
      u[64 + lane] = lane < NLS - 64
                         ? make_double2(fma(w00, r1.x, w01 * r1.y), fma(w10, r1.x, w11 * r1.y))
                         : make_double2(0.0, 0.0);
    wave_lds_sync();
    __builtin_amdgcn_sched_barrier(0);
    // p = P u
    stv_d4 pacc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < TP; ++t) {
      const int dof = (lc < 8 ? comp : 0) * CH + 2 * t + jhalf;
      const double x = ud[2 * dof + sel];
      const double b = lc < 8 ? sgn * x : 0.0;
      pacc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)ap[t], b, pacc, 0, 0, 0);
    }
    double pr[4], pi[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      pr[m] = (readlane_f64(pacc[m], 0) + readlane_f64(pacc[m], 18)) +
              (readlane_f64(pacc[m], 36) + readlane_f64(pacc[m], 54));
      pi[m] = (readlane_f64(pacc[m], 1) + readlane_f64(pacc[m], 19)) +
              (readlane_f64(pacc[m], 37) + readlane_f64(pacc[m], 55));
    }
    // this lane's operands of p in the velocity rows
    double bp[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double qr = jhalf ? pr[2 * h + 1] : pr[2 * h], qi = jhalf ? pi[2 * h + 1] : pi[2 * h];
      bp[h] = act ? sgn * (sel ? qi : qr) : 0.0;
    }
    if (pown) {
      const double qr = pm & 2 ? (pm & 1 ? pr[3] : pr[2]) : (pm & 1 ? pr[1] : pr[0]);
      const double qi = pm & 2 ? (pm & 1 ? pi[3] : pi[2]) : (pm & 1 ? pi[1] : pi[0]);
      const double val = fma(vr, qr, vi * qi);
      d[pgi] = zero_init ? omega * val : fma(omega, val, pold);
    }
    __builtin_amdgcn_sched_barrier(0);
    const double* uv = ud + 2 * ((act ? comp : 0) * NV + jhalf) + sel;
    for (int tile = 0; tile < R; tile += 16) {
      if (tile > 0) {
        load_v(tile, 0);
        load_g(tile);
        load_d(tile);
      }
      stv_d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int t = 0; t < TG; ++t)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)ag[t], comp == (t >> 1) ? bp[t & 1] : 0.0,
                                                   acc, 0, 0, 0);
      for (int c = 0; c < nvb; ++c) {
        if (c > 0) load_v(tile, c);
        const bool mine = act && (nvb == 1 || comp == c);
#pragma unroll
        for (int t = 0; t < TV; ++t) {
          const int j = 2 * t + jhalf;
          const double x = uv[4 * t];   // j = NV: a value not used
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)av[t], mine && j < NV ? sgn * x : 0.0,
                                                     acc, 0, 0, 0);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double y = acc[v], z = dpp_f64<0xB1>(y);   // the other part (lane ^ 1)
        const double val = part ? fma(vr, z, vi * y) : fma(vr, y, vi * z);
        if (gi[v] >= 0) d[gi[v]] = zero_init ? omega * val : fma(omega, val, dold[v]);
      }
    }
    wave_lds_sync();
  }
}

hipError_t launch_vanka_comp(hipStream_t s, const DevLevel& L, const double* rho, double* d,
                             double omega, int zero_init, int fp32, unsigned grid) {
  if (!L.comp_cell || !L.comp_dof) return hipErrorInvalidValue;
  if (fp32)
    launch(k_vanka_comp<float>, dim3(grid), dim3(256), 0, s, rho, d, L.cell_sdofs, L.comp_cell,
           L.comp_dof, (const float*)L.inv_store, omega, zero_init, L.n_cells, L.split);
  else
    launch(k_vanka_comp<double>, dim3(grid), dim3(256), 0, s, rho, d, L.cell_sdofs, L.comp_cell,
           L.comp_dof, (const double*)L.inv_store, omega, zero_init, L.n_cells, L.split);
  return hipGetLastError();
}

}  // namespace stv
