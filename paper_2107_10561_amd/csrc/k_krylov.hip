// FP64 vector kernels of flexible GMRES: several dot products against one
// vector in a single pass (classical Gram-Schmidt, applied twice), the
// matching multi-axpy, and normalisation.  A vector may hold several
// independent instances (segments): every reduction and update is done per
// segment with that segment's scalars.  Reductions use a fixed number of
// partial sums folded in a fixed order, so results are bitwise repeatable.
#include "stv_internal.h"

namespace stv {

constexpr int kGroup = 8;
constexpr int kStepCols = 256;

int seg_blocks(const Segs& g) {
  // kDotBlocks shared among the instances, at least 4 each; for a batch also
  // enough that a thread of the longest instance takes about 16 elements
  // (instances of uneven length otherwise leave the longest ones a few
  // blocks)
  const int per = kDotBlocks / (g.nseg > 0 ? g.nseg : 1);
  int nb = per < 4 ? 4 : per;
  if (g.nseg > 1) {
    const int64_t by_len = (g.max_seg + 16 * 256 - 1) / (16 * 256);
    if (by_len > nb) nb = (int)(by_len < 65535 ? by_len : 65535);
  }
  return nb;
}

// partial[(z*nblk + blk)*kGroup + k] = sum over this block's slice of segment
// z of V_k . w
template <int NV>
__global__ void __launch_bounds__(256) k_multidot(const double* __restrict__ V, int64_t n,
                                                  const double* __restrict__ w,
                                                  const int64_t* __restrict__ seg,
                                                  double* __restrict__ partial) {
  __shared__ double red[NV][4];
  const int z = blockIdx.y;
  const int64_t lo = seg[z], hi = seg[z + 1];
  double acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.0;
  for (int64_t i = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < hi;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double wi = w[i];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = fma(V[(int64_t)k * n + i], wi, acc[k]);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double v = acc[k];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) red[k][wv] = v;
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    const int k = threadIdx.x;
    partial[((int64_t)z * gridDim.x + blockIdx.x) * kGroup + k] =
        (red[k][0] + red[k][1]) + (red[k][2] + red[k][3]);
  }
}

// out[z*ostride + k] = sum_blk partial[(z*nblk + blk)*kGroup + k], pairwise in
// a fixed order.
__global__ void __launch_bounds__(256) k_reduce_partials(const double* __restrict__ partial,
                                                         int nblk, int nv,
                                                         double* __restrict__ out,
                                                         int64_t ostride) {
  __shared__ double red[4];
  const int k = blockIdx.x, z = blockIdx.y;
  if (k >= nv) return;
  const double* pz = partial + (int64_t)z * nblk * kGroup;
  double acc = 0.0;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) acc += pz[(int64_t)b * kGroup + k];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0) red[wv] = acc;
  __syncthreads();
  if (threadIdx.x == 0) out[(int64_t)z * ostride + k] = (red[0] + red[1]) + (red[2] + red[3]);
}

hipError_t launch_multidot(hipStream_t s, const double* V, int m, const double* w, int64_t n,
                           const Segs& g, double* partial, double* out, int64_t ostride) {
  const int nblk = seg_blocks(g);
  for (int k0 = 0; k0 < m; k0 += kGroup) {
    const int nv = (m - k0) < kGroup ? (m - k0) : kGroup;
    const double* Vk = V + (int64_t)k0 * n;
    dim3 grid((unsigned)nblk, (unsigned)g.nseg);
    switch (nv) {
      case 1: k_multidot<1><<<grid, 256, 0, s>>>(Vk, n, w, g.seg, partial); break;
      case 2: k_multidot<2><<<grid, 256, 0, s>>>(Vk, n, w, g.seg, partial); break;
      case 3: k_multidot<3><<<grid, 256, 0, s>>>(Vk, n, w, g.seg, partial); break;
      case 4: k_multidot<4><<<grid, 256, 0, s>>>(Vk, n, w, g.seg, partial); break;
      case 5: k_multidot<5><<<grid, 256, 0, s>>>(Vk, n, w, g.seg, partial); break;
      case 6: k_multidot<6><<<grid, 256, 0, s>>>(Vk, n, w, g.seg, partial); break;
      case 7: k_multidot<7><<<grid, 256, 0, s>>>(Vk, n, w, g.seg, partial); break;
      default: k_multidot<8><<<grid, 256, 0, s>>>(Vk, n, w, g.seg, partial); break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_reduce_partials<<<dim3((unsigned)nv, (unsigned)g.nseg), 256, 0, s>>>(partial, nblk, nv,
                                                                          out + k0, ostride);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// w += sign * sum_k coef[z*cstride + k] V_k on segment z
__global__ void __launch_bounds__(256) k_multiaxpy(const double* __restrict__ V, int m,
                                                   const double* __restrict__ coef,
                                                   int64_t cstride, double sign,
                                                   double* __restrict__ w, int64_t n,
                                                   const int64_t* __restrict__ seg) {
  const int z = blockIdx.y;
  const int64_t i = seg[z] + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= seg[z + 1]) return;
  const double* cz = coef + (int64_t)z * cstride;
  double acc = 0.0;
  for (int k = 0; k < m; ++k) acc = fma(cz[k], V[(int64_t)k * n + i], acc);
  w[i] = fma(sign, acc, w[i]);
}

hipError_t launch_multiaxpy(hipStream_t s, const double* V, int m, const double* coef,
                            int64_t cstride, double sign, double* w, int64_t n, const Segs& g) {
  if (m <= 0) return hipSuccess;
  dim3 grid((unsigned)((g.max_seg + 255) / 256), (unsigned)g.nseg);
  k_multiaxpy<<<grid, 256, 0, s>>>(V, m, coef, cstride, sign, w, n, g.seg);
  return hipGetLastError();
}

// The update of one Gram-Schmidt pass fused with the products of the next
// (one read of V instead of two): on segment z
//   w <- w + sign * sum_k coef[z*cstride + k] V_k   (k < NV),
// then, with the updated w, the partial sums of V_k . w as k_multidot writes
// them (same blocks, same order of operations: the results equal those of
// k_multiaxpy followed by k_multidot).
template <int NV>
__global__ void __launch_bounds__(256) k_multiaxpy_dot(const double* __restrict__ V, int64_t n,
                                                       const double* __restrict__ coef,
                                                       int64_t cstride, double sign,
                                                       double* __restrict__ w,
                                                       const int64_t* __restrict__ seg,
                                                       double* __restrict__ partial) {
  __shared__ double red[NV][4];
  const int z = blockIdx.y;
  const int64_t lo = seg[z], hi = seg[z + 1];
  const double* cz = coef + (int64_t)z * cstride;
  double c[NV], acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    c[k] = cz[k];
    acc[k] = 0.0;
  }
  for (int64_t i = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < hi;
       i += (int64_t)gridDim.x * blockDim.x) {
    double v[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = V[(int64_t)k * n + i];
    double a = 0.0;
#pragma unroll
    for (int k = 0; k < NV; ++k) a = fma(c[k], v[k], a);
    const double wi = fma(sign, a, w[i]);
    w[i] = wi;
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = fma(v[k], wi, acc[k]);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double t = acc[k];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, 64);
    if (lane == 0) red[k][wv] = t;
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    const int k = threadIdx.x;
    partial[((int64_t)z * gridDim.x + blockIdx.x) * kGroup + k] =
        (red[k][0] + red[k][1]) + (red[k][2] + red[k][3]);
  }
}

// The second pass's update fused with the squared norm of its result:
// w <- w + sign * sum_k coef[z*cstride + k] V_k (any m), and the partial sums
// of w . w (slot 0), as k_multiaxpy followed by k_multidot of w with itself.
__global__ void __launch_bounds__(256) k_multiaxpy_nrm(const double* __restrict__ V, int m,
                                                       int64_t n, const double* __restrict__ coef,
                                                       int64_t cstride, double sign,
                                                       double* __restrict__ w,
                                                       const int64_t* __restrict__ seg,
                                                       double* __restrict__ partial) {
  __shared__ double red[4];
  const int z = blockIdx.y;
  const int64_t lo = seg[z], hi = seg[z + 1];
  const double* cz = coef + (int64_t)z * cstride;
  double acc = 0.0;
  for (int64_t i = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < hi;
       i += (int64_t)gridDim.x * blockDim.x) {
    double a = 0.0;
    for (int k = 0; k < m; ++k) a = fma(cz[k], V[(int64_t)k * n + i], a);
    const double wi = fma(sign, a, w[i]);
    w[i] = wi;
    acc = fma(wi, wi, acc);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0) red[wv] = acc;
  __syncthreads();
  if (threadIdx.x == 0)
    partial[((int64_t)z * gridDim.x + blockIdx.x) * kGroup] = (red[0] + red[1]) + (red[2] + red[3]);
}

hipError_t launch_multiaxpy_dot(hipStream_t s, const double* V, int m, const double* coef,
                                int64_t cstride, double sign, double* w, int64_t n,
                                const Segs& g, double* partial, double* out, int64_t ostride) {
  if (m < 1 || m > kGroup) return hipErrorInvalidValue;
  const int nblk = seg_blocks(g);
  dim3 grid((unsigned)nblk, (unsigned)g.nseg);
#define STV_AXD(NN) k_multiaxpy_dot<NN><<<grid, 256, 0, s>>>(V, n, coef, cstride, sign, w, g.seg, partial)
  switch (m) {
    case 1: STV_AXD(1); break;
    case 2: STV_AXD(2); break;
    case 3: STV_AXD(3); break;
    case 4: STV_AXD(4); break;
    case 5: STV_AXD(5); break;
    case 6: STV_AXD(6); break;
    case 7: STV_AXD(7); break;
    default: STV_AXD(8); break;
  }
#undef STV_AXD
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_reduce_partials<<<dim3((unsigned)m, (unsigned)g.nseg), 256, 0, s>>>(partial, nblk, m, out,
                                                                        ostride);
  return hipGetLastError();
}

hipError_t launch_multiaxpy_nrm(hipStream_t s, const double* V, int m, const double* coef,
                                int64_t cstride, double sign, double* w, int64_t n,
                                const Segs& g, double* partial, double* out, int64_t ostride) {
  if (m < 1) return hipErrorInvalidValue;
  const int nblk = seg_blocks(g);
  k_multiaxpy_nrm<<<dim3((unsigned)nblk, (unsigned)g.nseg), 256, 0, s>>>(V, m, n, coef, cstride,
                                                                        sign, w, g.seg, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_reduce_partials<<<dim3(1u, (unsigned)g.nseg), 256, 0, s>>>(partial, nblk, 1, out, ostride);
  return hipGetLastError();
}

// v = w / sqrt(nrm2[z*nstride]) on segment z (0 where the norm is 0)
__global__ void k_scale_by_norm(const double* __restrict__ w, const double* __restrict__ nrm2,
                                int64_t nstride, double* __restrict__ v,
                                const int64_t* __restrict__ seg) {
  const int z = blockIdx.y;
  const int64_t i = seg[z] + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= seg[z + 1]) return;
  const double nr = sqrt(nrm2[(int64_t)z * nstride]);
  v[i] = nr > 0.0 ? w[i] / nr : 0.0;
}

hipError_t launch_scale_by_norm(hipStream_t s, const double* w, const double* nrm2,
                                int64_t nstride, double* v, const Segs& g) {
  dim3 grid((unsigned)((g.max_seg + 255) / 256), (unsigned)g.nseg);
  k_scale_by_norm<<<grid, 256, 0, s>>>(w, nrm2, nstride, v, g.seg);
  return hipGetLastError();
}

// One Arnoldi step's Gram-Schmidt on short segments, a workgroup per segment
// with its part of w in registers (E entries per thread):
//   h1 = V'w, w -= V h1, h2 = V'w, w -= V h2, nrm = w.w, v = w / ||w||
// (0 where the norm is 0), V's columns in groups of kGroup.  Bound by latency
// either way: the separate kernels are 7 launches up to 8 columns and 20 at 30.
constexpr int kStepThreads = 1024;   // 16 wavefronts (step_sums)

// Sum over the workgroup of acc[lane & 7], in every lane.
__device__ __forceinline__ double step_sums(double (&acc)[kGroup], double (*red)[kGroup]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  // eight sums over 64 lanes by exchange: lane l ends with sum l >> 3
#pragma unroll
  for (int half = 4, off = 32; half >= 1; half >>= 1, off >>= 1) {
    const bool hi = lane & off;
#pragma unroll
    for (int k = 0; k < half; ++k) {
      const double a = acc[k], b = acc[k + half];
      acc[k] = (hi ? b : a) + __shfl_xor(hi ? a : b, off, 64);
    }
  }
  double t = acc[0];
#pragma unroll
  for (int off = 4; off >= 1; off >>= 1) t += __shfl_xor(t, off, 64);
  __syncthreads();   // the last sums have been read
  if ((lane & 7) == 0) red[wv][lane >> 3] = t;
  __syncthreads();
  // 16 wavefronts' sums: two per lane, then over the lanes of equal lane & 7
  double u = red[lane >> 3][lane & 7] + red[8 + (lane >> 3)][lane & 7];
#pragma unroll
  for (int off = 8; off <= 32; off <<= 1) u += __shfl_xor(u, off, 64);
  return u;
}

template <int E>
__global__ void __launch_bounds__(kStepThreads) k_cgs2_step(const double* __restrict__ V, int m,
                                                            int64_t n,
                                                            const double* __restrict__ w,
                                                            const int64_t* __restrict__ seg,
                                                            double* __restrict__ h1,
                                                            double* __restrict__ h2,
                                                            int64_t hstride,
                                                            double* __restrict__ nrm,
                                                            double* __restrict__ v) {
  __shared__ double red[kStepThreads / 64][kGroup];
  __shared__ double coef[kStepCols];
  const int z = blockIdx.x, tid = threadIdx.x;
  const int64_t lo = seg[z], hi = seg[z + 1];
  // entries past the segment's end: its last one, weighted by zero
  int64_t at[E];
  double x[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int64_t i = lo + tid + (int64_t)e * kStepThreads;
    at[e] = i < hi ? i : hi - 1;
    x[e] = i < hi ? w[at[e]] : 0.0;
  }
  for (int pass = 0; pass < 2; ++pass) {
    double* h = (pass ? h2 : h1) + z * hstride;
    for (int k0 = 0; k0 < m; k0 += kGroup) {
      double acc[kGroup];
#pragma unroll
      for (int k = 0; k < kGroup; ++k) {
        const double* col = V + (int64_t)min(k0 + k, m - 1) * n;
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) s = fma(col[at[e]], x[e], s);
        acc[k] = s;
      }
      const double sum = step_sums(acc, red);
      if (tid < kGroup && k0 + tid < m) {
        coef[k0 + tid] = sum;
        h[k0 + tid] = sum;
      }
    }
    __syncthreads();
    double s[E];
#pragma unroll
    for (int e = 0; e < E; ++e) s[e] = 0.0;
#pragma unroll 4
    for (int k = 0; k < m; ++k) {
      const double c = coef[k];
#pragma unroll
      for (int e = 0; e < E; ++e) s[e] = fma(c, V[(int64_t)k * n + at[e]], s[e]);
    }
#pragma unroll
    for (int e = 0; e < E; ++e)
      x[e] = lo + tid + (int64_t)e * kStepThreads < hi ? x[e] - s[e] : 0.0;
    __syncthreads();   // coef has been read
  }
  double acc[kGroup] = {};
#pragma unroll
  for (int e = 0; e < E; ++e) acc[0] = fma(x[e], x[e], acc[0]);
  const double nr2 = __shfl(step_sums(acc, red), 0, 64);
  const double nr = sqrt(nr2);
  if (tid == 0) nrm[z] = nr2;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int64_t i = lo + tid + (int64_t)e * kStepThreads;
    if (i < hi) v[i] = nr > 0.0 ? x[e] / nr : 0.0;
  }
}

// Four entries per thread: one compute unit reads V's columns four times, which
// at 7,332 entries costs more than the launches (10 and 30 steps of FGMRES on
// 2d operators, separate kernels -> one: 402 entries 0.85 -> 0.65 and 3.44 ->
// 2.06 ms, 1,540 0.91 -> 0.73 and 3.65 -> 2.38, 3,012 0.93 -> 0.81 and 3.64 ->
// 2.77, 7,332 0.98 -> 1.07 and 3.81 -> 4.41).
bool cgs2_step_fits(int m, const Segs& g) {
  return m <= kStepCols && g.max_seg <= 4 * kStepThreads;
}

hipError_t launch_cgs2_step(hipStream_t s, const double* V, int m, const double* w, int64_t n,
                            const Segs& g, double* h1, double* h2, int64_t hstride, double* nrm,
                            double* v) {
  if (m < 1 || !cgs2_step_fits(m, g)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)g.nseg);
  const int64_t e = (g.max_seg + kStepThreads - 1) / kStepThreads;
#define STV_STEP(E) \
  k_cgs2_step<E><<<grid, kStepThreads, 0, s>>>(V, m, n, w, g.seg, h1, h2, hstride, nrm, v)
  if (e <= 1) STV_STEP(1);
  else if (e <= 2) STV_STEP(2);
  else STV_STEP(4);
#undef STV_STEP
  return hipGetLastError();
}

}  // namespace stv
