// K3: per-element tensor-product transfers between p-levels (Sec. 3.2):
//   out (=|+=) (T x T x T)(in - in2),  T: n_out x n_in,
// used for P (projection), R = I^T (restriction) and I (prolongation).
// K4: BLAS-1 pieces of SCG (Alg. 6) with fixed-shape two-stage reductions, so
// every dot product is bitwise reproducible.
#include <algorithm>

#include "device.hpp"
#include "kernels.hpp"
#include "blas.hpp"

namespace dgfas {

// A thread contracts whole lines: each of the three directions reads NI values of a line, gives NO,
// and the transfer's rows come through the scalar cache, so that a value crosses LDS once a step and
// no thread reads a row of T.  With NI >= NO the first step takes the lines along z straight from
// global memory (consecutive threads, consecutive nodes), then x, then y; with NI < NO it takes y
// first and z last, so that the larger array, then the output, is the one accessed node by node.
// Old output values (accumulate) are loaded before the first step.  Bound: the two arrays' bytes.
// EPB elements fill about 256 threads with the longer of the first and the last step's lines.
// Measured, p = 8 <-> 4 on 24^3: restriction 52.0 -> 15.5 us (6.1 TB/s), prolongation 57.8 -> 27.7 (7.0
// TB/s) against one node a thread; 5 <-> 2 on 24^3: 11.1 -> 4.6, 13.9 -> 7.8; 6^3 grids 4.3 as before.
template <int NI, int NO>
struct TrShape {
  static constexpr int ML = NI > NO ? NI * NI : NO * NO;
  static constexpr int EPB = 256 / ML;
  static constexpr int THREADS = ((EPB * ML + 63) / 64) * 64;
  static constexpr int RI = NI | 1, RO = NO | 1;   // odd rows: lines along a row read without bank conflicts
};

template <typename T>
using trtab = const __attribute__((address_space(4))) T*;

// out[m] = sum_k T[m][k] in[k], T at a uniform address
template <int NI, int NO, typename T>
__device__ __forceinline__ void line_transfer(trtab<T> Tm, const T (&in)[NI], T (&out)[NO]) {
#pragma unroll
  for (int m = 0; m < NO; ++m) {
    T s = 0;
#pragma unroll
    for (int k = 0; k < NI; ++k) s += Tm[m * NI + k] * in[k];
    out[m] = s;
  }
}

// Element e of the launch list, sub-block s = rhs * ncomp + comp:
//   in  + rhs * stride_in  + off_in[e]  * ncomp + comp * NI^3
//   out + rhs * stride_out + off_out[e] * ncomp + comp * NO^3
template <int NI, int NO, typename T>
__global__ void __launch_bounds__((TrShape<NI, NO>::THREADS))
tensor3_kernel(XferArgs<T> a) {
  using S = TrShape<NI, NO>;
  constexpr int EPB = S::EPB, RI = S::RI, RO = S::RO, I3 = NI * NI * NI, O3 = NO * NO * NO;
  constexpr int L1 = NI * NI, L2 = NI * NO, L3 = NO * NO;
  constexpr bool ZFIRST = NI >= NO;
  const int nsub = a.nrhs * a.ncomp;
  const int lbs = xcd_block(((a.nel + EPB - 1) / EPB) * nsub);
  if (lbs < 0) return;
  const int lb = lbs / nsub, sub = lbs - lb * nsub;
  const int rhs = sub / a.ncomp, comp = sub - rhs * a.ncomp;
  const int tid = threadIdx.x, here = min(EPB, a.nel - lb * EPB);   // elements of this block
  const trtab<T> Tm = (trtab<T>)(uintptr_t)a.Tm;
  __shared__ T s1[EPB][L2 * RI];   // first step's lines laid down along x: row (z or k, j or b), RI a row
  __shared__ T s2[EPB][L2 * RO];
  auto elem = [&](int le) {
    const int li = lb * EPB + le;
    return a.elist ? a.elist[li] : li;
  };
  const int le3 = tid / L3, q3 = tid - le3 * L3;
  const bool act3 = le3 < here && tid < EPB * L3;
  // node (c, b, a) of the last step's line: c (ZFIRST) or b, and a fixed
  const int o3 = ZFIRST ? (q3 / NO) * L3 + q3 % NO : q3;
  constexpr int so = ZFIRST ? NO : L3;
  T old[NO];
  T* op = nullptr;
  if (act3) {
    const int e = elem(le3);
    op = a.out + (int64_t)rhs * a.stride_out + (a.off_out ? a.off_out[e] : (int64_t)e * O3) * a.ncomp +
         (int64_t)comp * O3 + o3;
    if (a.accumulate) {
#pragma unroll
      for (int m = 0; m < NO; ++m) old[m] = op[m * so];
    }
  }
  {
    const int le = tid / L1, q = tid - le * L1;
    if (le < here && tid < EPB * L1) {
      const int e = elem(le);
      constexpr int si = ZFIRST ? NI * NI : NI;
      const int hi = q / NI, x = q - hi * NI;
      const int64_t ib = (int64_t)rhs * a.stride_in + (a.off_in ? a.off_in[e] : (int64_t)e * I3) * a.ncomp +
                         (int64_t)comp * I3 + (ZFIRST ? q : hi * NI * NI + x);
      T v[NI], w[NO];
#pragma unroll
      for (int k = 0; k < NI; ++k) v[k] = a.in[ib + k * si];
      if (a.in2) {
#pragma unroll
        for (int k = 0; k < NI; ++k) v[k] -= a.in2[ib + k * si];
      }
      line_transfer<NI, NO, T>(Tm, v, w);
#pragma unroll
      for (int m = 0; m < NO; ++m) s1[le][(ZFIRST ? m * NI + hi : hi * NO + m) * RI + x] = w[m];
    }
  }
  __syncthreads();
  {
    const int le = tid / L2, q = tid - le * L2;
    if (le < here && tid < EPB * L2) {
      T v[NI], w[NO];
#pragma unroll
      for (int k = 0; k < NI; ++k) v[k] = s1[le][q * RI + k];
      line_transfer<NI, NO, T>(Tm, v, w);
#pragma unroll
      for (int m = 0; m < NO; ++m) s2[le][q * RO + m] = w[m];
    }
  }
  __syncthreads();
  if (act3) {
    const int hi = q3 / NO, x = q3 - hi * NO;
    T v[NI], w[NO];
#pragma unroll
    for (int k = 0; k < NI; ++k) v[k] = s2[le3][(ZFIRST ? hi * NI + k : k * NO + hi) * RO + x];
    line_transfer<NI, NO, T>(Tm, v, w);
#pragma unroll
    for (int m = 0; m < NO; ++m) op[m * so] = a.accumulate ? old[m] + w[m] : w[m];
  }
}

template <int NI, int NO, typename T>
void launch_t3(const XferArgs<T>& a, hipStream_t st) {
  using S = TrShape<NI, NO>;
  const int nb = ((a.nel + S::EPB - 1) / S::EPB) * a.nrhs * a.ncomp;
  hipLaunchKernelGGL((tensor3_kernel<NI, NO, T>), dim3(xcd_grid(nb)), dim3(S::THREADS), 0, st, a);
}

template <typename T>
bool tensor3(int n_in, int n_out, const XferArgs<T>& a, hipStream_t st) {
  if (a.nel <= 0) return true;
#define T3C(x, y) \
  if (n_in == x && n_out == y) { launch_t3<x, y, T>(a, st); return true; }
  // p-coarsening pairs (p_c = max(1, p_f / 2)), identity-degree copies and the
  // interpolations between any two degrees 1..8 used on mixed-degree meshes
  T3C(2, 2) T3C(2, 3) T3C(2, 4) T3C(2, 5) T3C(2, 6) T3C(2, 7) T3C(2, 8) T3C(2, 9)
  T3C(3, 2) T3C(3, 3) T3C(3, 4) T3C(3, 5) T3C(3, 6) T3C(3, 7) T3C(3, 8) T3C(3, 9)
  T3C(4, 2) T3C(4, 3) T3C(4, 4) T3C(4, 5) T3C(4, 6) T3C(4, 7) T3C(4, 8) T3C(4, 9)
  T3C(5, 2) T3C(5, 3) T3C(5, 4) T3C(5, 5) T3C(5, 6) T3C(5, 7) T3C(5, 8) T3C(5, 9)
  T3C(6, 2) T3C(6, 3) T3C(6, 4) T3C(6, 5) T3C(6, 6) T3C(6, 7) T3C(6, 8) T3C(6, 9)
  T3C(7, 2) T3C(7, 3) T3C(7, 4) T3C(7, 5) T3C(7, 6) T3C(7, 7) T3C(7, 8) T3C(7, 9)
  T3C(8, 2) T3C(8, 3) T3C(8, 4) T3C(8, 5) T3C(8, 6) T3C(8, 7) T3C(8, 8) T3C(8, 9)
  T3C(9, 2) T3C(9, 3) T3C(9, 4) T3C(9, 5) T3C(9, 6) T3C(9, 7) T3C(9, 8) T3C(9, 9)
#undef T3C
  return false;
}

template bool tensor3<double>(int, int, const XferArgs<double>&, hipStream_t);
template bool tensor3<float>(int, int, const XferArgs<float>&, hipStream_t);

// One workgroup per (parent, component, right-hand side), one thread per node: kinds 0 and 1
// gather the eight children (each contracted with its bits' 1D matrices through LDS, summed in
// child order), kind 2 contracts the parent's block once per child and adds it there.
template <int N, typename T>
__global__ void __launch_bounds__((N * N * N + 63) / 64 * 64) htransfer_kernel(HXferArgs<T> a) {
  constexpr int N2 = N * N, N3 = N * N * N;
  const int nsub = a.nrhs * a.ncomp;
  const int pidx = blockIdx.x / nsub, sub = blockIdx.x - pidx * nsub;
  if (pidx >= a.ncoarse) return;
  const int parent = a.parents ? a.parents[pidx] : pidx;
  const int rhs = sub / a.ncomp, comp = sub - rhs * a.ncomp;
  const int q = threadIdx.x;
  const bool act = q < N3;
  const int x = q % N, y = (q / N) % N, z = q / N2;
  __shared__ T sM[6][N2];
  __shared__ T s0[N3], s1[N3], s2[N3];
  for (int t = q; t < 6 * N2; t += blockDim.x) sM[t / N2][t % N2] = a.M[t];
  const int64_t cb = (int64_t)rhs * a.stride_c + ((int64_t)parent * a.ncomp + comp) * N3;
  // out_node = sum_k Mz[z][k] sum_j My[y][j] sum_i Mx[x][i] s0[k][j][i]
  auto contract = [&](const T* Mx, const T* My, const T* Mz) -> T {
    __syncthreads();
    if (act) {
      T v = 0;
      for (int i = 0; i < N; ++i) v += Mx[x * N + i] * s0[(z * N + y) * N + i];
      s1[q] = v;
    }
    __syncthreads();
    if (act) {
      T v = 0;
      for (int j = 0; j < N; ++j) v += My[y * N + j] * s1[(z * N + j) * N + x];
      s2[q] = v;
    }
    __syncthreads();
    T v = 0;
    if (act)
      for (int k = 0; k < N; ++k) v += Mz[z * N + k] * s2[(k * N + y) * N + x];
    return v;
  };
  if (a.kind <= 1) {
    const int m0 = a.kind == 0 ? 0 : 2;
    T acc = 0;
    for (int c = 0; c < 8; ++c) {
      const int bx = c & 1, by = (c >> 1) & 1, bz = c >> 2;
      const int child = a.children[(int64_t)pidx * 8 + c];
      __syncthreads();   // the previous child's contraction has read s0
      if (act) s0[q] = a.in[(int64_t)rhs * a.stride_f + ((int64_t)child * a.ncomp + comp) * N3 + q];
      acc += contract(sM[m0 + bx], sM[m0 + by], sM[m0 + bz]);
    }
    if (act) a.out[cb + q] = a.accumulate ? a.out[cb + q] + acc : acc;
  } else {
    if (act) s0[q] = a.in[cb + q] - (a.in2 ? a.in2[cb + q] : T(0));
    for (int c = 0; c < 8; ++c) {
      const int bx = c & 1, by = (c >> 1) & 1, bz = c >> 2;
      const int child = a.children[(int64_t)pidx * 8 + c];
      const T v = contract(sM[4 + bx], sM[4 + by], sM[4 + bz]);
      if (act) {
        T& o = a.out[(int64_t)rhs * a.stride_f + ((int64_t)child * a.ncomp + comp) * N3 + q];
        o = a.accumulate ? o + v : v;   // every child node belongs to one parent: written once
      }
    }
  }
}

template <typename T>
bool htransfer(int p, const HXferArgs<T>& a, hipStream_t st) {
  if (a.ncoarse <= 0) return true;
  const dim3 g((unsigned)((int64_t)a.ncoarse * a.nrhs * a.ncomp));
  switch (p) {
#define HTC(P) \
  case P: hipLaunchKernelGGL((htransfer_kernel<P + 1, T>), g, dim3(((P + 1) * (P + 1) * (P + 1) + 63) / 64 * 64), 0, st, a); return true;
    HTC(1) HTC(2) HTC(3) HTC(4) HTC(5) HTC(6) HTC(7) HTC(8)
#undef HTC
    default: return false;
  }
}
template bool htransfer<double>(int, const HXferArgs<double>&, hipStream_t);

__global__ void __launch_bounds__(256) copy_rows_kernel(const int* __restrict__ list, int n, int n3,
                                                        const double* __restrict__ src, double* __restrict__ dst) {
  const int i = blockIdx.x;
  if (i >= n) return;
  const int64_t o = (int64_t)list[i] * n3;
  for (int q = threadIdx.x; q < n3; q += blockDim.x) dst[o + q] = src[o + q];
}

void copy_rows(const int* list, int n, int n3, const double* src, double* dst, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(copy_rows_kernel, dim3(n), dim3(256), 0, st, list, n, n3, src, dst);
}

__global__ void __launch_bounds__(256) rows_sumsq_kernel(const int* __restrict__ list, int n, int n3,
                                                         const double* __restrict__ v, double* __restrict__ out) {
  __shared__ double sh[256];
  const int i = blockIdx.x;
  if (i >= n) return;
  const int64_t o = (int64_t)list[i] * n3;
  double s = 0;
  for (int q = threadIdx.x; q < n3; q += blockDim.x) s += v[o + q] * v[o + q];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[i] = sh[0];
}

void rows_sumsq(const int* list, int n, int n3, const double* v, double* out, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(rows_sumsq_kernel, dim3(n), dim3(256), 0, st, list, n, n3, v, out);
}

// ---------------------------------------------------------------------------
constexpr int kRedThreads = 256;

int reduction_blocks(int64_t n) {
  int64_t b = (n + kRedThreads * 8 - 1) / (kRedThreads * 8);
  if (b < 1) b = 1;
  if (b > 1024) b = 1024;
  return (int)b;
}

// v -= mean(v), per right-hand side: block sums in a fixed order, then every thread adds the
// (at most 1024) block sums of its right-hand side in order and subtracts the mean
__global__ void __launch_bounds__(kRedThreads) sum_partial_kernel(int64_t n, const double* __restrict__ v,
                                                                 double* __restrict__ partial) {
  __shared__ double sh[kRedThreads];
  const double* x = v + (int64_t)blockIdx.y * n;
  double s = 0;
  for (int64_t i = (int64_t)blockIdx.x * kRedThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kRedThreads)
    s += x[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int k = kRedThreads / 2; k > 0; k >>= 1) {
    if (threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[(int64_t)blockIdx.y * 1024 + blockIdx.x] = sh[0];
}

__global__ void __launch_bounds__(kRedThreads) subtract_mean_kernel(int64_t n, int nb, double* __restrict__ v,
                                                                   const double* __restrict__ partial) {
  __shared__ double mean;
  if (threadIdx.x == 0) {
    double s = 0;
    for (int b = 0; b < nb; ++b) s += partial[(int64_t)blockIdx.y * 1024 + b];
    mean = s / (double)n;
  }
  __syncthreads();
  double* x = v + (int64_t)blockIdx.y * n;
  for (int64_t i = (int64_t)blockIdx.x * kRedThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kRedThreads)
    x[i] -= mean;
}

void project_mean(int64_t n, int nrhs, double* v, double* partial, hipStream_t st) {
  const int nb = reduction_blocks(n);
  hipLaunchKernelGGL(sum_partial_kernel, dim3(nb, nrhs), dim3(kRedThreads), 0, st, n, v, partial);
  hipLaunchKernelGGL(subtract_mean_kernel, dim3(nb, nrhs), dim3(kRedThreads), 0, st, n, nb, v, partial);
}

// sum over the workgroup in thread 0 (the wavefronts' sums in order); sh: one slot per wavefront
__device__ __forceinline__ double block_sum(double v, double* sh) {
  const int tid = threadIdx.x;
  v = wave_sum(v);
  if ((tid & 63) == 0) sh[tid >> 6] = v;
  __syncthreads();
  double s = 0;
  if (tid == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += sh[w];
  return s;
}

// Batched reductions: vectors are [nrhs][n]; block (blk, rhs) writes
// partial[rhs * 1024 + blk] = sum_i a_i (b_i - c_i) over its strided share of right-hand
// side rhs (b, c may be null: b := a, c := 0), accumulated in FP64.
template <typename T>
__global__ void __launch_bounds__(kRedThreads)
dot_partial_kernel(int64_t n, const T* __restrict__ a, const T* __restrict__ b, const T* __restrict__ c,
                   double* __restrict__ partial) {
  __shared__ double sh[kRedThreads / 64];
  const int64_t off = (int64_t)blockIdx.y * n;
  a += off;
  if (b) b += off;
  if (c) c += off;
  double s = 0;
  const int64_t stride = (int64_t)gridDim.x * kRedThreads;
  for (int64_t i = (int64_t)blockIdx.x * kRedThreads + threadIdx.x; i < n; i += stride) {
    const double bv = b ? (double)b[i] : (double)a[i];
    s += (double)a[i] * (c ? bv - (double)c[i] : bv);
  }
  const double t = block_sum(s, sh);
  if (threadIdx.x == 0) partial[blockIdx.y * 1024 + blockIdx.x] = t;
}

template <typename T>
void dot_partials(int64_t n, int nrhs, const T* a, const T* b, const T* c, double* partial, int nblocks,
                  hipStream_t st) {
  hipLaunchKernelGGL((dot_partial_kernel<T>), dim3(nblocks, nrhs), dim3(kRedThreads), 0, st, n, a, b, c, partial);
}
template void dot_partials<double>(int64_t, int, const double*, const double*, const double*, double*, int,
                                   hipStream_t);
template void dot_partials<float>(int64_t, int, const float*, const float*, const float*, double*, int, hipStream_t);

// Second stage, one block per right-hand side: sums its partials (for kOpBeta also the
// second set at partial2) and applies the SCG scalar update selected by `op`.
//   scal[rhs * 8 + k]: 0 gamma (z^T r)  1 beta  2 alpha  3 r^T r  4 breakdown flag
//                      5 iterations run before convergence  6 stopping threshold on |r|
//                      (0: none)  7 converged flag
// A right-hand side whose |r| has reached its threshold is frozen (alpha = 0 from then on),
// so that in a batch every right-hand side stops at the iteration it would stop at alone.
__global__ void __launch_bounds__(1024) finish_kernel(int nblocks, const double* __restrict__ partial,
                                                      const double* __restrict__ partial2, int op,
                                                      double* __restrict__ scal, double* __restrict__ out,
                                                      int pstride) {
  __shared__ double sh[2][16];
  const int tid = threadIdx.x, rhs = blockIdx.x, nt = blockDim.x;
  const double* __restrict__ p1 = partial + (int64_t)rhs * pstride;
  const double* __restrict__ p2 = partial2 + (int64_t)rhs * pstride;   // read for kOpBeta only
  const bool two = op == kOpBeta;
  double v0 = 0, v1 = 0;
  // eight partials per step, all loads ahead of the sums: one load at a time waited for memory
  // 32 times over the 32768 tiles of a 32^3, p = 7 level (17 us a launch; now 8)
  for (int b0 = tid; b0 < nblocks; b0 += 8 * nt) {
    double x[8], y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int b = min(b0 + k * nt, nblocks - 1);
      x[k] = p1[b];
      y[k] = two ? p2[b] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (b0 + k * nt < nblocks) {
        v0 += x[k];
        v1 += y[k];
      }
  }
  const double s0 = block_sum(v0, sh[0]);
  const double s1 = two ? block_sum(v1, sh[1]) : 0.0;
  if (tid != 0) return;
  double* sc = scal + rhs * 8;
  switch (op) {
    case kOpGamma:          // first iteration: gamma = z^T r
      sc[0] = s0;
      sc[1] = 0.0;
      break;
    case kOpBeta: {         // beta = z^T (r - r0) / gamma_old ; gamma = z^T r
      const double beta = s1 / sc[0];
      sc[1] = isfinite(beta) ? beta : 0.0;
      sc[0] = s0;
      if (!isfinite(beta)) sc[4] = 1.0;
      break;
    }
    case kOpAlpha: {        // alpha = gamma / p^T q; a converged right-hand side (p = 0) takes alpha = 0
      double alpha = (s0 != 0.0) ? sc[0] / s0 : 0.0;
      if (sc[7] != 0.0) alpha = 0.0;
      else if (s0 < 0.0 || !isfinite(alpha)) { sc[4] = 1.0; alpha = 0.0; }
      sc[2] = alpha;
      break;
    }
    case kOpNorm2:          // r^T r
      sc[3] = s0;
      if (!isfinite(s0)) sc[4] = 1.0;
      if (sc[7] == 0.0) {
        sc[5] += 1.0;
        if (sc[6] > 0.0 && sqrt(s0) <= sc[6]) sc[7] = 1.0;
      }
      break;
    case kOpStore:
      out[rhs] = s0;
      break;
  }
}

void finish(int nblocks, int nrhs, const double* partial, const double* partial2, int op, double* scal, double* out,
            hipStream_t st, int pstride) {
  // as many wavefronts as the partial sums fill with eight each, at most sixteen
  const int thr = std::min(1024, std::max(64, (nblocks / 8 + 63) / 64 * 64));
  hipLaunchKernelGGL(finish_kernel, dim3(nrhs), dim3(thr), 0, st, nblocks, partial, partial2, op, scal, out, pstride);
}

// p = beta p + z   (first: p = z), per right-hand side beta
template <typename T>
__global__ void pupdate_kernel(int64_t n, int nrhs, const T* __restrict__ z, T* __restrict__ p, T* __restrict__ x,
                               const double* __restrict__ scal, int first) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * nrhs) return;
  const int rhs = (int)(i / n);
  if (first) {
    p[i] = z[i];
    return;
  }
  const T po = p[i];
  if (x) x[i] += (T)scal[rhs * 8 + 2] * po;     // the previous iteration's u += alpha p
  p[i] = (T)scal[rhs * 8 + 1] * po + z[i];
}

// x += alpha p (the last iteration's update)
template <typename T>
__global__ void xupdate_kernel(int64_t n, int nrhs, T* __restrict__ x, const T* __restrict__ p,
                               const double* __restrict__ scal) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * nrhs) return;
  x[i] += (T)scal[(i / n) * 8 + 2] * p[i];
}

// y += (double)(x + alpha p): the last SCG update of an FP32 correction added straight to the
// FP64 iterate (the correction itself is not needed afterwards)
__global__ void xupdate_acc_kernel(int64_t n, int nrhs, const float* __restrict__ x, const float* __restrict__ p,
                                   const double* __restrict__ scal, double* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * nrhs) return;
  const float xn = x[i] + (float)scal[(i / n) * 8 + 2] * p[i];
  y[i] = y[i] + (double)xn;
}

void xupdate_acc(int64_t n, int nrhs, const float* x, const float* p, const double* scal, double* y, hipStream_t st) {
  const int64_t tot = n * nrhs;
  hipLaunchKernelGGL(xupdate_acc_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, nrhs, x, p, scal, y);
}

// rout = rin - alpha q (rout may be rin); partial[rhs*1024 + blk] = sum rout^2 (partial null: no sums)
template <typename T>
__global__ void __launch_bounds__(kRedThreads)
cg_update_kernel(int64_t n, const T* __restrict__ rin, T* __restrict__ rout, const T* __restrict__ q,
                 const double* __restrict__ scal, double* __restrict__ partial) {
  __shared__ double sh[kRedThreads / 64];
  const int rhs = blockIdx.y;
  const int64_t off = (int64_t)rhs * n;
  rin += off; rout += off; q += off;
  const T alpha = (T)scal[rhs * 8 + 2];
  double s = 0;
  const int64_t stride = (int64_t)gridDim.x * kRedThreads;
  for (int64_t i = (int64_t)blockIdx.x * kRedThreads + threadIdx.x; i < n; i += stride) {
    const T rn = rin[i] - alpha * q[i];
    rout[i] = rn;
    s += (double)rn * (double)rn;
  }
  if (!partial) return;   // no norm wanted (uniform over the grid)
  const double t = block_sum(s, sh);
  if (threadIdx.x == 0) partial[rhs * 1024 + blockIdx.x] = t;
}

template <typename T>
void pupdate(int64_t n, int nrhs, const T* z, T* p, T* x, const double* scal, int first, hipStream_t st) {
  const int64_t tot = n * nrhs;
  hipLaunchKernelGGL((pupdate_kernel<T>), dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, nrhs, z, p, x,
                     scal, first);
}

template <typename T>
void xupdate(int64_t n, int nrhs, T* x, const T* p, const double* scal, hipStream_t st) {
  const int64_t tot = n * nrhs;
  hipLaunchKernelGGL((xupdate_kernel<T>), dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, nrhs, x, p, scal);
}

template <typename T>
void cg_update(int64_t n, int nrhs, const T* rin, T* rout, const T* q, const double* scal, double* partial,
               int nblocks, hipStream_t st) {
  hipLaunchKernelGGL((cg_update_kernel<T>), dim3(nblocks, nrhs), dim3(kRedThreads), 0, st, n, rin, rout, q, scal,
                     partial);
}
template void pupdate<double>(int64_t, int, const double*, double*, double*, const double*, int, hipStream_t);
template void pupdate<float>(int64_t, int, const float*, float*, float*, const double*, int, hipStream_t);
template void xupdate<double>(int64_t, int, double*, const double*, const double*, hipStream_t);
template void xupdate<float>(int64_t, int, float*, const float*, const double*, hipStream_t);
template void cg_update<double>(int64_t, int, const double*, double*, const double*, const double*, double*, int,
                                hipStream_t);
template void cg_update<float>(int64_t, int, const float*, float*, const float*, const double*, double*, int,
                               hipStream_t);

// y = x (with optional conversion) / y += x
template <typename TI, typename TO>
__global__ void convert_kernel(int64_t n, const TI* __restrict__ x, TO* __restrict__ y, int accumulate) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  y[i] = accumulate ? (TO)(y[i] + (TO)x[i]) : (TO)x[i];
}

template <typename TI, typename TO>
void convert(int64_t n, const TI* x, TO* y, int accumulate, hipStream_t st) {
  hipLaunchKernelGGL((convert_kernel<TI, TO>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, x, y,
                     accumulate);
}
template void convert<double, double>(int64_t, const double*, double*, int, hipStream_t);
template void convert<double, float>(int64_t, const double*, float*, int, hipStream_t);
template void convert<float, double>(int64_t, const float*, double*, int, hipStream_t);
template void convert<float, float>(int64_t, const float*, float*, int, hipStream_t);

__global__ void mask_mul_kernel(int64_t n, double* __restrict__ y, const double* __restrict__ m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] *= m[i];
}
void mask_mul(int64_t n, double* y, const double* m, hipStream_t st) {
  hipLaunchKernelGGL(mask_mul_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, y, m);
}

__global__ void fill_kernel(int64_t n, double* __restrict__ y, double v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = v;
}
void fill(int64_t n, double* y, double v, hipStream_t st) {
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, y, v);
}
__global__ void fillf_kernel(int64_t n, float* __restrict__ y, float v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = v;
}
void fill(int64_t n, float* y, float v, hipStream_t st) {
  hipLaunchKernelGGL(fillf_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, y, v);
}

}  // namespace dgfas
