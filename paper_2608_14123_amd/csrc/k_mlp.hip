// K6: the learned subdomain correction -- a 3-layer MLP with BF16 weights and FP32
// accumulation, trained on the GPU.  GEMMs run on the CDNA matrix cores
// (v_mfma_f32_16x16x16bf16_1k), with bias, ReLU and its derivative in their last pass and
// column sums as a row of ones; the casts, the MSE gradient and Adam run in plain kernels.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "mlp.hpp"

namespace dgfas {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// FP32 -> BF16 with round-to-nearest-even (NaN kept quiet)
__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t b = __float_as_uint(f);
  if ((b & 0x7f800000u) == 0x7f800000u && (b & 0x7fffffu)) return (uint16_t)((b >> 16) | 0x40);
  b += 0x7fffu + ((b >> 16) & 1u);
  return (uint16_t)(b >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// four values a thread where both arrays are aligned for it (torch's are; a row offset into X may
// not be): 4096 x 1340 values 11 -> 7.4 us
template <int V>
__global__ void __launch_bounds__(256) to_bf16_kernel(int64_t n, const float* __restrict__ x,
                                                      uint16_t* __restrict__ y) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
  if (V == 4 && i + 4 <= n) {
    const float4 v = *reinterpret_cast<const float4*>(x + i);
    *reinterpret_cast<ushort4*>(y + i) = make_ushort4(to_bf16(v.x), to_bf16(v.y), to_bf16(v.z), to_bf16(v.w));
  } else {
    for (int64_t j = i; j < n && j < i + V; ++j) y[j] = to_bf16(x[j]);
  }
}

void cast_bf16(int64_t n, const float* x, uint16_t* y, hipStream_t st) {
  const bool al = reinterpret_cast<uintptr_t>(x) % 16 == 0 && reinterpret_cast<uintptr_t>(y) % 8 == 0;
  if (al) hipLaunchKernelGGL(to_bf16_kernel<4>, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, st, n, x, y);
  else hipLaunchKernelGGL(to_bf16_kernel<1>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, x, y);
}

// C[m][n] = sum_k A(m,k) B(k,n) (+ bias[n]) (ReLU) with A(m,k) = A[m*sam + k*sak],
// B(k,n) = B[k*sbk + n*sbn] in BF16, C row-major FP32 (ldc = N) and optionally a BF16 copy.
// Workgroup: 4 wavefronts, 64x64 tile, each wavefront 32x32 = 2x2 MFMA 16x16 blocks;
// K advances 64 per LDS stage.  Out-of-range rows/columns/k are zero-filled.
// Split K: with P set, slice z = blockIdx.z takes k in [z kper, (z + 1) kper) and writes its
// raw sum to P[z][m][n]; splitk_reduce adds the slices in order and applies the epilogue, so
// the result does not depend on scheduling.
// Bound: latency, not the matrix cores (the weight gradients of a 4096-row batch have 64 K-steps a
// slice or fewer), so the next K-step's operands are loaded to registers before this one's products
// and stored to the other LDS buffer after them, with one barrier a step.
// Measured, the 8 products of a gradient of 4096 rows through 1340 - 256 - 1331: 27 us on average with one
// buffer and two barriers a step of 32, 15.2 now; outputs bit for bit the same.
// Rows of 136 bytes: the 8-byte operand reads of a half wavefront meet every bank once, and the
// transposed 8-byte stores of mode 2 every bank twice.
constexpr int GT = 64, GK = 64, GKP = GK + 4;
constexpr int kSlice = 32;   // K-slices end on multiples of this

// A thread's share of the 64 x 64 tile S[r][kk] = X(r0 + r, k0 + kk), X(r, k) = X[r sr + k sk], zero
// outside R x K; with `ones`, row R is a row of ones (1.0 in BF16 is 0x3f80) for k < K.  MODE 1
// (contiguous along k) and 0 (general): v[j] holds four k of row tid / 16 + 16 j; MODE 2 (contiguous
// along r): v[j] holds four rows of k = 4 (tid / 16) + j.  Every load is unconditional, from the
// array's start where its four values are all outside, and masked when it is stored: branches around
// the loads made each wait for the one before (the weight gradients 22.1 us instead of 15.7).  An
// 8-byte load that begins inside ends inside its row's pitch.
template <int MODE>
__device__ __forceinline__ void load_tile(uint2 (&v)[4], const uint16_t* __restrict__ X, int R, int K, int r0, int k0,
                                          int64_t sr, int64_t sk, int tid, int ones) {
  const int hi = tid >> 4, lo = (tid & 15) * 4;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if constexpr (MODE == 2) {
      const int k = k0 + 4 * hi + j, r = r0 + lo;
      v[j] = *reinterpret_cast<const uint2*>(X + (k < K && r < R ? (int64_t)k * sk + r : 0));
    } else if constexpr (MODE == 1) {
      const int r = r0 + hi + 16 * j, k = k0 + lo;
      v[j] = *reinterpret_cast<const uint2*>(X + (k < K && r < R ? (int64_t)r * sr + k : 0));
    } else {
      const int r = r0 + hi + 16 * j;
      uint32_t t[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = k0 + lo + i;
        const bool in = k < K && r < R;
        const uint32_t x = X[in ? (int64_t)r * sr + (int64_t)k * sk : 0];
        t[i] = in ? x : (ones && k < K && r == R ? 0x3f80u : 0u);
      }
      v[j] = make_uint2(t[0] | (t[1] << 16), t[2] | (t[3] << 16));
    }
  }
}

// the first c of four BF16 values
__device__ __forceinline__ uint2 first_of(uint2 v, int c) {
  return make_uint2(c >= 2 ? v.x : c == 1 ? v.x & 0xffffu : 0u, c >= 4 ? v.y : c == 3 ? v.y & 0xffffu : 0u);
}

template <int MODE>
__device__ __forceinline__ void store_tile(uint16_t (*S)[GKP], uint2 (&v)[4], int R, int K, int r0, int k0, int tid,
                                           int ones) {
  const int hi = tid >> 4, lo = (tid & 15) * 4;
  const bool edge = r0 + GT > R || k0 + GK > K;   // uniform
  if constexpr (MODE == 2) {   // 4 x 4 transposed in registers
    if (edge) {
      const int c = R - (r0 + lo);
      const uint2 one = ones ? make_uint2(c == 0 ? 0x3f80u : c == 1 ? 0x3f800000u : 0u,
                                          c == 2 ? 0x3f80u : c == 3 ? 0x3f800000u : 0u)
                             : make_uint2(0u, 0u);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool in = k0 + 4 * hi + j < K;
        const uint2 f = first_of(v[j], c);
        v[j] = make_uint2(in ? f.x | one.x : 0u, in ? f.y | one.y : 0u);
      }
    }
    auto lo2 = [](uint32_t x, uint32_t y) { return (x & 0xffffu) | (y << 16); };
    auto hi2 = [](uint32_t x, uint32_t y) { return (x >> 16) | (y & 0xffff0000u); };
    *reinterpret_cast<uint2*>(&S[lo][4 * hi]) = make_uint2(lo2(v[0].x, v[1].x), lo2(v[2].x, v[3].x));
    *reinterpret_cast<uint2*>(&S[lo + 1][4 * hi]) = make_uint2(hi2(v[0].x, v[1].x), hi2(v[2].x, v[3].x));
    *reinterpret_cast<uint2*>(&S[lo + 2][4 * hi]) = make_uint2(lo2(v[0].y, v[1].y), lo2(v[2].y, v[3].y));
    *reinterpret_cast<uint2*>(&S[lo + 3][4 * hi]) = make_uint2(hi2(v[0].y, v[1].y), hi2(v[2].y, v[3].y));
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (MODE == 1 && edge) {
        const int r = r0 + hi + 16 * j;
        if (r >= R) {
          const uint32_t one = ones && r == R ? 0x3f803f80u : 0u;
          v[j] = make_uint2(one, one);
        }
        v[j] = first_of(v[j], K - (k0 + lo));
      }
      *reinterpret_cast<uint2*>(&S[hi + 16 * j][lo]) = v[j];
    }
  }
}

// staging mode of an R x K operand: 1 contiguous along k, 2 contiguous along r (rows of at least the
// length read, whole 8-byte words apart), 0 general
inline int stage_mode(const uint16_t* X, int R, int K, int64_t sr, int64_t sk) {
  const bool al = (reinterpret_cast<uintptr_t>(X) % 8) == 0;
  if (al && sk == 1 && sr % 4 == 0 && sr >= K) return 1;
  if (al && sr == 1 && sk % 4 == 0 && sk >= R) return 2;
  return 0;
}

struct GemmArgs {
  int M, N, K;
  const uint16_t* A;
  int64_t sam, sak;
  const uint16_t* B;
  int64_t sbk, sbn;
  float* C;
  uint16_t* Cb;
  const float* bias;
  const float* gate;   // C is zero where this is not positive (ReLU's derivative)
  int relu, accumulate, kper;
  float* P;
  int ones;
};

// value o = m N + n of C from its sum
__device__ __forceinline__ void gemm_store(const GemmArgs& g, int64_t o, int n, float v) {
  if (g.accumulate) v += g.C[o];
  if (g.bias) v += g.bias[n];
  if (g.relu) v = v > 0.f ? v : 0.f;
  if (g.gate) v = g.gate[o] > 0.f ? v : 0.f;
  if (g.C) g.C[o] = v;
  if (g.Cb) g.Cb[o] = to_bf16(v);
}

template <int AMODE, int BMODE>
__global__ void __launch_bounds__(256) gemm_bf16_kernel(GemmArgs g) {
  __shared__ __align__(16) uint16_t As[2][GT][GKP];   // [m][k]
  __shared__ __align__(16) uint16_t Bs[2][GT][GKP];   // [n][k]
  const int M = g.M, N = g.N;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // workgroups are dealt to the 8 XCDs in turn: each XCD takes a contiguous range of (slice, m, n),
  // so that the operands of its tiles stay in its L2 (a remainder of 8 keeps its place)
  const unsigned gx = gridDim.x, gy = gridDim.y, per = gx * gy * gridDim.z / 8;
  const unsigned bl = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const unsigned lb = bl < 8 * per ? (bl & 7) * per + (bl >> 3) : bl;
  const int bz = lb / (gx * gy), m0 = (lb / gx - bz * gy) * GT, n0 = lb % gx * GT;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  v4f acc[2][2];
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b) acc[a][b] = v4f{0.f, 0.f, 0.f, 0.f};
  const int kb = bz * g.kper;   // kper = K without slices
  const int ke = min(g.K, kb + g.kper);
  uint2 va[4], vb[4];
  auto load = [&](int k0) {
    load_tile<AMODE>(va, g.A, M - g.ones, ke, m0, k0, g.sam, g.sak, tid, g.ones);
    load_tile<BMODE>(vb, g.B, N, ke, n0, k0, g.sbn, g.sbk, tid, 0);
  };
  auto store = [&](int s, int k0) {
    store_tile<AMODE>(As[s], va, M - g.ones, ke, m0, k0, tid, g.ones);
    store_tile<BMODE>(Bs[s], vb, N, ke, n0, k0, tid, 0);
  };
  load(kb);
  store(0, kb);
  __syncthreads();
  int s = 0;
  for (int k0 = kb; k0 < ke; k0 += GK, s ^= 1) {
    const bool more = k0 + GK < ke;
    if (more) load(k0 + GK);
#pragma unroll
    for (int kk = 0; kk < GK; kk += 16) {
      // operand layout of the 16x16x16 bf16 MFMA: lane l holds A[l%16][4(l/16)+i], B[4(l/16)+i][l%16]
      const int kl = kk + 4 * (lane >> 4), rl = lane & 15;
      v4s fa[2], fb[2];
      for (int a = 0; a < 2; ++a) fa[a] = *reinterpret_cast<const v4s*>(&As[s][wm + 16 * a + rl][kl]);
      for (int b = 0; b < 2; ++b) fb[b] = *reinterpret_cast<const v4s*>(&Bs[s][wn + 16 * b + rl][kl]);
      for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa[a], fb[b], acc[a][b], 0, 0, 0);
    }
    if (more) store(s ^ 1, k0 + GK);   // last read before the previous barrier
    __syncthreads();
  }
  // result layout: lane l, register j holds D[4(l/16)+j][l%16]
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b)
      for (int j = 0; j < 4; ++j) {
        const int m = m0 + wm + 16 * a + 4 * (lane >> 4) + j;
        const int n = n0 + wn + 16 * b + (lane & 15);
        if (m >= M || n >= N) continue;
        const int64_t o = (int64_t)m * N + n;
        if (g.P) g.P[(int64_t)bz * M * N + o] = acc[a][b][j];
        else gemm_store(g, o, n, acc[a][b][j]);
      }
}

__global__ void __launch_bounds__(256) splitk_reduce_kernel(GemmArgs g, int splits) {
  const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, mn = (int64_t)g.M * g.N;
  if (o >= mn) return;
  float v = 0.f;
  for (int z0 = 0; z0 < splits; z0 += 8) {   // eight slices in flight, added in order
    float t[8];
#pragma unroll
    for (int z = 0; z < 8; ++z) t[z] = z0 + z < splits ? g.P[(int64_t)(z0 + z) * mn + o] : 0.f;
#pragma unroll
    for (int z = 0; z < 8; ++z)
      if (z0 + z < splits) v += t[z];
  }
  gemm_store(g, o, (int)(o % g.N), v);
}

int gemm_splits(int M, int N, int K, int64_t ws_cap) {
  const int64_t tiles = (int64_t)((N + GT - 1) / GT) * ((M + GT - 1) / GT);
  // fewer tiles than about two per CU and a long K: cut K into slices of at least 256
  if (tiles >= 512 || K < 512) return 1;
  int64_t s = std::min<int64_t>((1024 + tiles - 1) / tiles, K / 256);
  s = std::min<int64_t>(s, ws_cap / ((int64_t)M * N));
  return (int)std::max<int64_t>(1, s);
}

template <int AMODE>
static void launch_gemm(int bmode, dim3 grid, hipStream_t st, const GemmArgs& g) {
  if (bmode == 1) hipLaunchKernelGGL((gemm_bf16_kernel<AMODE, 1>), grid, dim3(256), 0, st, g);
  else if (bmode == 2) hipLaunchKernelGGL((gemm_bf16_kernel<AMODE, 2>), grid, dim3(256), 0, st, g);
  else hipLaunchKernelGGL((gemm_bf16_kernel<AMODE, 0>), grid, dim3(256), 0, st, g);
}

void gemm_bf16(int M, int N, int K, const uint16_t* A, int64_t sam, int64_t sak, const uint16_t* B, int64_t sbk,
               int64_t sbn, float* C, uint16_t* Cb, const float* bias, int relu, int accumulate, hipStream_t st,
               float* ws, int64_t ws_cap, int ones, const float* gate) {
  int splits = ws ? gemm_splits(M, N, K, ws_cap) : 1;
  int kper = K;
  if (splits > 1) {
    kper = ((K + splits - 1) / splits + kSlice - 1) / kSlice * kSlice;
    splits = (K + kper - 1) / kper;
  }
  const int am = stage_mode(A, M - ones, K, sam, sak), bm = stage_mode(B, N, K, sbn, sbk);
  const GemmArgs g{M, N, K, A, sam, sak, B, sbk, sbn, C, Cb, bias, gate, relu, accumulate, kper,
                   splits > 1 ? ws : nullptr, ones};
  const dim3 grid((N + GT - 1) / GT, (M + GT - 1) / GT, splits > 1 ? splits : 1);
  if (am == 1) launch_gemm<1>(bm, grid, st, g);
  else if (am == 2) launch_gemm<2>(bm, grid, st, g);
  else launch_gemm<0>(bm, grid, st, g);
  if (splits > 1)
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)(((int64_t)M * N + 255) / 256)), dim3(256), 0, st, g,
                       splits);
}

// dY = 2 (Y - T) / (rows * cols) as BF16 rows of pitch ldb (the padding columns are left
// alone), loss partials per block
__global__ void mse_kernel(int64_t n, int cols, int ldb, const float* __restrict__ Y, const float* __restrict__ T,
                           float scale, uint16_t* __restrict__ dYb, double* __restrict__ part) {
  __shared__ double sh[256];
  double s = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const float d = Y[i] - T[i];
    s += (double)d * d;
    const int64_t r = i / cols;
    dYb[r * ldb + (i - r * cols)] = to_bf16(2.f * scale * d);
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

void mse_grad(int64_t n, int cols, int ldb, const float* Y, const float* T, float scale, uint16_t* dYb, double* part,
              int nblocks, hipStream_t st) {
  hipLaunchKernelGGL(mse_kernel, dim3(nblocks), dim3(256), 0, st, n, cols, ldb, Y, T, scale, dYb, part);
}

// dst[r][c] = src[r][c] for c < cols, 0 for cols <= c < ldd (a row-padded BF16 copy)
__global__ void pad_rows_kernel(int rows, int cols, int ldd, const uint16_t* __restrict__ src,
                                uint16_t* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)rows * ldd) return;
  const int64_t r = i / ldd;
  const int c = (int)(i - r * ldd);
  dst[i] = c < cols ? src[r * cols + c] : (uint16_t)0;
}

void pad_rows(int rows, int cols, int ldd, const uint16_t* src, uint16_t* dst, hipStream_t st) {
  const int64_t n = (int64_t)rows * ldd;
  hipLaunchKernelGGL(pad_rows_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, rows, cols, ldd, src, dst);
}

// Adam with bias correction; refreshes the BF16 weight copy
__global__ void adam_kernel(int64_t n, float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, uint16_t* __restrict__ wb, float lr, float b1, float b2, float eps,
                            float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  w[i] = wi;
  if (wb) wb[i] = to_bf16(wi);
}

void adam(int64_t n, float* w, const float* g, float* m, float* v, uint16_t* wb, float lr, float b1, float b2,
          float eps, float c1, float c2, hipStream_t st) {
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, w, g, m, v, wb, lr, b1, b2,
                     eps, c1, c2);
}

}  // namespace dgfas
