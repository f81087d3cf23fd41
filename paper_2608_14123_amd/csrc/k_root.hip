// The root solve of a small hierarchy in one launch: Schwarz-preconditioned inexact CG (Alg. 6) on a
// p = 1 level of at most 64 elements, one workgroup per right-hand side.
//
// On such a level every kernel of the general solve is far below one wave of the chip, and an
// iteration is a chain of eight launches whose 2 to 5 us each are launch and drain latency: the
// 4^3 root of the unit-cube p = 4 hierarchy (about 20 iterations to 1e-12, seven cycles a solve) took
// nine tenths of the solve.  Here a thread keeps its node's vector entries from iteration to iteration, what
// other threads read goes through LDS, and an iteration is five workgroup barriers: 8 us, and the whole
// solve went from 7.4 to 2.6 ms, of which these launches are still nearly half.  1024 threads leave each 128
// registers; 54 values that it holds over the loop (indices, destinations, weights) are in scratch memory.
// The steps are those of the general kernels: gather, fast-diagonalisation solve and weighted
// scatter per subdomain (sixteen threads, one xi_3 column each; the exchanges stay inside a
// wavefront), the inbox sum per node, the SIPG operator from the node's own element and its three face
// neighbours, and the scalars of the finish kernel.
#include "device.hpp"
#include "kernels.hpp"

namespace dgfas {

namespace {
constexpr int kE = kSmallRootElems, kNodes = 8 * kE, kNS = 4;
constexpr int kRow = kNS + 1, kTile = kNS * kNS * kRow, kSP = kNS * kNS + 2;
constexpr int kThreads = 16 * kE;   // one per subdomain column; the first 8 E own the nodes

struct RootSmem {
  double v[kNodes];                 // r for the gathers, p for the operator
  double z[kNodes + kE * 56];       // the subdomains' own parts, then the overlap inboxes, whose
                                    // regions that nobody writes stay zero
  double G[6][kNodes];              // the metric
  double gn[9][kNodes];             // per axis the face neighbour's metric row
  // pitches that put the lanes of half a wavefront on distinct banks, along every direction and over
  // the two subdomains (or variants) they belong to
  double tile[kE][kTile];
  alignas(16) double S[16][kSP];    // S[v][q][c], all side variants
  double lam[16][kNS], W[16][kNS];
  double red[4][2][kThreads / 64];
  int off[27];                      // inbox region offsets
};
static_assert(Regions<2, 1>{}.size == 56, "inbox slots of an element");

// LDS written by one lane of a wavefront is read by another after this
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// sums of a and b over the workgroup, in every thread; slot: red[slot] is not read by anybody who
// has not yet passed the previous barrier
__device__ __forceinline__ void sum2(RootSmem& sm, int slot, double& a, double& b) {
  const int tid = threadIdx.x, nw = blockDim.x >> 6;
  a = wave_sum(a);
  b = wave_sum(b);
  if ((tid & 63) == 0) {
    sm.red[slot][0][tid >> 6] = a;
    sm.red[slot][1][tid >> 6] = b;
  }
  __syncthreads();
  // lanes 0..15 take the wavefronts' sums of a, lanes 32..47 those of b
  const int l = tid & 63, w = l & 31;
  double v = w < nw ? sm.red[slot][l >> 5][w] : 0.0;
  v = row_sum(v);
  a = lane_value(v, 15);
  b = lane_value(v, 47);
}

// side variant v = left * 4 + right, an interior side (code 0) has one overlap layer:
// (delta + 1) * 64 + local node of position q, or -1
__device__ __forceinline__ int map2(int v, int q) {
  const int d = q - ((v >> 2) == 0 ? 1 : 0);
  if (d < 0) return 1;
  if (d < 2) return 64 + d;
  return d == 2 && (v & 3) == 0 ? 128 : -1;
}
}  // namespace

__global__ void __launch_bounds__(kThreads) small_root_kernel(SmallRootArgs a) {
  __shared__ RootSmem sm;
  const int tid = threadIdx.x, rhs = blockIdx.x, E = a.E, nd = 8 * E;
  constexpr Regions<2, 1> R{};
  const bool node = tid < nd;
  const int e = node ? tid >> 3 : 0, n = tid & 7;
  const int64_t at = (int64_t)rhs * nd + (node ? tid : 0);

  // tables, and an empty inbox
  for (int t = tid; t < 16 * kNS * kNS; t += blockDim.x) sm.S[t / (kNS * kNS)][t % (kNS * kNS)] = a.S[t];
  for (int t = tid; t < 16 * kNS; t += blockDim.x) {
    sm.lam[t / kNS][t % kNS] = a.lam[t];
    sm.W[t / kNS][t % kNS] = a.W[t];
  }
  for (int t = tid; t < kNodes + 56 * E; t += blockDim.x) sm.z[t] = 0.0;
  if (tid < 27) sm.off[tid] = R.off[tid];
  __syncthreads();

  // the node's metric, and per axis its face: neighbour, penalty, the neighbour's metric row
  double wj = 0, pen[3];
  int nb[3], bc[3];
#pragma unroll
  for (int c = 0; c < 6; ++c)
    if (node) sm.G[c][tid] = a.G[(int64_t)c * nd + tid];
  if (a.WJ) wj = a.kappa * a.WJ[node ? tid : 0];
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    const int bit = (n >> ax) & 1, phi = 2 * ax + bit;
    // face layouts (first, second): (k, j), (k, i), (j, i)
    const int f = ax == 0 ? (n >> 2 & 1) * 2 + (n >> 1 & 1) : (ax == 1 ? (n >> 2 & 1) * 2 + (n & 1) : (n >> 1 & 1) * 2 + (n & 1));
    nb[ax] = a.nbr[e * 6 + phi];
    bc[ax] = a.bc[e * 6 + phi];
    pen[ax] = a.pen[(e * 6 + phi) * 4 + f];
    const int on = (nb[ax] >= 0 ? nb[ax] : e) * 8 + (n ^ (1 << ax));   // its node at the shared face
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (node) sm.gn[3 * ax + c][tid] = a.G[(int64_t)sym_index(ax, c) * nd + on];
  }
  // D[i][m] without an indexed register array
  const double D00 = a.D[0], D01 = a.D[1], D10 = a.D[2], D11 = a.D[3];
  auto D0 = [&](int i) { return i ? D10 : D00; };
  auto D1 = [&](int i) { return i ? D11 : D01; };

  // the thread's column (s1, s2) of subdomain es: gather nodes, destinations and weights by s3
  const int es = min(tid >> 4, E - 1), c = tid & 15, c1 = c & 3, c2 = c >> 2;
  const bool col = (tid >> 4) < E;
  const int v0 = a.var[es * 3], v1 = a.var[es * 3 + 1], v2 = a.var[es * 3 + 2];
  int map[kNS];   // index into v, and index into z in the upper half; -1: nothing there
  const double w12 = a.W[v0 * kNS + c1] * a.W[v1 * kNS + c2];
  {
    const int m1 = map2(v0, c1), m2 = map2(v1, c2);
#pragma unroll
    for (int s3 = 0; s3 < kNS; ++s3) {
      const int m3 = map2(v2, s3);
      map[s3] = -1;
      if (!col || m1 < 0 || m2 < 0 || m3 < 0) continue;
      const int q = a.nb27[es * 27 + (m3 >> 6) * 9 + (m2 >> 6) * 3 + (m1 >> 6)];
      if (q < 0) continue;
      const int l1 = m1 & 63, l2 = m2 & 63, l3 = m3 & 63;
      const int d1 = (m1 >> 6) - 1, d2 = (m2 >> 6) - 1, d3 = (m3 >> 6) - 1;
      const int src = q * 8 + (l3 * 2 + l2) * 2 + l1;
      int dst = src;
      if (d1 != 0 || d2 != 0 || d3 != 0) {
        const int r = (1 - d3) * 9 + (1 - d2) * 3 + (1 - d1);   // direction from the receiver back to es
        const int k1 = d1 < 0 ? l1 - 1 : l1, k2 = d2 < 0 ? l2 - 1 : l2, k3 = d3 < 0 ? l3 - 1 : l3;
        const int x1 = d1 ? 1 : 2, x2 = d2 ? 1 : 2;
        dst = kNodes + q * 56 + sm.off[r] + (k3 * x2 + k2) * x1 + k1;
      }
      map[s3] = src | dst << 16;
    }
  }
  // the node's seven inbox slots in the order of the overlap add
  int slot[7];
  {
    const int l[3] = {n & 1, n >> 1 & 1, n >> 2 & 1};
#pragma unroll
    for (int bits = 1; bits < 8; ++bits) {
      int dd[3], k[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        dd[d] = (bits >> d & 1) ? (l[d] ? 1 : -1) : 0;
        k[d] = dd[d] > 0 ? l[d] - 1 : l[d];
      }
      const int r = (dd[2] + 1) * 9 + (dd[1] + 1) * 3 + dd[0] + 1;
      const int x1 = dd[0] ? 1 : 2, x2 = dd[1] ? 1 : 2;
      slot[bits - 1] = kNodes + e * 56 + sm.off[r] + (k[2] * x2 + k[1]) * x1 + k[0];
    }
  }
  double g0, g1, g2, g3;
  g0 = a.gco[es * 4];
  g1 = a.gco[es * 4 + 1];
  g2 = a.gco[es * 4 + 2];
  g3 = a.gco[es * 4 + 3];
  double* const tile = sm.tile[es];
  __syncthreads();

  // out = S^T in (tr) or S in for the 4 x 4 eigenvectors of variant v
  auto apply = [&](int v, bool tr, double (&t)[kNS]) {
    double S[kNS][kNS], o[kNS] = {0, 0, 0, 0};
    asm volatile("" ::: "memory");   // read anew: kept over the iterations, the tables would spill
#pragma unroll
    for (int q = 0; q < kNS; ++q)
#pragma unroll
      for (int k = 0; k < kNS; ++k) S[q][k] = sm.S[v][q * kNS + k];
#pragma unroll
    for (int q = 0; q < kNS; ++q)
#pragma unroll
      for (int k = 0; k < kNS; ++k) o[k] += (tr ? S[q][k] : S[k][q]) * t[q];
#pragma unroll
    for (int k = 0; k < kNS; ++k) t[k] = o[k];
  };
  auto load = [&](int at, int stride, double (&t)[kNS]) {
#pragma unroll
    for (int q = 0; q < kNS; ++q) t[q] = tile[at + q * stride];
  };
  auto store = [&](int at, int stride, const double (&t)[kNS]) {
#pragma unroll
    for (int q = 0; q < kNS; ++q) tile[at + q * stride] = t[q];
    wave_sync();
  };
  // z = B v: the node's preconditioned value
  auto schwarz = [&]() -> double {
    if (col) {
      const int z0 = c2 * kRow + c1, sz = kNS * kRow;   // column (s1 = c1, s2 = c2) along xi_3
      const int y0 = c2 * kNS * kRow + c1;              // line (s1 = c1, s3 = c2) along xi_2
      const int x0 = c * kRow;                          // line (s2 = c1, s3 = c2) along xi_1
      double t[kNS];
#pragma unroll
      for (int s = 0; s < kNS; ++s) t[s] = map[s] >= 0 ? sm.v[map[s] & 0xffff] : 0.0;
      apply(v2, true, t);
      store(z0, sz, t);
      load(y0, kRow, t);
      apply(v1, true, t);
      store(y0, kRow, t);
      load(x0, 1, t);
      apply(v0, true, t);
      const double base = g0 + g2 * sm.lam[v1][c1] + g3 * sm.lam[v2][c2];
#pragma unroll
      for (int k = 0; k < kNS; ++k) t[k] /= base + g1 * sm.lam[v0][k];
      apply(v0, false, t);
      store(x0, 1, t);
      load(y0, kRow, t);
      apply(v1, false, t);
      store(y0, kRow, t);
      load(z0, sz, t);
      apply(v2, false, t);
#pragma unroll
      for (int k = 0; k < kNS; ++k)
        if (map[k] >= 0) sm.z[map[k] >> 16] = w12 * sm.W[v2][k] * t[k];
    }
    __syncthreads();
    double z = 0;
    if (node) {
      double acc = 0;
#pragma unroll
      for (int k = 0; k < 7; ++k) acc += sm.z[slot[k]];
      z = sm.z[tid] + acc;
    }
    return z;
  };

  // (A u) at the node, u in sm.v
  auto op = [&](double u) -> double {
    double F[3], G[6], row = 0;
    asm volatile("" ::: "memory");   // as in apply
    const int b8 = e * 8;
    {
      double d[3];
#pragma unroll
      for (int ax = 0; ax < 3; ++ax) {
        const int i = n >> ax & 1, m = 1 << ax;
        d[ax] = D0(i) * sm.v[b8 + (n & ~m)] + D1(i) * sm.v[b8 + (n | m)];
      }
#pragma unroll
      for (int c = 0; c < 6; ++c) G[c] = sm.G[c][tid & (kNodes - 1)];
      F[0] = G[0] * d[0] + G[1] * d[1] + G[2] * d[2];
      F[1] = G[1] * d[0] + G[3] * d[1] + G[4] * d[2];
      F[2] = G[2] * d[0] + G[4] * d[1] + G[5] * d[2];
    }
    double sg[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      const int i = n >> ax & 1, m = 1 << ax;
      const double w = i ? a.inv_wend : -a.inv_wend;
      sg[ax] = 0;
      if (nb[ax] >= 0) {
        const int o8 = nb[ax] * 8, on = n ^ m;
        const double tr = sm.v[o8 + on], far = sm.v[o8 + n];   // its face node, and the line's other end
        double du[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          const int mt = 1 << t, it = n >> t & 1;
          if (t == ax) du[t] = i ? D00 * tr + D01 * far : D10 * far + D11 * tr;
          else du[t] = D0(it) * sm.v[o8 + (on & ~mt)] + D1(it) * sm.v[o8 + (on | mt)];
        }
        const double fl = sm.gn[3 * ax][tid & (kNodes - 1)] * du[0] + sm.gn[3 * ax + 1][tid & (kNodes - 1)] * du[1] +
                          sm.gn[3 * ax + 2][tid & (kNodes - 1)] * du[2];
        const double jmp = u - tr;
        row += pen[ax] * jmp - 0.5 * w * (F[ax] + fl);
        sg[ax] = -0.5 * jmp * w;
      } else if (bc[ax] == 1) {
        row += pen[ax] * u - w * F[ax];
        sg[ax] = -u * w;
      }
    }
#pragma unroll
    for (int ax = 0; ax < 3; ++ax)
#pragma unroll
      for (int t = 0; t < 3; ++t) F[t] += sg[ax] * G[sym_index(ax, t)];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      const int i = n >> ax & 1;
      row += (i ? D11 : D00) * F[ax] + (i ? D01 : D10) * __shfl_xor(F[ax], 1 << ax);
    }
    return row + wj * u;
  };
  // v minus its mean over the level, for the semidefinite operator (slot: see sum2); called by every
  // thread of the workgroup, as it meets at a barrier
  auto project = [&](double v, int s) -> double {
    double m = node ? v : 0.0, o = 0;
    sum2(sm, s, m, o);
    return node ? v - m / (double)nd : 0.0;
  };

  double x = a.u[at];
  if (node) sm.v[tid] = x;
  __syncthreads();
  double r = a.g[at] - op(x);
  if (!node) r = 0;
  if (a.project) r = project(r, 3);
  double rr = r * r, o = 0;
  sum2(sm, 0, rr, o);
  const double stop = a.rtol > 0 ? a.rtol * sqrt(rr) : 0.0;
  int it = 0;
  bool bad = a.rtol > 0 && isnan(rr), conv = false;   // with a stop of NaN there is no iteration to find it
  double gamma = 0, p = 0, r0 = 0;
  if (!(a.rtol > 0) || stop > 0) {
    if (node) sm.v[tid] = r;
    __syncthreads();
    for (int i = 1; i <= a.n; ++i) {
      double z = schwarz();
      if (a.project) z = project(z, 3);
      double zr = z * r, zd = i > 1 ? z * (r - r0) : 0.0;
      sum2(sm, 1, zr, zd);
      double beta = 0;
      if (i > 1) {
        beta = zd / gamma;
        if (!isfinite(beta)) {
          beta = 0;
          bad = true;
        }
      }
      gamma = zr;
      p = i > 1 ? beta * p + z : z;
      if (node) sm.v[tid] = p;
      __syncthreads();
      const double q = node ? op(p) : 0.0;
      double pq = p * q;
      o = 0;
      sum2(sm, 2, pq, o);
      double alpha = pq != 0.0 ? gamma / pq : 0.0;
      if (pq < 0.0 || !isfinite(alpha)) {
        bad = true;
        alpha = 0;
      }
      x += alpha * p;
      r0 = r;
      r -= alpha * q;
      if (node) sm.v[tid] = r;
      it = i;
      if (a.rtol > 0) {
        rr = r * r;
        o = 0;
        sum2(sm, 0, rr, o);
        if (!isfinite(rr)) bad = true;
        conv = sqrt(rr) <= stop;
        // a breakdown ends the solve where the general path looks for it
        if (conv || (bad && (i % a.check == 0 || i == a.n))) break;
      } else {
        __syncthreads();
      }
    }
  }
  if (node) a.u[at] = x;
  if (tid == 0) {
    double* sc = a.scal + rhs * 8;
    sc[4] = bad ? 1.0 : 0.0;
    sc[5] = it;
    sc[7] = conv ? 1.0 : 0.0;
  }
}

void small_root(const SmallRootArgs& a, int nrhs, hipStream_t st) {
  hipLaunchKernelGGL(small_root_kernel, dim3(nrhs), dim3((16 * a.E + 63) / 64 * 64), 0, st, a);
}

}  // namespace dgfas
