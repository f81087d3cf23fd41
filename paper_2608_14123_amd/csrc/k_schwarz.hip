// K2: weighted overlapping Schwarz application z = sum_e R_s^T W^e (A~_s^e)^-1 R_s r
// (Sec. 4.3.1, eq. schwarz:correction) with fast-diagonalisation subdomain solves
//   (A~_s)^-1 = (S3 x S2 x S1) D^-1 (S3^T x S2^T x S1^T),
//   D = g0 + g1 lam1_i + g2 lam2_j + g3 lam3_k.
//
// schwarz_solve: the NS^3 tile (NS = N + 2M, smaller variants zero-padded) is gathered from the
// element and its 26 neighbours, contracted along xi_3, xi_2, xi_1, divided, and contracted back.  Three forms:
// one workgroup per subdomain and a thread per tile line (schwarz_tile, n >= 4), several small subdomains
// to a workgroup with a thread per line (schwarz_pack_tile), one small subdomain and a thread per point
// (schwarz_point_tile).  The weighted own part goes straight to z (or is added to u), the weighted overlap
// parts go to a per-element overlap buffer.
// schwarz_overlap_add: gather form of the scatter, z[node] += contributions of
// the neighbours' subdomains in a fixed order -- deterministic, no atomics.
#include <type_traits>

#include "device.hpp"
#include "kernels.hpp"

namespace dgfas {

template <int N, int M>
struct SzShape {
  static constexpr int NS = N + 2 * M;
  static constexpr int LS = NS | 1;                 // odd pitch of xi_1 rows
  static constexpr int TILE = NS * NS * LS;
  static constexpr int THREADS = ((NS * NS + 63) / 64) * 64 < 64 ? 64 : ((NS * NS + 63) / 64) * 64;
};

// first DOF of element e, and first inbox slot of element e
template <int N, typename T>
__device__ __forceinline__ int64_t elem_base(const SchwarzArgs<T>& a, int e) {
  return a.off ? a.off[e] : (int64_t)e * (N * N * N);
}
template <int N, int M, typename T>
__device__ __forceinline__ int64_t inbox_base(const SchwarzArgs<T>& a, int e) {
  constexpr Regions<N, M> R{};
  return a.offO ? a.offO[e] : (int64_t)e * R.size;
}

int overlap_size(int p, int m) {
  const int n = p + 1;
  return 6 * m * n * n + 12 * m * m * n + 8 * m * m * m;
}

template <int N, int M, typename T>
struct SzSmem {
  T tA[SzShape<N, M>::TILE];   // the subdomain tile; every contraction updates its own lines in place
  int sOff[27];
};

// side variant v = left * 4 + right; only an interior side, code 0, has overlap
template <int M>
__device__ __forceinline__ int lo_layers(int v) {
  return (v >> 2) == 0 ? M : 0;
}
template <int M>
__device__ __forceinline__ int hi_layers(int v) {
  return (v & 3) == 0 ? M : 0;
}
// node of subdomain position q along a direction of variant v: (delta + 1) * 64 + local index, or
// -1 for padding.  The same as the host's table SchwarzArgs::map1d, without a load that waits
// for the variant.
template <int N, int M>
__device__ __forceinline__ int tile_map(int v, int q) {
  const int d = q - lo_layers<M>(v);
  if (d < 0) return N - M + q;
  if (d < N) return 64 + d;
  return d - N < hi_layers<M>(v) ? 128 + d - N : -1;
}

// read-only table at a uniform address, through the scalar cache
template <typename T>
using ctab = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ ctab<T> table(const T* p) {
  return (ctab<T>)(uintptr_t)p;
}

// table in LDS
template <typename T>
using ltab = const __attribute__((address_space(3))) T*;

// out_c = sum_q Mt[c][q] in_q for a tile line in registers
template <int NS, typename T>
__device__ __forceinline__ T line_row(ctab<T> Mt, int c, const T (&in)[NS]) {
  T s = 0;
#pragma unroll
  for (int q = 0; q < NS; ++q) s += Mt[c * NS + q] * in[q];
  return s;
}

// One subdomain solve (logical block lbr = element in the list, right-hand side fastest).
// Threads at or beyond THR (wider batched workgroups) only pass the barriers.
//
// The contractions run xi_3, xi_2, xi_1, divide, xi_1, xi_2, xi_3 with one thread per tile line: the
// first takes the gathered column from registers, the two around the division stay in registers
// and the last one's results go straight to their destinations, so the tile passes through LDS
// four times (8 accesses a point) and the workgroup meets at four barriers.  With the xi_3 pair in
// the middle, and the gather, the scatter and every contraction through LDS (14 accesses, seven
// barriers, node maps and weights staged behind one more), the 32^3, p = 7 solve took
// 204 us in FP64 (157 in FP32), now 174 (126); m = 3, 20^3, p = 8: 185, now 156.
// A column's destinations in z or an inbox are one pointer and a stride.
// The eigenvector rows are uniform over the workgroup and come through the scalar cache into SGPR
// operands.
template <int N, int M, typename T>
__device__ __forceinline__ void schwarz_tile(SchwarzArgs<T> a, const int lbr, SzSmem<N, M, T>& sm, int tid_in = -1) {
  using Sh = SzShape<N, M>;
  constexpr int NS = Sh::NS, LS = Sh::LS;
  constexpr Regions<N, M> R{};
  const int li = lbr / a.nrhs, rhs = lbr - li * a.nrhs;   // right-hand side fastest
  const int e = __builtin_amdgcn_readfirstlane(a.elist ? a.elist[li] : li);
  if (a.sel && !a.sel[e]) return;
  a.r += (int64_t)rhs * a.ndof;
  a.z += (int64_t)rhs * a.ndof;
  a.O += (int64_t)rhs * a.nin;
  const int tid = tid_in >= 0 ? tid_in : (int)threadIdx.x;   // tid_in: from a persistent batch
  T(&tA)[Sh::TILE] = sm.tA;
  int(&sOff)[27] = sm.sOff;
  if (M > 0 && tid < 27) sOff[tid] = R.off[tid];

  // variant per direction: uniform over the workgroup
  const int v0 = __builtin_amdgcn_readfirstlane(a.var[(int64_t)e * 3 + 0]);
  const int v1 = __builtin_amdgcn_readfirstlane(a.var[(int64_t)e * 3 + 1]);
  const int v2 = __builtin_amdgcn_readfirstlane(a.var[(int64_t)e * 3 + 2]);
  const ctab<T> S1 = table(a.S) + v0 * NS * NS, S1T = table(a.ST) + v0 * NS * NS;
  const ctab<T> S2 = table(a.S) + v1 * NS * NS, S2T = table(a.ST) + v1 * NS * NS;
  const ctab<T> S3 = table(a.S) + v2 * NS * NS, S3T = table(a.ST) + v2 * NS * NS;

  // gather r_s = R_s r, one thread per xi_3 column (s1, s2) of the tile: the column's
  // node (l1, l2) in each of the three elements it crosses is found once, the xi_3
  // positions (uniform over the workgroup) then only select the element and the layer
  const bool act = tid < NS * NS;
  const int c1 = tid % NS, c2 = tid / NS;
  const int m1 = tile_map<N, M>(v0, c1), m2 = act ? tile_map<N, M>(v1, c2) : -1;
  const bool in = m1 >= 0 && m2 >= 0;
  int nb[3] = {-1, -1, -1};   // the elements the column crosses; absent ones: zeros, no scatter
  if (in) {
#pragma unroll
    for (int d3 = 0; d3 < 3; ++d3) nb[d3] = a.nb27[(int64_t)e * 27 + d3 * 9 + (m2 >> 6) * 3 + (m1 >> 6)];
    if (a.deg) {
#pragma unroll
      for (int d3 = 0; d3 < 3; ++d3)
        if (nb[d3] >= 0 && a.deg[nb[d3]] != N - 1) nb[d3] = -1;   // another degree: zero fill, no scatter
    }
  }
  const int l12 = (m2 & 63) * N + (m1 & 63);
  const bool lo3 = M > 0 && lo_layers<M>(v2) != 0, hi3 = M > 0 && hi_layers<M>(v2) != 0;
  T line[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) line[q] = 0;
  // the column's layers below, in and above the element; LO = M or 0, the layers below in use
  auto gather = [&](auto lo) {
    constexpr int LO = decltype(lo)::value;
    if (nb[1] >= 0) {
      const T* __restrict__ p = a.r + elem_base<N>(a, nb[1]) + l12;
#pragma unroll
      for (int l = 0; l < N; ++l) line[LO + l] = p[l * N * N];
    }
    if (LO > 0 && nb[0] >= 0) {
      const T* __restrict__ p = a.r + elem_base<N>(a, nb[0]) + l12;
#pragma unroll
      for (int l = 0; l < LO; ++l) line[l] = p[(N - M + l) * N * N];
    }
    if (hi3 && nb[2] >= 0) {
      const T* __restrict__ p = a.r + elem_base<N>(a, nb[2]) + l12;
#pragma unroll
      for (int l = 0; l < M; ++l) line[LO + N + l] = p[l * N * N];
    }
  };
  if (lo3) gather(std::integral_constant<int, M>{});
  else gather(std::integral_constant<int, 0>{});
  // xi_3 with S3^T   (thread: s1 = c1, s2 = c2)
  if (act) {
#pragma unroll
    for (int c = 0; c < NS; ++c) tA[(c * NS + c2) * LS + c1] = line_row<NS, T>(S3T, c, line);
  }
  __syncthreads();
  // xi_2 with S2^T   (thread: s1 = c1, s3 = c2)
  if (act) {
#pragma unroll
    for (int q = 0; q < NS; ++q) line[q] = tA[(c2 * NS + q) * LS + c1];
#pragma unroll
    for (int c = 0; c < NS; ++c) tA[(c2 * NS + c) * LS + c1] = line_row<NS, T>(S2T, c, line);
  }
  __syncthreads();
  // xi_1 with S1^T, divide by D, xi_1 with S1   (thread: s2 = c1, s3 = c2)
  if (act) {
    const int b = (c2 * NS + c1) * LS;
#pragma unroll
    for (int q = 0; q < NS; ++q) line[q] = tA[b + q];
    const T g0 = a.gco[(int64_t)e * 4 + 0], g1 = a.gco[(int64_t)e * 4 + 1];
    const T g2 = a.gco[(int64_t)e * 4 + 2], g3 = a.gco[(int64_t)e * 4 + 3];
    const ctab<T> lam1 = table(a.lam) + v0 * NS;
    const T base = g0 + g2 * a.lam[v1 * NS + c1] + g3 * a.lam[v2 * NS + c2];
    T w[NS];
#pragma unroll
    for (int c = 0; c < NS; ++c) w[c] = line_row<NS, T>(S1T, c, line) / (base + g1 * lam1[c]);
#pragma unroll
    for (int c = 0; c < NS; ++c) tA[b + c] = line_row<NS, T>(S1, c, w);
  }
  __syncthreads();
  // xi_2 with S2   (thread: s1 = c1, s3 = c2)
  if (act) {
#pragma unroll
    for (int q = 0; q < NS; ++q) line[q] = tA[(c2 * NS + q) * LS + c1];
#pragma unroll
    for (int c = 0; c < NS; ++c) tA[(c2 * NS + c) * LS + c1] = line_row<NS, T>(S2, c, line);
  }
  __syncthreads();
  // xi_3 with S3 and the weighted scatter   (thread: s1 = c1, s2 = c2): own part to z, each overlap
  // part into the receiving element's inbox (region seen from the receiver), read back by
  // overlap_add.  The destination of the column in each of the three xi_3 elements is found once;
  // the xi_3 positions select it.
  if (in) {
#pragma unroll
    for (int q = 0; q < NS; ++q) line[q] = tA[(q * NS + c2) * LS + c1];
    const int d1 = (m1 >> 6) - 1, d2 = (m2 >> 6) - 1, l1 = m1 & 63, l2 = m2 & 63;
    const bool own = d1 == 0 && d2 == 0;
    const T w12 = a.W[v0 * NS + c1] * a.W[v1 * NS + c2];
    const ctab<T> W3 = table(a.W) + v2 * NS;
    // weighted value of position s3, whose node is l12 + l N^2 of element en
    auto value = [&](int s3, int en, int l) -> T {
      T t = line_row<NS, T>(S3, s3, line);
      if (a.corr) t += (T)(a.cscale[e] * (double)a.corr[(int64_t)e * (NS * NS * NS) + (s3 * NS + c2) * NS + c1]);
      T v = a.unweighted ? t : w12 * W3[s3] * t;
      if (a.cinv && !a.unweighted) v *= a.cinv[elem_base<N>(a, en) + l12 + l * (N * N)];   // normalised weight
      return v;
    };
    // first inbox slot of the column in the element at xi_3 offset d3, and the slots per layer
    const int x1 = d1 ? M : N, x2 = d2 ? M : N;
    const int cc = (d2 < 0 ? l2 - (N - M) : l2) * x1 + (d1 < 0 ? l1 - (N - M) : l1);
    const int ds = own ? N * N : x2 * x1;
    auto inbox = [&](int d3) -> T* {
      const int r = (1 - d3) * 9 + (1 - d2) * 3 + (1 - d1);      // direction from the receiver back to e
      return a.O + inbox_base<N, M>(a, nb[d3 + 1]) + sOff[r] + cc;
    };
    auto scatter = [&](auto lo) {
      constexpr int LO = decltype(lo)::value;
      if (nb[1] >= 0) {
        T* __restrict__ p = own ? a.z + elem_base<N>(a, e) + l12 : inbox(0);
#pragma unroll
        for (int l = 0; l < N; ++l) {
          T v = value(LO + l, nb[1], l);
          if (own && a.mode != 0) v += p[l * N * N];
          p[l * ds] = v;
        }
      }
      if (LO > 0 && nb[0] >= 0) {
        T* __restrict__ p = inbox(-1);
#pragma unroll
        for (int l = 0; l < LO; ++l) p[l * x2 * x1] = value(l, nb[0], N - M + l);
      }
      if (hi3 && nb[2] >= 0) {
        T* __restrict__ p = inbox(1);
#pragma unroll
        for (int l = 0; l < M; ++l) p[l * x2 * x1] = value(LO + N + l, nb[2], l);
      }
    };
    if (lo3) scatter(std::integral_constant<int, M>{});
    else scatter(std::integral_constant<int, 0>{});
  }
}

// Small subdomains (n <= 3, ns <= 5): several to a workgroup, one thread per xi_3 column as in
// schwarz_tile, with its order of contractions and its arithmetic.  The eigenvector tables of all 16 side
// variants (at most 3.2 KB) are staged in LDS, as the subdomains of a wavefront may differ; a
// wavefront whose subdomains share their variants takes the scalar cache instead.  One subdomain a
// workgroup with one thread per point read 12 values from LDS per point and contraction step and
// waited alone for its neighbour ids (p = 1: 26.7 us, now 15.8; p = 2: 59 us, now 30.7 on 32^3).
// Below kPackSubs subdomains (elements times right-hand sides) the chip is not full and one thread per point
// (schwarz_point_tile) has the shorter chain.  Point and pack form, p = 1 and 2 with one overlap layer:
//   FP64  2744: 5.9, 6.5 and 8.3, 9.4 us   4096: 6.7, 6.7 and 10.1, 10.0   5832: 8.3, 7.5 and 12.3, 11.4
//   FP32  4096: 5.7, 6.5 and 7.4, 8.4      5832: 6.7, 6.9 and 9.8, 8.9     8000: 7.5, 7.1 and 11.4, 10.1
// Four right-hand sides on 10^3 elements meet alike (6.6, 6.9 and 10.0, 9.9); both forms give the same bits.
template <typename T>
constexpr int64_t kPackSubs = sizeof(T) == 8 ? 4096 : 5632;

template <int N, int M, typename T, int THR>
struct PackSmem {
  static constexpr int NS = N + 2 * M, NS2 = NS * NS, SPW = THR / NS2, ROW = NS | 1;
  T tile[SPW][NS2 * ROW];
  T S[16][NS2 + 1];
  T lam[16][NS];
  T W[16][NS];
  int nb[SPW][27];
  int off[27];
};

// Subdomains lbt SPW .. of the list (element in the list, right-hand side fastest)
template <int N, int M, typename T, int THR>
__device__ __forceinline__ void schwarz_pack_tile(const SchwarzArgs<T>& a, const int lbt, PackSmem<N, M, T, THR>& sm,
                                                   const int tid) {
  using Sm = PackSmem<N, M, T, THR>;
  constexpr int NS = Sm::NS, NS2 = Sm::NS2, SPW = Sm::SPW, ROW = Sm::ROW;
  constexpr Regions<N, M> R{};
  const int sd = tid / NS2, c = tid - sd * NS2, c1 = c % NS, c2 = c / NS;
  const int lbr = lbt * SPW + sd;
  bool act = sd < SPW && lbr < a.nel * a.nrhs;
  const int li = act ? lbr / a.nrhs : 0, rhs = act ? lbr - li * a.nrhs : 0;
  const int e = a.elist ? a.elist[li] : li;
  if (a.sel && !a.sel[e]) act = false;
  const T* __restrict__ r = a.r + (int64_t)rhs * a.ndof;
  T* __restrict__ z = a.z + (int64_t)rhs * a.ndof;
  T* __restrict__ O = a.O + (int64_t)rhs * a.nin;
  const int v0 = a.var[(int64_t)e * 3 + 0], v1 = a.var[(int64_t)e * 3 + 1], v2 = a.var[(int64_t)e * 3 + 2];
  for (int t = tid; t < 16 * NS2; t += THR) sm.S[t / NS2][t % NS2] = a.S[t];
  for (int t = tid; t < 16 * NS; t += THR) {
    sm.lam[t / NS][t % NS] = a.lam[t];
    sm.W[t / NS][t % NS] = a.W[t];
  }
  if (M > 0 && tid < 27) sm.off[tid] = R.off[tid];
  // the neighbour ids go through LDS, so that they do not wait for the variants
  if (sd < SPW)
    for (int t = c; t < 27; t += NS2) sm.nb[sd][t] = a.nb27[(int64_t)e * 27 + t];
  const T g0 = a.gco[(int64_t)e * 4 + 0], g1 = a.gco[(int64_t)e * 4 + 1];
  const T g2 = a.gco[(int64_t)e * 4 + 2], g3 = a.gco[(int64_t)e * 4 + 3];
  __syncthreads();
  const int m1 = tile_map<N, M>(v0, c1), m2 = act ? tile_map<N, M>(v1, c2) : -1;
  const bool in = m1 >= 0 && m2 >= 0;
  const int l1 = m1 & 63, l2 = m2 & 63, l12 = l2 * N + l1;
  int nb[3] = {-1, -1, -1};   // the elements the column crosses; absent ones: zeros, no scatter
  if (in) {
#pragma unroll
    for (int d3 = 0; d3 < 3; ++d3) nb[d3] = sm.nb[sd][d3 * 9 + (m2 >> 6) * 3 + (m1 >> 6)];
    if (a.deg) {
#pragma unroll
      for (int d3 = 0; d3 < 3; ++d3)
        if (nb[d3] >= 0 && a.deg[nb[d3]] != N - 1) nb[d3] = -1;   // another degree: zero fill, no scatter
    }
  }
  T line[NS];
#pragma unroll
  for (int s3 = 0; s3 < NS; ++s3) {
    const int m3 = tile_map<N, M>(v2, s3);
    const int q = m3 < 0 ? -1 : (m3 < 64 ? nb[0] : (m3 < 128 ? nb[1] : nb[2]));
    line[s3] = 0;
    if (q >= 0) line[s3] = r[elem_base<N>(a, q) + l12 + (m3 & 63) * (N * N)];
  }
  // out_c = sum_q (S^T or S)[c][q] in_q with the table of variant v: v packs the three variants, `dir`
  // selects one, so that one test per wavefront covers all three
  const int code = (v0 * 16 + v1) * 16 + v2, first = __builtin_amdgcn_readfirstlane(code);
  const bool same = __ballot(code != first) == 0;
  const int u0 = first >> 8, u1 = (first >> 4) & 15, u2 = first & 15;
  auto apply = [&](int v, int u, bool tr, T (&t)[NS]) {
    T o[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) o[k] = 0;
    if (same) {
      const ctab<T> S = table(a.S) + u * NS2;
#pragma unroll
      for (int k = 0; k < NS; ++k)
#pragma unroll
        for (int q = 0; q < NS; ++q) o[k] += S[tr ? q * NS + k : k * NS + q] * t[q];
    } else {
      // one address in a register, the entries at offsets from it: left to itself the compiler adds a
      // constant per entry and keeps these constants in registers over a persistent loop
      ltab<T> S = (ltab<T>)sm.S[v];
      asm volatile("" : "+v"(S));
#pragma unroll
      for (int k = 0; k < NS; ++k)
#pragma unroll
        for (int q = 0; q < NS; ++q) o[k] += S[tr ? q * NS + k : k * NS + q] * t[q];
    }
#pragma unroll
    for (int k = 0; k < NS; ++k) t[k] = o[k];
  };
  T* const tile = sm.tile[sd < SPW ? sd : 0];
  const bool own = sd < SPW;
  auto load = [&](int at, int stride) {
#pragma unroll
    for (int q = 0; q < NS; ++q) line[q] = tile[at + q * stride];
  };
  auto store = [&](int at, int stride) {
    if (own) {
#pragma unroll
      for (int q = 0; q < NS; ++q) tile[at + q * stride] = line[q];
    }
    __syncthreads();
  };
  const int z0 = c2 * ROW + c1, sz = NS * ROW;   // column (s1 = c1, s2 = c2) along xi_3
  const int y0 = c2 * NS * ROW + c1;             // line (s1 = c1, s3 = c2) along xi_2
  const int x0 = c * ROW;                        // line (s2 = c1, s3 = c2) along xi_1
  apply(v2, u2, true, line);
  store(z0, sz);
  load(y0, ROW);
  apply(v1, u1, true, line);
  store(y0, ROW);
  load(x0, 1);
  apply(v0, u0, true, line);
  const T base = g0 + g2 * sm.lam[v1][c1] + g3 * sm.lam[v2][c2];
#pragma unroll
  for (int k = 0; k < NS; ++k) line[k] = line[k] / (base + g1 * sm.lam[v0][k]);
  apply(v0, u0, false, line);
  store(x0, 1);
  load(y0, ROW);
  apply(v1, u1, false, line);
  store(y0, ROW);
  load(z0, sz);
  apply(v2, u2, false, line);
  // weighted scatter: own part to z, overlap parts into the receivers' inboxes
  if (!in) return;
  const int d1 = (m1 >> 6) - 1, d2 = (m2 >> 6) - 1;
  const T w12 = sm.W[v0][c1] * sm.W[v1][c2];
  const int x1 = d1 ? M : N, x2 = d2 ? M : N;
  const int cc = (d2 < 0 ? l2 - (N - M) : l2) * x1 + (d1 < 0 ? l1 - (N - M) : l1);
#pragma unroll
  for (int s3 = 0; s3 < NS; ++s3) {
    const int m3 = tile_map<N, M>(v2, s3);
    if (m3 < 0) continue;
    const int l3 = m3 & 63, d3 = (m3 >> 6) - 1;
    const int q = d3 < 0 ? nb[0] : (d3 == 0 ? nb[1] : nb[2]);
    if (q < 0) continue;
    T t = line[s3];
    if (a.corr) t += (T)(a.cscale[e] * (double)a.corr[(int64_t)e * (NS2 * NS) + (s3 * NS + c2) * NS + c1]);
    T val = a.unweighted ? t : w12 * sm.W[v2][s3] * t;
    const int64_t gi = elem_base<N>(a, q) + l12 + l3 * (N * N);
    if (a.cinv && !a.unweighted) val *= a.cinv[gi];   // normalised weight
    if (d1 == 0 && d2 == 0 && d3 == 0) {
      if (a.mode == 0) z[gi] = val;
      else z[gi] += val;
    } else {
      const int rr = (1 - d3) * 9 + (1 - d2) * 3 + (1 - d1);      // direction from the receiver back to e
      const int c3 = d3 < 0 ? l3 - (N - M) : l3;
      O[inbox_base<N, M>(a, q) + sm.off[rr] + c3 * x2 * x1 + cc] = val;
    }
  }
}

template <int N, int M, typename T, int THR>
__global__ void __launch_bounds__(THR) schwarz_pack_kernel(SchwarzArgs<T> a) {
  using Sm = PackSmem<N, M, T, THR>;
  __shared__ Sm sm;
  const int lbt = xcd_block((a.nel * a.nrhs + Sm::SPW - 1) / Sm::SPW);
  if (lbt < 0) return;
  schwarz_pack_tile<N, M, T, THR>(a, lbt, sm, threadIdx.x);
}

// The same with one subdomain a workgroup and one thread per tile point, for few subdomains; the three
// directions' tables are staged in LDS.  Bound: the chain of gather, six contractions and scatter.  A thread
// finds its position, its element and its node once and keeps its value in a register: finding them anew
// in every step took 5.3 us on 4^3 and 6.0 on 12^3 at p = 1, now 4.6 and 5.2 (p = 2: 5.4 and 7.4, now 4.6 and 6.5).
template <int N, int M, typename T>
struct PtSmem {
  static constexpr int NS = N + 2 * M, NT = NS * NS * NS;
  T tile[NT];
  T S[3][NS * NS];
  T lam[3][NS];
  T W[3][NS];
  int map[3][NS];
  int nb[27];
  int off[27];
};

template <int N, int M, typename T>
__device__ __forceinline__ void schwarz_point_tile(SchwarzArgs<T> a, const int lbr, PtSmem<N, M, T>& sm) {
  using Sm = PtSmem<N, M, T>;
  constexpr int NS = Sm::NS, NT = Sm::NT, THR = (NT + 63) / 64 * 64;
  constexpr Regions<N, M> R{};
  const int li = lbr / a.nrhs, rhs = lbr - li * a.nrhs;
  const int e = a.elist ? a.elist[li] : li;
  if (a.sel && !a.sel[e]) return;
  a.r += (int64_t)rhs * a.ndof;
  a.z += (int64_t)rhs * a.ndof;
  a.O += (int64_t)rhs * a.nin;
  const int q = threadIdx.x;
  const int vv[3] = {__builtin_amdgcn_readfirstlane(a.var[(int64_t)e * 3 + 0]),
                     __builtin_amdgcn_readfirstlane(a.var[(int64_t)e * 3 + 1]),
                     __builtin_amdgcn_readfirstlane(a.var[(int64_t)e * 3 + 2])};
  for (int t = q; t < 3 * NS * NS; t += THR) {
    const int d = t / (NS * NS), k = t - d * NS * NS;
    sm.S[d][k] = a.S[vv[d] * NS * NS + k];
  }
  for (int t = q; t < 3 * NS; t += THR) {
    const int d = t / NS, k = t - d * NS;
    sm.lam[d][k] = a.lam[vv[d] * NS + k];
    sm.W[d][k] = a.W[vv[d] * NS + k];
    sm.map[d][k] = a.map1d[vv[d] * NS + k];
  }
  if (q < 27) {
    int nb = a.nb27[(int64_t)e * 27 + q];
    if (nb >= 0 && a.deg && a.deg[nb] != N - 1) nb = -1;   // another degree: zero fill, no scatter
    sm.nb[q] = nb;
    sm.off[q] = R.off[q];
  }
  const T g0 = a.gco[(int64_t)e * 4 + 0], g1 = a.gco[(int64_t)e * 4 + 1];
  const T g2 = a.gco[(int64_t)e * 4 + 2], g3 = a.gco[(int64_t)e * 4 + 3];
  __syncthreads();
  // gather r_s = R_s r
  const bool act = q < NT;   // threads beyond the tile only meet at the barriers
  const int s1 = q % NS, s2 = (q / NS) % NS, s3 = act ? q / (NS * NS) : 0;
  const int m1 = sm.map[0][s1], m2 = sm.map[1][s2], m3 = sm.map[2][s3];
  const bool in = act && m1 >= 0 && m2 >= 0 && m3 >= 0;
  const int src = in ? sm.nb[(m3 >> 6) * 9 + (m2 >> 6) * 3 + (m1 >> 6)] : -1;
  const int local = ((m3 & 63) * N + (m2 & 63)) * N + (m1 & 63);
  T v = 0;
  if (src >= 0) v = a.r[elem_base<N>(a, src) + local];
  if (act) sm.tile[q] = v;
  __syncthreads();
  // six contractions: xi_3 S3^T, xi_2 S2^T, xi_1 S1^T and 1/D, xi_1 S1, xi_2 S2, xi_3 S3
#pragma unroll 1
  for (int step = 0; step < 6; ++step) {
    const int dir = step < 3 ? 2 - step : step - 3;
    const bool tr = step < 3;
    const int c = dir == 0 ? s1 : dir == 1 ? s2 : s3, stride = dir == 0 ? 1 : (dir == 1 ? NS : NS * NS);
    if (act) {
      const T* line = sm.tile + (q - c * stride);
      v = 0;
#pragma unroll
      for (int k = 0; k < NS; ++k) v += (tr ? sm.S[dir][k * NS + c] : sm.S[dir][c * NS + k]) * line[k * stride];
      if (step == 2) v = v / (g0 + g2 * sm.lam[1][s2] + g3 * sm.lam[2][s3] + g1 * sm.lam[0][s1]);
    }
    if (step == 5) break;
    __syncthreads();
    if (act) sm.tile[q] = v;
    __syncthreads();
  }
  // weighted scatter: own part to z, overlap parts into the receivers' inboxes
  if (src < 0) return;
  T t = v;
  if (a.corr) t += (T)(a.cscale[e] * (double)a.corr[(int64_t)e * NT + q]);
  T val = a.unweighted ? t : sm.W[0][s1] * sm.W[1][s2] * sm.W[2][s3] * t;
  const int64_t gi = elem_base<N>(a, src) + local;
  if (a.cinv && !a.unweighted) val *= a.cinv[gi];   // normalised weight
  const int d1 = (m1 >> 6) - 1, d2 = (m2 >> 6) - 1, d3 = (m3 >> 6) - 1;
  const int l1 = m1 & 63, l2 = m2 & 63, l3 = m3 & 63;
  if (d1 == 0 && d2 == 0 && d3 == 0) {
    if (a.mode == 0) a.z[gi] = val;
    else a.z[gi] += val;
  } else {
    const int r = (1 - d3) * 9 + (1 - d2) * 3 + (1 - d1);      // direction from the receiver back to e
    const int c1 = d1 < 0 ? l1 - (N - M) : l1, c2 = d2 < 0 ? l2 - (N - M) : l2, c3 = d3 < 0 ? l3 - (N - M) : l3;
    const int x1 = d1 ? M : N, x2 = d2 ? M : N;
    a.O[inbox_base<N, M>(a, src) + sm.off[r] + (c3 * x2 + c2) * x1 + c1] = val;
  }
}

template <int N, int M, typename T>
__global__ void __launch_bounds__(((N + 2 * M) * (N + 2 * M) * (N + 2 * M) + 63) / 64 * 64)
schwarz_point_kernel(SchwarzArgs<T> a) {
  __shared__ PtSmem<N, M, T> sm;
  const int lbr = xcd_block(a.nel * a.nrhs);
  if (lbr < 0) return;
  schwarz_point_tile<N, M, T>(a, lbr, sm);
}

template <int N, int EPB>
struct AddShape {
  static constexpr int N3 = N * N * N, THREADS = 256;
  static constexpr int KN = (EPB * N3 + THREADS - 1) / THREADS;   // nodes per thread
};

// Waves per SIMD asked of the compiler: eight (64 registers), or what the tiles leave room for in the CU's
// 160 KB of LDS: in FP64 at p = 8 seven with one overlap layer and six with two or three.  The two-wave
// workgroups hide each other's gather and barriers (32^3, p = 7: 180 us at six waves, 174 at eight; 20^3,
// p = 8, m = 1 to 3: 59, 100 and 159 us with a bound of eight, 58, 97 and 158 with these).
template <int N, int M, typename T>
constexpr int solve_waves() {
  const int w = 163840 / (int)sizeof(SzSmem<N, M, T>) * (SzShape<N, M>::THREADS / 64) / 4;
  return w < 8 ? w : 8;
}

template <int N, int M, typename T>
__global__ void __launch_bounds__((SzShape<N, M>::THREADS), (solve_waves<N, M, T>()))
schwarz_solve_kernel(SchwarzArgs<T> a) {
  __shared__ SzSmem<N, M, T> sm;
  const int lbr = xcd_block(a.nel * a.nrhs);
  if (lbr < 0) return;
  schwarz_tile<N, M, T>(a, lbr, sm);
}

template <int N, int M, typename T, int EPB = kAddElems[N]>
struct AddSmem {
  static constexpr int OSZ = Regions<N, M>{}.size;
  static constexpr bool STAGED = N > 3;   // else the few entries are read where they are
  T box[STAGED ? EPB : 1][STAGED ? OSZ : 1];   // the elements' inboxes
  int sOff[27];
  double red[2][AddShape<N, EPB>::THREADS / 64];   // per-wavefront partial sums of the fused dot products
};

// Sum of the neighbours' overlap contributions to node (l0, l1, l2) from the element's
// inbox, in a fixed order (the up to 7 regions whose overlap covers the node).  Inbox regions of
// absent neighbours stay zero.
template <int N, int M, typename T>
__device__ __forceinline__ T inbox_sum(const T* box, const int* sOff, const int (&l)[3], const int (&od)[3]) {
  // every load is issued unconditionally (invalid ones read entry 0 and are masked), so that none
  // waits on another
  T vals[7];
  bool ok[7];
#pragma unroll
  for (int bits = 1; bits < 8; ++bits) {
    const bool valid = ((bits & 1) == 0 || od[0] != 0) && ((bits & 2) == 0 || od[1] != 0) &&
                       ((bits & 4) == 0 || od[2] != 0);
    const int dd[3] = {(bits & 1) ? od[0] : 0, (bits & 2) ? od[1] : 0, (bits & 4) ? od[2] : 0};
    const int r = (dd[2] + 1) * 9 + (dd[1] + 1) * 3 + (dd[0] + 1);
    const int c1 = dd[0] > 0 ? l[0] - (N - M) : l[0];
    const int c2 = dd[1] > 0 ? l[1] - (N - M) : l[1];
    const int c3 = dd[2] > 0 ? l[2] - (N - M) : l[2];
    const int x1 = dd[0] ? M : N, x2 = dd[1] ? M : N;
    ok[bits - 1] = valid;
    vals[bits - 1] = box[valid ? sOff[r] + (c3 * x2 + c2) * x1 + c1 : 0];
  }
  T acc = 0;
#pragma unroll
  for (int t = 0; t < 7; ++t) acc += ok[t] ? vals[t] : T(0);
  return acc;
}

// z[node] += sum of the neighbours' overlap contributions in the element's own inbox.  From n = 4 on the
// inbox, one contiguous block, comes into LDS with coalesced loads: reading the up to 7 entries of
// every node from global memory is seven short gathers a node (32^3, p = 7: 128 us that way, 104 from LDS with one node a thread, now 73; with the dot
// products 154, now 123, in FP32 122, now 71).  With dotz set, also the tile's sums of z dr and
// z (dr - dr0) over every node (deterministic order).
template <int N, int M, typename T, int EPB>
__device__ __forceinline__ void overlap_add_tile(SchwarzArgs<T> a, const int lbr, AddSmem<N, M, T, EPB>& sm,
                                                 int tid_in = -1) {
  using Sh = AddShape<N, EPB>;
  using Sm = AddSmem<N, M, T, EPB>;
  constexpr int N3 = Sh::N3, KN = Sh::KN, THR = Sh::THREADS, OSZ = Sm::OSZ;
  constexpr int NB = (EPB * OSZ + THR - 1) / THR;
  constexpr Regions<N, M> R{};
  const int lb = lbr / a.nrhs, rhs = lbr - lb * a.nrhs;
  a.z += (int64_t)rhs * a.ndof;
  a.O += (int64_t)rhs * a.nin;
  const int tid = tid_in >= 0 ? tid_in : (int)threadIdx.x;
  if (tid < 27) sm.sOff[tid] = R.off[tid];
  const int ne = min(EPB, a.nel - lb * EPB);   // elements of this tile
  auto element = [&](int le) {
    const int li = lb * EPB + min(le, ne - 1);
    return a.elist ? a.elist[li] : li;
  };
  T in[NB], z0[KN];
  if constexpr (Sm::STAGED) {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int t = min(tid + k * THR, EPB * OSZ - 1), le = t / OSZ;
      in[k] = a.O[inbox_base<N, M>(a, element(le)) + (t - le * OSZ)];
    }
  }
  int64_t gi[KN];
  double rv[KN], r0v[KN];
#pragma unroll
  for (int k = 0; k < KN; ++k) {
    const int t = min(tid + k * THR, EPB * N3 - 1), le = t / N3;
    gi[k] = elem_base<N>(a, element(le)) + (t - le * N3);
    z0[k] = a.z[gi[k]];
    rv[k] = r0v[k] = 0;
    if (a.dotz) {
      const int64_t ri = (int64_t)rhs * a.ndof + gi[k];
      rv[k] = (double)a.dr[ri];
      if (a.dr0) r0v[k] = (double)a.dr0[ri];
    }
  }
  if constexpr (Sm::STAGED) {
#pragma unroll
    for (int k = 0; k < NB; ++k)
      if (tid + k * THR < EPB * OSZ) sm.box[(tid + k * THR) / OSZ][(tid + k * THR) % OSZ] = in[k];
  }
  __syncthreads();
  double pz = 0, pz2 = 0;
#pragma unroll
  for (int k = 0; k < KN; ++k) {
    const int t = tid + k * THR, le = t / N3, node = t - le * N3;
    if (le >= ne) continue;
    const int l[3] = {node % N, (node / N) % N, node / (N * N)};
    // per direction the offset towards the one neighbour whose overlap can cover this node
    int od[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) od[d] = (l[d] < M) ? -1 : ((l[d] >= N - M) ? 1 : 0);
    T zv = z0[k];
    if (od[0] != 0 || od[1] != 0 || od[2] != 0) {
      if constexpr (Sm::STAGED) zv += inbox_sum<N, M, T>(sm.box[le], sm.sOff, l, od);
      else zv += inbox_sum<N, M, T>(a.O + inbox_base<N, M>(a, element(le)), sm.sOff, l, od);
      a.z[gi[k]] = zv;
    }
    pz += (double)zv * rv[k];
    if (a.dr0) pz2 += (double)zv * (rv[k] - r0v[k]);
  }
  if (a.dotz) {
    pz = wave_sum(pz);
    pz2 = wave_sum(pz2);
    if ((tid & 63) == 0) {
      sm.red[0][tid >> 6] = pz;
      sm.red[1][tid >> 6] = pz2;
    }
    __syncthreads();
    if (tid == 0) {
      double s = 0, s2 = 0;
      for (int w = 0; w < THR / 64; ++w) {
        s += sm.red[0][w];
        s2 += sm.red[1][w];
      }
      const int ntiles = (a.nel + EPB - 1) / EPB;
      a.dotz[(int64_t)rhs * ntiles + lb] = s;
      if (a.dotz2) a.dotz2[(int64_t)rhs * ntiles + lb] = s2;
    }
  }
}

template <int N, int M, typename T, int EPB>
__global__ void __launch_bounds__((AddShape<N, EPB>::THREADS))
schwarz_overlap_add_kernel(SchwarzArgs<T> a) {
  __shared__ AddSmem<N, M, T, EPB> sm;
  const int lbr = xcd_block(((a.nel + EPB - 1) / EPB) * a.nrhs);
  if (lbr < 0) return;
  overlap_add_tile<N, M, T, EPB>(a, lbr, sm);
}

// ---------------------------------------------------------------------------
// Tile helpers for the learned correction.  A tile is the NS^3 subdomain block of a
// vector in the layout of the FD solve (padded positions zero).
template <int N, int M>
struct TileCtx {
  static constexpr int NS = N + 2 * M, NT = NS * NS * NS;
  int map[3][NS];
  int nb[27];
};

template <int N, int M, typename T>
__device__ void load_tile_ctx(const SchwarzArgs<T>& a, int e, TileCtx<N, M>& c) {
  constexpr int NS = N + 2 * M;
  for (int t = threadIdx.x; t < 3 * NS; t += blockDim.x) {
    const int d = t / NS, q = t - d * NS;
    c.map[d][q] = a.map1d[a.var[(int64_t)e * 3 + d] * NS + q];
  }
  for (int t = threadIdx.x; t < 27; t += blockDim.x) c.nb[t] = a.nb27[(int64_t)e * 27 + t];
}

// global index of tile position q of the element, or -1 (padding / absent neighbour)
template <int N, int M>
__device__ __forceinline__ int64_t tile_index(const TileCtx<N, M>& c, int q) {
  constexpr int NS = N + 2 * M;
  const int s1 = q % NS, s2 = (q / NS) % NS, s3 = q / (NS * NS);
  const int m1 = c.map[0][s1], m2 = c.map[1][s2], m3 = c.map[2][s3];
  if (m1 < 0 || m2 < 0 || m3 < 0) return -1;
  const int src = c.nb[(m3 >> 6) * 9 + (m2 >> 6) * 3 + (m1 >> 6)];
  if (src < 0) return -1;
  return (int64_t)src * (N * N * N) + ((m3 & 63) * N + (m2 & 63)) * N + (m1 & 63);
}

// X[row] = [tile(v) / |tile(v)|, J9[e]], norms[row] = |tile(v)|
template <int N, int M, typename T>
__global__ void __launch_bounds__(256) tile_features_kernel(SchwarzArgs<T> a, const int* ids, int n,
                                                            const double* __restrict__ v, const double* __restrict__ J9,
                                                            float* __restrict__ X, double* __restrict__ norms) {
  using C = TileCtx<N, M>;
  __shared__ C c;
  __shared__ double tile[C::NT];
  __shared__ double red[256];
  const int row = blockIdx.x;
  if (row >= n) return;
  const int e = ids ? ids[row] : row;
  load_tile_ctx<N, M, T>(a, e, c);
  __syncthreads();
  double s = 0;
  for (int q = threadIdx.x; q < C::NT; q += 256) {
    const int64_t gi = tile_index<N, M>(c, q);
    const double x = gi >= 0 ? v[gi] : 0.0;
    tile[q] = x;
    s += x * x;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  const double nrm = sqrt(red[0]);
  const double inv = nrm > 0 ? 1.0 / nrm : 0.0;
  const int64_t in = C::NT + 9;
  for (int q = threadIdx.x; q < C::NT; q += 256) X[(int64_t)row * in + q] = (float)(tile[q] * inv);
  if (threadIdx.x < 9) X[(int64_t)row * in + C::NT + threadIdx.x] = (float)J9[(int64_t)e * 9 + threadIdx.x];
  if (threadIdx.x == 0) norms[row] = nrm;
}

// out[row] = (tile(v1) - tile(v2)) / norms[row]
template <int N, int M, typename T>
__global__ void __launch_bounds__(256) tile_diff_kernel(SchwarzArgs<T> a, const int* ids, int n,
                                                        const double* __restrict__ v1, const double* __restrict__ v2,
                                                        const double* __restrict__ norms, float* __restrict__ out) {
  using C = TileCtx<N, M>;
  __shared__ C c;
  const int row = blockIdx.x;
  if (row >= n) return;
  const int e = ids ? ids[row] : row;
  load_tile_ctx<N, M, T>(a, e, c);
  __syncthreads();
  const double inv = norms[row] > 0 ? 1.0 / norms[row] : 0.0;
  for (int q = threadIdx.x; q < C::NT; q += 256) {
    const int64_t gi = tile_index<N, M>(c, q);
    out[(int64_t)row * C::NT + q] = gi >= 0 ? (float)((v1[gi] - v2[gi]) * inv) : 0.f;
  }
}

// mask = 1 on every node of the listed subdomains
template <int N, int M, typename T>
__global__ void __launch_bounds__(256) mark_kernel(SchwarzArgs<T> a, const int* ids, int n, double* __restrict__ mask) {
  using C = TileCtx<N, M>;
  __shared__ C c;
  const int row = blockIdx.x;
  if (row >= n) return;
  const int e = ids ? ids[row] : row;
  load_tile_ctx<N, M, T>(a, e, c);
  __syncthreads();
  for (int q = threadIdx.x; q < C::NT; q += 256) {
    const int64_t gi = tile_index<N, M>(c, q);
    if (gi >= 0) mask[gi] = 1.0;
  }
}

template <int N, int M, typename T>
void launch_features(const SchwarzArgs<T>& a, const int* ids, int n, const double* v, const double* J9, float* X,
                     double* norms, hipStream_t st) {
  hipLaunchKernelGGL((tile_features_kernel<N, M, T>), dim3(n), dim3(256), 0, st, a, ids, n, v, J9, X, norms);
}
template <int N, int M, typename T>
void launch_diff(const SchwarzArgs<T>& a, const int* ids, int n, const double* v1, const double* v2,
                 const double* norms, float* out, hipStream_t st) {
  hipLaunchKernelGGL((tile_diff_kernel<N, M, T>), dim3(n), dim3(256), 0, st, a, ids, n, v1, v2, norms, out);
}
template <int N, int M, typename T>
void launch_mark(const SchwarzArgs<T>& a, const int* ids, int n, double* mask, hipStream_t st) {
  hipLaunchKernelGGL((mark_kernel<N, M, T>), dim3(n), dim3(256), 0, st, a, ids, n, mask);
}

#define DGFAS_TILE_CASES(CALL)                           \
  switch (p * 16 + m) {                                  \
    case 1 * 16 + 1: CALL(2, 1); break;                  \
    case 2 * 16 + 1: CALL(3, 1); break;                  \
    case 3 * 16 + 1: CALL(4, 1); break;                  \
    case 4 * 16 + 1: CALL(5, 1); break;                  \
    case 5 * 16 + 1: CALL(6, 1); break;                  \
    case 6 * 16 + 1: CALL(7, 1); break;                  \
    case 7 * 16 + 1: CALL(8, 1); break;                  \
    case 8 * 16 + 1: CALL(9, 1); break;                  \
    default: break;                                      \
  }

template <typename T>
void tile_features(int p, int m, const SchwarzArgs<T>& a, const int* ids, int n, const double* v, const double* J9,
                   float* X, double* norms, hipStream_t st) {
#define CALLF(NN, MM) launch_features<NN, MM, T>(a, ids, n, v, J9, X, norms, st)
  DGFAS_TILE_CASES(CALLF)
#undef CALLF
}
template <typename T>
void tile_diff(int p, int m, const SchwarzArgs<T>& a, const int* ids, int n, const double* v1, const double* v2,
               const double* norms, float* out, hipStream_t st) {
#define CALLD(NN, MM) launch_diff<NN, MM, T>(a, ids, n, v1, v2, norms, out, st)
  DGFAS_TILE_CASES(CALLD)
#undef CALLD
}
template <typename T>
void mark_subdomains(int p, int m, const SchwarzArgs<T>& a, const int* ids, int n, double* mask, hipStream_t st) {
#define CALLM(NN, MM) launch_mark<NN, MM, T>(a, ids, n, mask, st)
  DGFAS_TILE_CASES(CALLM)
#undef CALLM
}
template void tile_features<double>(int, int, const SchwarzArgs<double>&, const int*, int, const double*,
                                    const double*, float*, double*, hipStream_t);
template void tile_diff<double>(int, int, const SchwarzArgs<double>&, const int*, int, const double*, const double*,
                                const double*, float*, hipStream_t);
template void mark_subdomains<double>(int, int, const SchwarzArgs<double>&, const int*, int, double*, hipStream_t);

template <int N, int M, typename T>
void launch_schwarz(const SchwarzArgs<T>& a, hipStream_t st) {
  if constexpr (N <= 3) {
    constexpr int NS = N + 2 * M, NT = (NS * NS * NS + 63) / 64 * 64, SPW = PackSmem<N, M, T, 256>::SPW;
    if ((int64_t)a.nel * a.nrhs >= kPackSubs<T>)
      hipLaunchKernelGGL((schwarz_pack_kernel<N, M, T, 256>), dim3(xcd_grid((a.nel * a.nrhs + SPW - 1) / SPW)), dim3(256),
                         0, st, a);
    else
      hipLaunchKernelGGL((schwarz_point_kernel<N, M, T>), dim3(xcd_grid(a.nel * a.nrhs)), dim3(NT), 0, st, a);
  } else {
    hipLaunchKernelGGL((schwarz_solve_kernel<N, M, T>), dim3(xcd_grid(a.nel * a.nrhs)), dim3(SzShape<N, M>::THREADS),
                       0, st, a);
  }
}

template <int N, int M, typename T, int EPB>
void launch_overlap_tiles(const SchwarzArgs<T>& a, hipStream_t st) {
  const int nb = ((a.nel + EPB - 1) / EPB) * a.nrhs;
  hipLaunchKernelGGL((schwarz_overlap_add_kernel<N, M, T, EPB>), dim3(xcd_grid(nb)), dim3(AddShape<N, EPB>::THREADS), 0, st,
                     a);
}
template <int N, int M, typename T>
void launch_overlap(const SchwarzArgs<T>& a, hipStream_t st) {
  if constexpr (M > 0) {
    if constexpr (add_elems(N, 0) != kAddElems[N]) {   // one element a tile on few elements
      if (add_elems(N, a.nel) == 1) return launch_overlap_tiles<N, M, T, 1>(a, st);
    }
    launch_overlap_tiles<N, M, T, kAddElems[N]>(a, st);
  }
}

#define DGFAS_SZ_CASES(F)                                                       \
  switch (p * 16 + m) {                                                         \
    case 1 * 16 + 0: F<2, 0, T>(a, st); break;                                  \
    case 1 * 16 + 1: F<2, 1, T>(a, st); break;                                  \
    case 2 * 16 + 0: F<3, 0, T>(a, st); break;                                  \
    case 2 * 16 + 1: F<3, 1, T>(a, st); break;                                  \
    case 3 * 16 + 0: F<4, 0, T>(a, st); break;                                  \
    case 3 * 16 + 1: F<4, 1, T>(a, st); break;                                  \
    case 4 * 16 + 0: F<5, 0, T>(a, st); break;                                  \
    case 4 * 16 + 1: F<5, 1, T>(a, st); break;                                  \
    case 4 * 16 + 2: F<5, 2, T>(a, st); break;                                  \
    case 5 * 16 + 0: F<6, 0, T>(a, st); break;                                  \
    case 5 * 16 + 1: F<6, 1, T>(a, st); break;                                  \
    case 6 * 16 + 0: F<7, 0, T>(a, st); break;                                  \
    case 6 * 16 + 1: F<7, 1, T>(a, st); break;                                  \
    case 7 * 16 + 0: F<8, 0, T>(a, st); break;                                  \
    case 7 * 16 + 1: F<8, 1, T>(a, st); break;                                  \
    case 8 * 16 + 0: F<9, 0, T>(a, st); break;                                  \
    case 8 * 16 + 1: F<9, 1, T>(a, st); break;                                  \
    case 8 * 16 + 2: F<9, 2, T>(a, st); break;                                  \
    case 8 * 16 + 3: F<9, 3, T>(a, st); break;                                  \
    default: break;                                                             \
  }

template <typename T>
void schwarz_solve(int p, int m, const SchwarzArgs<T>& a, hipStream_t st) {
  DGFAS_SZ_CASES(launch_schwarz)
}
template <typename T>
void schwarz_overlap_add(int p, int m, const SchwarzArgs<T>& a, hipStream_t st) {
  if (m == 0) return;
  DGFAS_SZ_CASES(launch_overlap)
}

// ---------------------------------------------------------------------------
// Batched launches over the degree buckets of a mixed-degree level (overlap m = 1).
template <typename T, int N, int THR>
constexpr size_t sz_smem_upto() {
  if constexpr (N < 2) {
    return 0;
  } else {
    constexpr size_t a = N <= 3 ? sizeof(PackSmem<N, 1, T, THR>) : sizeof(SzSmem<N, 1, T>),
                     b = sz_smem_upto<T, N - 1, THR>();
    return a > b ? a : b;
  }
}

// The persistent form is held to six waves per SIMD in FP64 and eight in FP32: without a bound the
// compiler keeps the constants of every degree's tile live over the loop (162 and 132 registers, three
// waves; 27^3 hp front, largest degree 8: application 162 us, now 110; FP32 smoothing of four steps 1.62 ms,
// now 1.43).  The one-tile form has no loop and needs no bound (96 us).
template <typename T, bool PERSIST>
constexpr int kSolveWaves = !PERSIST ? 1 : sizeof(T) == 8 ? 6 : 8;

template <int NMAX, typename T, bool PERSIST>
__global__ void __launch_bounds__((SzShape<NMAX, 1>::THREADS), (kSolveWaves<T, PERSIST>))
schwarz_batched_kernel(SchwarzArgs<T> a, const BucketDesc<T>* __restrict__ bd, int nb, int ntiles) {
  constexpr int THR = SzShape<NMAX, 1>::THREADS;
  __shared__ __align__(16) char smem[sz_smem_upto<T, NMAX, THR>()];
  // tiles dealt round-robin over the XCDs (the hardware order): the work list runs from the
  // largest degree to the smallest, and contiguous ranges per XCD would leave one XCD all
  // the large tiles.  The persistent form strides through the list, with a barrier between
  // tiles for the shared memory.
  auto tile = [&](int t) {
    int tid = -1;   // persistent form: an opaque copy per tile (see sipg_batched_kernel)
    if constexpr (PERSIST) {
      tid = threadIdx.x;
      asm volatile("v_mov_b32 %0, %1" : "=v"(tid) : "v"(tid));
    }
    const int k = find_bucket(bd, nb, kStageSolve, t);
    SchwarzArgs<T> x = a;
    x.nel = bd[k].nel;
    x.elist = bd[k].elist;
    x.S = bd[k].S;
    x.ST = bd[k].ST;
    x.lam = bd[k].lam;
    x.W = bd[k].W;
    x.map1d = bd[k].map1d;
    const int lbr = t - bd[k].tile0[kStageSolve];
    switch (bd[k].p) {
#define DGFAS_SZB(P)                                                                                  \
  case P:                                                                                             \
    if constexpr (P + 1 <= 3) schwarz_pack_tile<P + 1, 1, T, THR>(x, lbr, *reinterpret_cast<PackSmem<P + 1, 1, T, THR>*>(smem), tid < 0 ? (int)threadIdx.x : tid); \
    else if constexpr (P + 1 <= NMAX) schwarz_tile<P + 1, 1, T>(x, lbr, *reinterpret_cast<SzSmem<P + 1, 1, T>*>(smem), tid); \
    break;
      DGFAS_SZB(1) DGFAS_SZB(2) DGFAS_SZB(3) DGFAS_SZB(4) DGFAS_SZB(5) DGFAS_SZB(6) DGFAS_SZB(7) DGFAS_SZB(8)
#undef DGFAS_SZB
      default: break;
    }
  };
  if constexpr (PERSIST) {
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
      if (t != (int)blockIdx.x) __syncthreads();
      tile(t);
    }
  } else {
    if ((int)blockIdx.x < ntiles) tile(blockIdx.x);
  }
}

template <typename T, int N>
constexpr size_t add_smem_upto() {
  if constexpr (N < 2) {
    return 0;
  } else {
    constexpr size_t a = sizeof(AddSmem<N, 1, T>), b = add_smem_upto<T, N - 1>();
    return a > b ? a : b;
  }
}

template <int NMAX, typename T, bool PERSIST>
__global__ void __launch_bounds__((AddShape<NMAX, 1>::THREADS))
overlap_add_batched_kernel(SchwarzArgs<T> a, const BucketDesc<T>* __restrict__ bd, int nb, int ntiles) {
  __shared__ __align__(16) char smem[add_smem_upto<T, NMAX>()];
  // tiles dealt round-robin over the XCDs (the hardware order), strided in the persistent form
  auto tile = [&](int t) {
    int tid = -1;   // persistent form: an opaque copy per tile (see sipg_batched_kernel)
    if constexpr (PERSIST) {
      tid = threadIdx.x;
      asm volatile("v_mov_b32 %0, %1" : "=v"(tid) : "v"(tid));
    }
    const int k = find_bucket(bd, nb, kStageAdd, t);
    SchwarzArgs<T> x = a;
    x.nel = bd[k].nel;
    x.elist = bd[k].elist;
    const int lbr = t - bd[k].tile0[kStageAdd];
    switch (bd[k].p) {
#define DGFAS_ADB(P)                                                          \
  case P:                                                                     \
    if constexpr (P + 1 <= NMAX) overlap_add_tile<P + 1, 1, T, kAddElems[P + 1]>(x, lbr, *reinterpret_cast<AddSmem<P + 1, 1, T>*>(smem), tid); \
    break;
      DGFAS_ADB(1) DGFAS_ADB(2) DGFAS_ADB(3) DGFAS_ADB(4) DGFAS_ADB(5) DGFAS_ADB(6) DGFAS_ADB(7) DGFAS_ADB(8)
#undef DGFAS_ADB
      default: break;
    }
  };
  if constexpr (PERSIST) {
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
      if (t != (int)blockIdx.x) __syncthreads();
      tile(t);
    }
  } else {
    if ((int)blockIdx.x < ntiles) tile(blockIdx.x);
  }
}

#define DGFAS_BATCH_ONE(KERNEL, NM)                                                                     \
  if (l.persistent) hipLaunchKernelGGL((KERNEL<NM, T, true>), g, b, 0, st, a, bd, l.nb, l.ntiles);     \
  else hipLaunchKernelGGL((KERNEL<NM, T, false>), g, b, 0, st, a, bd, l.nb, l.ntiles);
#define DGFAS_BATCH_LAUNCH(KERNEL, STAGE)                                                              \
  if (l.ntiles <= 0) return;                                                                           \
  const dim3 g(l.grid), b(stage_threads(STAGE, pmax));                                                 \
  if (pmax <= 5) { DGFAS_BATCH_ONE(KERNEL, 6) }                                                        \
  else if (pmax == 6) { DGFAS_BATCH_ONE(KERNEL, 7) }                                                   \
  else if (pmax == 7) { DGFAS_BATCH_ONE(KERNEL, 8) }                                                   \
  else { DGFAS_BATCH_ONE(KERNEL, 9) }

template <typename T>
void schwarz_solve_batched(int pmax, const SchwarzArgs<T>& a, const BucketDesc<T>* bd, const BatchLaunch& l,
                           hipStream_t st) {
  DGFAS_BATCH_LAUNCH(schwarz_batched_kernel, kStageSolve)
}
template <typename T>
void schwarz_overlap_add_batched(int pmax, const SchwarzArgs<T>& a, const BucketDesc<T>* bd, const BatchLaunch& l,
                                 hipStream_t st) {
  DGFAS_BATCH_LAUNCH(overlap_add_batched_kernel, kStageAdd)
}
#undef DGFAS_BATCH_LAUNCH
#undef DGFAS_BATCH_ONE

template void schwarz_solve_batched<double>(int, const SchwarzArgs<double>&, const BucketDesc<double>*,
                                            const BatchLaunch&, hipStream_t);
template void schwarz_solve_batched<float>(int, const SchwarzArgs<float>&, const BucketDesc<float>*,
                                           const BatchLaunch&, hipStream_t);
template void schwarz_overlap_add_batched<double>(int, const SchwarzArgs<double>&, const BucketDesc<double>*,
                                                  const BatchLaunch&, hipStream_t);
template void schwarz_overlap_add_batched<float>(int, const SchwarzArgs<float>&, const BucketDesc<float>*,
                                                 const BatchLaunch&, hipStream_t);

template void schwarz_solve<double>(int, int, const SchwarzArgs<double>&, hipStream_t);
template void schwarz_solve<float>(int, int, const SchwarzArgs<float>&, hipStream_t);
template void schwarz_overlap_add<double>(int, int, const SchwarzArgs<double>&, hipStream_t);
template void schwarz_overlap_add<float>(int, int, const SchwarzArgs<float>&, hipStream_t);

}  // namespace dgfas
