// K1: sum-factorised SIPG operator apply / residual on curvilinear hexahedra
// (eq. helmholtz:dgm) and the one-time geometry kernels (Sec. 2.2).
//
// Face terms use the identity
//   nu * omega * s * (n_out . grad xi_c) = +-G_bc / w_end     (normal axis b)
// with the contravariant fluxes F_b = sum_c G_bc d_c u (G_bc = w J nu grad xi_b . grad xi_c):
// the own normal flux is F_b / w_end at the face node and the lifting term adds
// sigma * G_bc / w_end to F_c there; the neighbour's flux is rebuilt from its normal node line
// (L2-resident) and its metric at the shared face.  Every node's terms are summed by its owner in
// a fixed order: the result is deterministic without atomics.
// On unstructured meshes (ORIENT) the neighbour may meet a face with any of its faces and any
// relative orientation (Sec. 5.1): its node line is then read at the orientation-mapped face
// node, and its tangential derivatives are the own face grid's, exchanged and negated as the
// orientation requires.
#include "device.hpp"
#include "kernels.hpp"


namespace dgfas {

// elements per workgroup of the kernels with one thread per node
template <int N>
struct OpShape {
  static constexpr int N2 = N * N, N3 = N * N * N;
  static constexpr int EPB = (N3 >= 256) ? 1 : (256 / N3);
  static constexpr int THREADS = ((EPB * N3 + 63) / 64) * 64;
};

// The operator's tile: EPB elements, H threads per xi_3 column (i, j) of an element, each owning
// KPT = ceil(N / H) of the column's nodes.  A node's metric, fluxes and lifting stay in its owner's
// registers, a row of D is read once per thread and direction, and only u, the neighbours' traces,
// the face terms and the fluxes on their way into the transposed contractions go through LDS.
// One thread per node with everything in LDS needs about 105 LDS reads a node and, at p = 8, a
// 768-thread workgroup of which one fits a CU; here a p = 8 element takes 243 threads and three
// fit.  H and EPB were measured on 20^3 to 32^3 elements (one thread per node, chosen; best of the
// other splits): p = 1: 9.1, 7.2; 7.5 us, p = 2: 26.1, 22.3; 23.2, p = 3: 55.6, 40.5; 41.4,
// p = 4: 126.8, 111.5; 121.6, p = 5: 47.3, 37.9; 39.9, p = 7: 418, 377; 387, p = 8: 215, 141; 236.
// p = 6 takes one node a thread: 96, 76 us on 20^3, 5.3, 5.1 on 4^3, where four threads a column take 72
// and 6.0; the batched launches (WIDE) take four there, which fit their 256-thread workgroups.
template <int N, bool WIDE = false>
struct ColShape {
  static constexpr int N2 = N * N, N3 = N * N * N;
  static constexpr int HS[10] = {0, 0, 2, 3, 2, 3, 6, WIDE ? 4 : 7, 4, 3}, ES[10] = {0, 0, 8, 7, 4, 3, 1, 1, 1, 1};
  static constexpr int H = HS[N], EPB = ES[N];
  static constexpr int KPT = (N + H - 1) / H;
  static constexpr int NR = (6 + H - 1) / H;                   // face tasks per thread
  static constexpr int TE = N2 * H;                            // threads per element
  static constexpr int THREADS = ((EPB * TE + 63) / 64) * 64;
  static constexpr int P = N | 1, V3 = N2 * P, F2 = N * P;     // odd pitches: the lanes that read one
                                                               // column of rows hit distinct banks
  static constexpr bool FULL = EPB * TE == THREADS;
  static constexpr bool UNIH = N2 == 64;                       // a wavefront is one slice of the columns
};

template <typename T>
struct alignas(2 * sizeof(T)) FacePair {
  T a, s;   // a face node's row term without the own flux, and its lifting weight
};

template <int N, typename T, bool WIDE = false>
struct OpSmem {
  using S = ColShape<N, WIDE>;
  T sD[S::N2];                         // D[i][m] at i N + m
  T su[S::EPB][S::V3];                 // u, then the xi_1 fluxes
  T sTr[S::EPB][6 * S::F2 > S::V3 ? 6 * S::F2 : S::V3];   // neighbour traces, then the xi_2 fluxes
  T sF2[S::EPB][S::V3];                // xi_3 fluxes
  FacePair<T> sAS[S::EPB][6][S::N2];
  T sQ[S::EPB][6];                     // weight of the own flux in the row term: interior 1/2, Dirichlet 1
  double red[6];                       // per-wavefront partial sums of the fused dot product
};

// nothing is moved across: keeps the loads of a later stage (and their registers) out of an
// earlier one
__device__ __forceinline__ void stage_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// x is computed here: keeps the compiler from moving a sum to its use, which holds every operand
// in a register until then
template <typename T>
__device__ __forceinline__ void pin(T& x) {
  asm volatile("" : "+v"(x));
}
// s + a0 b0 + a1 b1 + a2 b2 with the roundings spelled out, so that every form of the tile (its own
// launch, one launch over several degrees, persistent) gives the same bits
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
template <typename T>
__device__ __forceinline__ T add3(T s, T a0, T b0, T a1, T b1, T a2, T b2) {
  return fma_(a2, b2, fma_(a1, b1, fma_(a0, b0, s)));
}
template <typename T>
__device__ __forceinline__ T dot3(T a0, T b0, T a1, T b1, T a2, T b2) {
  return fma_(a2, b2, fma_(a1, b1, a0 * b0));
}
// read-only data at a uniform address comes through the scalar cache also after a fence (the
// constant address space has no aliases); vector loads of D and of the neighbour ids held the
// p = 7 operator at 417 us (32^3), scalar ones brought it to 377
template <typename T>
using cptr = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ cptr<T> uniform_ptr(const T* p) {
  return (cptr<T>)(uintptr_t)p;
}

// the neighbour's face node of own face node f under orientation code o (bit 0: exchange the
// face axes, bits 1 and 2: reverse the first and the second)
template <int N>
__device__ __forceinline__ int orient_face_node(int f, int o) {
  const int a = f / N, b = f - (f / N) * N;
  const int x = (o & 1) ? b : a, y = (o & 1) ? a : b;
  return ((o & 2) ? N - 1 - x : x) * N + ((o & 4) ? N - 1 - y : y);
}

// first face axis of face phi (layout: phi 0/1 -> (xi_3, xi_2), 2/3 -> (xi_3, xi_1), 4/5 -> (xi_2, xi_1))
__device__ __forceinline__ int face_axis_first(int phi) { return phi < 4 ? 2 : 1; }

// One tile: EPB elements of one right-hand side (logical block lbr = (element block, right-hand
// side) with the right-hand side fastest, so that the batch of one element reads its geometry while
// it is resident in L2).  Threads without an element load what another thread loads and write
// nothing, so that no load sits behind a branch; the wavefronts of a wider batched workgroup
// (WIDE) beyond THREADS only pass the barriers.
// tid: the thread index (opaque in the persistent batches).
// MIXED: a level of several degrees (per-element offsets; a neighbour of another degree is left
// to the mortar face kernel, whose terms the tile adds through OpArgs::fmapE).
template <int N, typename T, bool ORIENT, bool MIXED, bool WIDE>
__device__ __forceinline__ void sipg_tile(const OpArgs<T>& a, const int lbr, OpSmem<N, T, WIDE>& sm, const int tid) {
  using S = ColShape<N, WIDE>;
  constexpr int N2 = S::N2, N3 = S::N3, H = S::H, KPT = S::KPT, NR = S::NR, TE = S::TE, EPB = S::EPB;
  constexpr int P = S::P, F2 = S::F2;
  constexpr bool CUT = N % H != 0;      // the last slice is short
  constexpr bool ODD = 6 % H != 0;      // the last round of face tasks leaves slices idle
  const bool live = !WIDE || tid < S::THREADS;
  const int nrhs = a.nrhs, mode = a.mode;
  const int lb = lbr / nrhs, rhs = lbr - lb * nrhs;
  const int64_t ndof = a.ndof;
  const T* __restrict__ u = a.u + (int64_t)rhs * ndof;
  const T* __restrict__ g = a.g ? a.g + (int64_t)rhs * ndof : nullptr;
  T* __restrict__ out = a.out + (int64_t)rhs * ndof;
  const T* __restrict__ G = a.G;
  const cptr<T> Dg = uniform_ptr(a.D);
  const T inv_wend = a.inv_wend;
  const int le0 = EPB == 1 ? 0 : tid / TE, t0 = tid - le0 * TE;
  const bool act = S::FULL && !WIDE ? (EPB == 1 || lb * EPB + le0 < a.nel)
                                    : (t0 < TE && le0 < EPB && lb * EPB + le0 < a.nel);
  const int le = EPB == 1 || act ? le0 : 0, t = (S::FULL && !WIDE) || act ? t0 : 0;
  int h = H == 1 ? 0 : t / N2;
  const int col = t - h * N2;
  if constexpr (S::UNIH) h = __builtin_amdgcn_readfirstlane(h);
  const int i = col % N, j = col / N;
  // the thread's q-th node along xi_3, and its r-th face; a thread beyond the last node or face
  // repeats the last one
  auto node = [&](int q) { return CUT ? min(h * KPT + q, N - 1) : h * KPT + q; };
  auto face = [&](int r) { return ODD ? min(r * H + h, 5) : r * H + h; };
  int e = lb * EPB + le;
  if (a.elist) e = a.elist[e];
  if constexpr (EPB == 1) e = __builtin_amdgcn_readfirstlane(e);
  const int64_t base = MIXED ? a.off[e] : (int64_t)e * N3;

  T uv[KPT], pf[NR], gn[NR][3], dn[NR], trv[NR], G6[KPT][6], F[KPT][3], row[KPT], gv[KPT];
  int en[NR], fo[NR];
  int8_t bcv[NR];
  if (live) {
    for (int q = tid; q < N2; q += S::THREADS) sm.sD[q] = a.D[q];
    const int64_t fbase = MIXED ? a.offF[e] : (int64_t)e * 6 * N2;
#pragma unroll
    for (int q = 0; q < KPT; ++q) uv[q] = u[base + node(q) * N2 + col];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int phi = face(r);
      en[r] = S::UNIH && EPB == 1 ? uniform_ptr(a.nbr)[(int64_t)e * 6 + phi] : a.nbr[(int64_t)e * 6 + phi];
      bcv[r] = a.bc[(int64_t)e * 6 + phi];
      pf[r] = a.pen[fbase + phi * N2 + col];
      fo[r] = ORIENT && en[r] >= 0 ? a.nfo[(int64_t)e * 6 + phi] : 0;
      if (MIXED && en[r] >= 0 && a.deg[en[r]] != N - 1) en[r] = -2;
    }
    {
      // the neighbour's node line along its normal and its metric row at the shared face; a face
      // without one reads the element itself and uses nothing of it
      T ln[NR][N];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int phi = face(r);
        const int phio = ORIENT ? (fo[r] & 7) : (phi ^ 1);
        const int f = ORIENT ? orient_face_node<N>(col, fo[r] >> 3) : col;
        const int axo = phio >> 1;
        const int nb = en[r] >= 0 ? en[r] : e;
        const int64_t nbase = MIXED ? a.off[nb] : (int64_t)nb * N3;
        const T* __restrict__ line = u + nbase + face_node<N>(phio, f, 0);
        const int st = axis_stride<N>(axo);
#pragma unroll
        for (int m = 0; m < N; ++m) ln[r][m] = line[m * st];
        const int64_t gi = nbase + face_node<N>(phio, f, (phio & 1) ? N - 1 : 0);
#pragma unroll
        for (int c = 0; c < 3; ++c) gn[r][c] = G[sym_index(axo, c) * ndof + gi];
      }
      if (act) {
#pragma unroll
        for (int q = 0; q < KPT; ++q)
          if (!CUT || h * KPT + q < N) sm.su[le][(node(q) * N + j) * P + i] = uv[q];
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int phi = face(r);
        const int endo = ((ORIENT ? fo[r] : (phi ^ 1)) & 1) ? N - 1 : 0;
        T s = 0, l0 = ln[r][0], l1 = ln[r][N - 1];
#pragma unroll
        for (int m = 0; m < N; ++m) s = fma_(endo ? Dg[(N - 1) * N + m] : Dg[m], ln[r][m], s);
        dn[r] = s;
        if constexpr (ORIENT) {   // both ends stay in registers: a selected index would spill the line
          pin(l0);
          pin(l1);
        }
        trv[r] = endo ? l1 : l0;
        pin(dn[r]);
        pin(trv[r]);
        if (act && (!ODD || r * H + h < 6)) sm.sTr[le][phi * F2 + j * P + i] = trv[r];
      }
    }
    stage_fence();
    // the metric arrives while the derivatives are taken
#pragma unroll
    for (int q = 0; q < KPT; ++q)
#pragma unroll
      for (int c = 0; c < 6; ++c) G6[q][c] = G[c * ndof + base + node(q) * N2 + col];
  }
  __syncthreads();

  if (live) {
    // reference derivatives of the own nodes and tangential derivatives of the neighbours'
    // traces, one direction (and one row of D) after another
    T dlast[NR], dfirst[NR];
    {
      T Dr[N];
#pragma unroll
      for (int m = 0; m < N; ++m) Dr[m] = sm.sD[i * N + m];
#pragma unroll
      for (int q = 0; q < KPT; ++q) {
        T s = 0;
#pragma unroll
        for (int m = 0; m < N; ++m) s = fma_(Dr[m], sm.su[le][(node(q) * N + j) * P + m], s);
        F[q][0] = s;
        pin(F[q][0]);
        if (q & 1) stage_fence();
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        T s = 0;
#pragma unroll
        for (int m = 0; m < N; ++m) s = fma_(Dr[m], sm.sTr[le][face(r) * F2 + j * P + m], s);
        dlast[r] = s;
        pin(dlast[r]);
        stage_fence();
      }
#pragma unroll
      for (int m = 0; m < N; ++m) Dr[m] = sm.sD[j * N + m];
#pragma unroll
      for (int q = 0; q < KPT; ++q) {
        T s = 0;
#pragma unroll
        for (int m = 0; m < N; ++m) s = fma_(Dr[m], sm.su[le][(node(q) * N + m) * P + i], s);
        F[q][1] = s;
        pin(F[q][1]);
        if (q & 1) stage_fence();
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        T s = 0;
#pragma unroll
        for (int m = 0; m < N; ++m) s = fma_(Dr[m], sm.sTr[le][face(r) * F2 + m * P + i], s);
        dfirst[r] = s;
        pin(dfirst[r]);
        stage_fence();
      }
#pragma unroll
      for (int q = 0; q < KPT; ++q) F[q][2] = 0;
#pragma unroll
      for (int m = 0; m < N; ++m) {
        const T um = sm.su[le][(m * N + j) * P + i];
#pragma unroll
        for (int q = 0; q < KPT; ++q) F[q][2] = fma_(S::UNIH ? Dg[node(q) * N + m] : sm.sD[node(q) * N + m], um, F[q][2]);
      }
#pragma unroll
      for (int q = 0; q < KPT; ++q) pin(F[q][2]);
    }
    stage_fence();
    // face terms that need no flux of the own element
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int phi = r * H + h, ax = phi >> 1;
      if (ODD && phi > 5) continue;
      const int vi = face_node<N>(phi, col, (phi & 1) ? N - 1 : 0);
      const T uo = sm.su[le][(vi / N) * P + vi % N];
      T A = 0, sig = 0, fq = 0;
      if (en[r] >= 0) {
        T du0, du1, du2, qn;   // the neighbour's reference derivatives and outward flux
        if constexpr (ORIENT) {
          // along its normal from its node line, along its face axes from the own face grid
          // through the orientation
          const int phio = fo[r] & 7, o = fo[r] >> 3;
          const T dA = ((o & 2) ? T(-1) : T(1)) * ((o & 1) ? dlast[r] : dfirst[r]);
          const T dB = ((o & 4) ? T(-1) : T(1)) * ((o & 1) ? dfirst[r] : dlast[r]);
          const int an = phio >> 1, af = face_axis_first(phio);   // the third axis takes dB
          du0 = an == 0 ? dn[r] : (af == 0 ? dA : dB);
          du1 = an == 1 ? dn[r] : (af == 1 ? dA : dB);
          du2 = an == 2 ? dn[r] : (af == 2 ? dA : dB);
          qn = ((phio & 1) ? T(1) : T(-1)) * inv_wend * dot3(gn[r][0], du0, gn[r][1], du1, gn[r][2], du2);
        } else {
          if (ax == 0) { du0 = dn[r]; du1 = dlast[r]; du2 = dfirst[r]; }
          else if (ax == 1) { du0 = dlast[r]; du1 = dn[r]; du2 = dfirst[r]; }
          else { du0 = dlast[r]; du1 = dfirst[r]; du2 = dn[r]; }
          qn = ((phi & 1) ? T(-1) : T(1)) * inv_wend * dot3(gn[r][0], du0, gn[r][1], du1, gn[r][2], du2);
        }
        const T jmp = uo - trv[r];
        A = fma_(pf[r], jmp, T(0.5) * qn);
        sig = T(-0.5) * jmp;
        fq = T(0.5);
      } else if (en[r] == -1 && bcv[r] == 1) {   // Dirichlet: 2 mu nu omega s u - q, lifting -u
        A = pf[r] * uo;
        sig = -uo;
        fq = 1;
      }
      if (act) {
        sm.sAS[le][phi][j * N + i] = FacePair<T>{A, sig};
        if (col == 0) sm.sQ[le][phi] = fq;
      }
    }
    stage_fence();
    // contravariant fluxes F_b = sum_c G_bc d_c u
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
      const T d0 = F[q][0], d1 = F[q][1], d2 = F[q][2];
      F[q][0] = dot3(G6[q][0], d0, G6[q][1], d1, G6[q][2], d2);
      F[q][1] = dot3(G6[q][1], d0, G6[q][3], d1, G6[q][4], d2);
      F[q][2] = dot3(G6[q][2], d0, G6[q][4], d1, G6[q][5], d2);
      pin(F[q][0]);
      pin(F[q][1]);
      pin(F[q][2]);
    }
  }
  __syncthreads();

  if (live) {
    // the owner of a face node adds its row term and lifts
    const bool onx = i == 0 || i == N - 1, ony = j == 0 || j == N - 1;
    const int px = i == 0 ? 0 : 1, py = j == 0 ? 2 : 3;
    const T wx = i == 0 ? -inv_wend : inv_wend, wy = j == 0 ? -inv_wend : inv_wend;
    T fx = 0, fy = 0;
    if (onx) fx = sm.sQ[le][px] * wx;
    if (ony) fy = sm.sQ[le][py] * wy;
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
      const int k = h * KPT + q;
      row[q] = 0;
      if (CUT && k >= N) continue;
      T sx = 0, sy = 0, sz = 0;
      if (onx) {
        const FacePair<T> f = sm.sAS[le][px][k * N + j];
        row[q] += fma_(-fx, F[q][0], f.a);
        sx = f.s * wx;
      }
      if (ony) {
        const FacePair<T> f = sm.sAS[le][py][k * N + i];
        row[q] += fma_(-fy, F[q][1], f.a);
        sy = f.s * wy;
      }
      if (k == 0 || k == N - 1) {
        const int pz = k == 0 ? 4 : 5;
        const T wz = k == 0 ? -inv_wend : inv_wend;
        const FacePair<T> f = sm.sAS[le][pz][j * N + i];
        row[q] += fma_(-(sm.sQ[le][pz] * wz), F[q][2], f.a);
        sz = f.s * wz;
      }
      F[q][0] = add3(F[q][0], sx, G6[q][0], sy, G6[q][1], sz, G6[q][2]);
      F[q][1] = add3(F[q][1], sx, G6[q][1], sy, G6[q][3], sz, G6[q][4]);
      F[q][2] = add3(F[q][2], sx, G6[q][2], sy, G6[q][4], sz, G6[q][5]);
      if constexpr (MIXED) {
        // a face to another degree: its row and lifting terms from the mortar face kernel
        if (a.fmapE) {
          auto mortar = [&](int phi, int ff) {
            const int kf = a.fmapE[(int64_t)e * 6 + phi];
            if (kf < 0) return;
            const T* __restrict__ m = a.fres + (int64_t)rhs * a.fres_stride + (int64_t)kf * kMortarFaceRes;
            row[q] += m[ff];
            F[q][0] += m[81 + ff];
            F[q][1] += m[162 + ff];
            F[q][2] += m[243 + ff];
          };
          if (onx) mortar(px, k * N + j);
          if (ony) mortar(py, k * N + i);
          if (k == 0 || k == N - 1) mortar(k == 0 ? 4 : 5, j * N + i);
        }
      }
      if (act) {
        const int l = (k * N + j) * P + i;
        sm.su[le][l] = F[q][0];
        sm.sTr[le][l] = F[q][1];
        sm.sF2[le][l] = F[q][2];
      }
    }
  }
  __syncthreads();

  double pq = 0;
  if (live) {
#pragma unroll
    for (int q = 0; q < KPT; ++q) gv[q] = mode == 0 ? g[base + node(q) * N2 + col] : T(0);
    T Dr[N];
#pragma unroll
    for (int m = 0; m < N; ++m) Dr[m] = sm.sD[m * N + i];
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
#pragma unroll
      for (int m = 0; m < N; ++m) row[q] = fma_(Dr[m], sm.su[le][(node(q) * N + j) * P + m], row[q]);
      pin(row[q]);
      if (q & 1) stage_fence();
    }
    stage_fence();
#pragma unroll
    for (int m = 0; m < N; ++m) Dr[m] = sm.sD[m * N + j];
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
#pragma unroll
      for (int m = 0; m < N; ++m) row[q] = fma_(Dr[m], sm.sTr[le][(node(q) * N + m) * P + i], row[q]);
      pin(row[q]);
      if (q & 1) stage_fence();
    }
    stage_fence();
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const T fm = sm.sF2[le][(m * N + j) * P + i];
#pragma unroll
      for (int q = 0; q < KPT; ++q) row[q] = fma_(S::UNIH ? Dg[m * N + node(q)] : sm.sD[m * N + node(q)], fm, row[q]);
    }
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
      if (!act || (CUT && h * KPT + q >= N)) continue;
      const int64_t o = base + node(q) * N2 + col;
      T acc = row[q];
      if (a.WJ) acc = fma_(a.kappa * a.WJ[o], uv[q], acc);
      out[o] = mode == 0 ? gv[q] - acc : acc;
      pq += (double)uv[q] * (double)acc;
    }
  }
  if (!MIXED && a.dotp) {
    // u^T (A u) over the tile: the wavefronts' sums in order (deterministic)
    pq = wave_sum(pq);
    if ((tid & 63) == 0) sm.red[tid >> 6] = pq;
    __syncthreads();
    if (tid == 0) {
      double s = 0;
      for (int w = 0; w < S::THREADS / 64; ++w) s += sm.red[w];
      a.dotp[(int64_t)rhs * ((a.nel + EPB - 1) / EPB) + lb] = s;
    }
  }
}

template <int N, typename T, bool ORIENT, bool MIXED>
__global__ void __launch_bounds__(ColShape<N>::THREADS)
sipg_apply_kernel(OpArgs<T> a) {
  using S = ColShape<N>;
  __shared__ OpSmem<N, T> sm;
  const int lbr = xcd_block(((a.nel + S::EPB - 1) / S::EPB) * a.nrhs);
  if (lbr < 0) return;
  sipg_tile<N, T, ORIENT, MIXED, false>(a, lbr, sm, threadIdx.x);
}

template <int N, typename T>
void launch_sipg(const OpArgs<T>& a, hipStream_t st) {
  using S = ColShape<N>;
  const int nb = ((a.nel + S::EPB - 1) / S::EPB) * a.nrhs;
  const dim3 gr(xcd_grid(nb)), bl(S::THREADS);
  if (a.nfo) hipLaunchKernelGGL((sipg_apply_kernel<N, T, true, false>), gr, bl, 0, st, a);
  else if (a.off) hipLaunchKernelGGL((sipg_apply_kernel<N, T, false, true>), gr, bl, 0, st, a);
  else hipLaunchKernelGGL((sipg_apply_kernel<N, T, false, false>), gr, bl, 0, st, a);
}

// largest tile workspace and widest tile of the degrees with n <= N
template <typename T, int N>
constexpr size_t op_smem_upto() {
  if constexpr (N < 2) {
    return 0;
  } else {
    constexpr size_t a = sizeof(OpSmem<N, T, true>), b = op_smem_upto<T, N - 1>();
    return a > b ? a : b;
  }
}
template <int N>
constexpr int op_threads_upto() {
  if constexpr (N < 2) {
    return 0;
  } else {
    constexpr int a = ColShape<N, true>::THREADS, b = op_threads_upto<N - 1>();
    return a > b ? a : b;
  }
}

// all degrees up to NMAX - 1 in one launch; the workgroup is the widest tile's
template <int NMAX, typename T, bool PERSIST>
__global__ void __launch_bounds__(op_threads_upto<NMAX>())
sipg_batched_kernel(OpArgs<T> a, const BucketDesc<T>* __restrict__ bd, int nb, int ntiles) {
  __shared__ __align__(16) char smem[op_smem_upto<T, NMAX>()];
  // tiles dealt round-robin over the XCDs (the hardware order): the work list runs from the
  // largest degree to the smallest, and contiguous ranges per XCD would leave one XCD all
  // the large tiles.  The persistent form (fewer workgroups than tiles) strides through the
  // list, with a barrier between tiles for the shared memory.  It takes the thread index
  // through an opaque register copy in every tile, so that no degree branch's index arithmetic
  // is hoisted above the loop and kept live across it.  Constants of the branches still are: at p = 8
  // in FP64 it takes 159 registers, the one-tile form 136, three waves per SIMD both.
  auto tile = [&](int t) {
    int tid = threadIdx.x;
    if constexpr (PERSIST) asm volatile("v_mov_b32 %0, %1" : "=v"(tid) : "v"(tid));
    const int k = find_bucket(bd, nb, kStageOp, t);
    OpArgs<T> x = a;
    x.nel = bd[k].nel;
    x.elist = bd[k].elist;
    x.D = bd[k].D;
    x.inv_wend = bd[k].inv_wend;
    const int lbr = t - bd[k].tile0[kStageOp];
    switch (bd[k].p) {
#define DGFAS_OPB(P)                                                                        \
  case P:                                                                                   \
    if constexpr (P + 1 <= NMAX) sipg_tile<P + 1, T, false, true, true>(x, lbr, *reinterpret_cast<OpSmem<P + 1, T, true>*>(smem), tid); \
    break;
      DGFAS_OPB(1) DGFAS_OPB(2) DGFAS_OPB(3) DGFAS_OPB(4) DGFAS_OPB(5) DGFAS_OPB(6) DGFAS_OPB(7) DGFAS_OPB(8)
#undef DGFAS_OPB
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

int stage_tiles(int stage, int p, int nel, int nrhs, int pmax) {
  if (stage == kStageSolve) {   // degrees 1 and 2: as many subdomains as columns fit the workgroup
    const int spw = p <= 2 ? stage_threads(kStageSolve, pmax) / ((p + 3) * (p + 3)) : 1;
    return (nel * nrhs + spw - 1) / spw;
  }
  const int epb = stage == kStageOp ? ColShape<2>::ES[p + 1] : kAddElems[p + 1];   // elements per tile
  return ((nel + epb - 1) / epb) * nrhs;
}

int stage_threads(int stage, int pmax) {
  if (stage == kStageSolve) return pmax + 3 >= 9 ? 128 : 64;   // overlap 1: ns^2 lines, rounded to waves
  return 256;   // the operator's widest tile (of every NMAX that is launched) and the overlap add's
}
static_assert(op_threads_upto<6>() == 256 && op_threads_upto<9>() == 256, "workgroup of the batched operator");

template <typename T>
void sipg_apply_batched(int pmax, const OpArgs<T>& a, const BucketDesc<T>* bd, const BatchLaunch& l, hipStream_t st) {
  if (l.ntiles <= 0) return;
  const dim3 g(l.grid), b(stage_threads(kStageOp, pmax));
#define DGFAS_OPL(NM)                                                                                     \
  if (l.persistent) hipLaunchKernelGGL((sipg_batched_kernel<NM, T, true>), g, b, 0, st, a, bd, l.nb, l.ntiles); \
  else hipLaunchKernelGGL((sipg_batched_kernel<NM, T, false>), g, b, 0, st, a, bd, l.nb, l.ntiles);
  if (pmax <= 5) { DGFAS_OPL(6) }
  else if (pmax == 6) { DGFAS_OPL(7) }
  else if (pmax == 7) { DGFAS_OPL(8) }
  else { DGFAS_OPL(9) }
#undef DGFAS_OPL
}

template void sipg_apply_batched<double>(int, const OpArgs<double>&, const BucketDesc<double>*, const BatchLaunch&,
                                         hipStream_t);
template void sipg_apply_batched<float>(int, const OpArgs<float>&, const BucketDesc<float>*, const BatchLaunch&,
                                        hipStream_t);

template <typename T>
void sipg_apply(int p, const OpArgs<T>& a, hipStream_t st) {
  switch (p) {
    case 1: launch_sipg<2, T>(a, st); break;
    case 2: launch_sipg<3, T>(a, st); break;
    case 3: launch_sipg<4, T>(a, st); break;
    case 4: launch_sipg<5, T>(a, st); break;
    case 5: launch_sipg<6, T>(a, st); break;
    case 6: launch_sipg<7, T>(a, st); break;
    case 7: launch_sipg<8, T>(a, st); break;
    case 8: launch_sipg<9, T>(a, st); break;
    default: break;
  }
}

template void sipg_apply<double>(int, const OpArgs<double>&, hipStream_t);
template void sipg_apply<float>(int, const OpArgs<float>&, hipStream_t);

// ---------------------------------------------------------------------------
// Geometry (one-time): G_bc = w J nu grad xi_b . grad xi_c, w J, omega*s at face
// nodes (from the cross product of the two tangential columns of the Jacobian,
// i.e. tangential derivatives only), element volume and face areas, and the
// linear Legendre coefficients of the map (surrogate cuboid, Sec. 4.3.1).
template <int N>
__global__ void __launch_bounds__(OpShape<N>::THREADS)
geometry_kernel(GeoArgs g, const double* __restrict__ Dg, const double* __restrict__ w1,
                const double* __restrict__ x1, double nu) {
  using S = OpShape<N>;
  constexpr int N2 = S::N2, N3 = S::N3, EPB = S::EPB;
  const double* __restrict__ X = g.X;
  double* __restrict__ G = g.G;
  double* __restrict__ WJ = g.WJ;
  double* __restrict__ ws = g.ws;
  double* __restrict__ vol = g.vol;
  double* __restrict__ area = g.area;
  double* __restrict__ lin = g.lin;
  const int lb = blockIdx.x;
  const int tid = threadIdx.x;
  const int le = tid / N3;
  const int node = tid - le * N3;
  const int li = lb * EPB + le;
  const bool active = (le < EPB) && (li < g.nel);
  const int e = active ? (g.elist ? g.elist[li] : li) : 0;
  const int64_t base = g.off ? g.off[e] : (int64_t)e * N3;
  const int64_t fbase = g.offF ? g.offF[e] : (int64_t)e * 6 * N2;
  __shared__ double sX[EPB][3][N3];
  __shared__ double sWJ[EPB][N3];
  __shared__ double sWJnu[EPB][N3];
  __shared__ double sws[EPB][6][N2];
  if (active)
    for (int a = 0; a < 3; ++a) sX[le][a][node] = X[3 * base + (int64_t)a * N3 + node];
  __syncthreads();
  const int i = node % N, j = (node / N) % N, k = node / N2;
  if (active) {
    double J[3][3];
    for (int a = 0; a < 3; ++a) {
      double d0 = 0, d1 = 0, d2 = 0;
      for (int m = 0; m < N; ++m) {
        d0 += Dg[i * N + m] * sX[le][a][(k * N + j) * N + m];
        d1 += Dg[j * N + m] * sX[le][a][(k * N + m) * N + i];
        d2 += Dg[k * N + m] * sX[le][a][(m * N + j) * N + i];
      }
      J[a][0] = d0; J[a][1] = d1; J[a][2] = d2;
    }
    // cofactor matrix C[a][b] = d det / d J[a][b]; column b of C = J grad(xi_b) (times det)
    double C[3][3];
    C[0][0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
    C[0][1] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
    C[0][2] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
    C[1][0] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
    C[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
    C[1][2] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
    C[2][0] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
    C[2][1] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
    C[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
    const double det = J[0][0] * C[0][0] + J[0][1] * C[0][1] + J[0][2] * C[0][2];
    if (!(det > 0)) atomicOr(g.bad, 1);
    const double wq = w1[i] * w1[j] * w1[k];
    // grad xi_b = C[:, b] / det  ->  G_bc = w nu (C[:,b] . C[:,c]) / det, nu at the node
    const int64_t ndof = g.ndof, gi = base + node;
    const double nuq = g.nun ? g.nun[gi] : nu;
    const double sc = wq * nuq / det;
    double Gb[6];
    Gb[0] = sc * (C[0][0] * C[0][0] + C[1][0] * C[1][0] + C[2][0] * C[2][0]);
    Gb[1] = sc * (C[0][0] * C[0][1] + C[1][0] * C[1][1] + C[2][0] * C[2][1]);
    Gb[2] = sc * (C[0][0] * C[0][2] + C[1][0] * C[1][2] + C[2][0] * C[2][2]);
    Gb[3] = sc * (C[0][1] * C[0][1] + C[1][1] * C[1][1] + C[2][1] * C[2][1]);
    Gb[4] = sc * (C[0][1] * C[0][2] + C[1][1] * C[1][2] + C[2][1] * C[2][2]);
    Gb[5] = sc * (C[0][2] * C[0][2] + C[1][2] * C[1][2] + C[2][2] * C[2][2]);
    for (int c = 0; c < 6; ++c) G[c * ndof + gi] = Gb[c];
    WJ[gi] = wq * det;
    sWJ[le][node] = wq * det;
    sWJnu[le][node] = wq * det * nuq;
    // face nodes: omega * s with N = dx/dxi_t1 x dx/dxi_t2 (tangential columns of J)
    const int idx[3] = {i, j, k};
    for (int ax = 0; ax < 3; ++ax) {
      const int t1 = (ax + 1) % 3, t2 = (ax + 2) % 3;
      if (idx[ax] != 0 && idx[ax] != N - 1) continue;
      const double nx = J[1][t1] * J[2][t2] - J[2][t1] * J[1][t2];
      const double ny = J[2][t1] * J[0][t2] - J[0][t1] * J[2][t2];
      const double nz = J[0][t1] * J[1][t2] - J[1][t1] * J[0][t2];
      const double s = sqrt(nx * nx + ny * ny + nz * nz) * w1[idx[t1]] * w1[idx[t2]];
      int f;
      if (ax == 0) f = k * N + j;
      else if (ax == 1) f = k * N + i;
      else f = j * N + i;
      if (idx[ax] == 0) sws[le][2 * ax][f] = s;
      if (idx[ax] == N - 1) sws[le][2 * ax + 1][f] = s;
    }
  }
  __syncthreads();
  // per-element sums: tasks 0..5 face areas, 6 volume, 7..15 linear Legendre coefficients
  for (int task = node; active && task < 16; task += N3) {
    if (task < 6) {
      double a = 0;
      for (int f = 0; f < N2; ++f) a += sws[le][task][f];
      area[(int64_t)e * 6 + task] = a;
      for (int f = 0; f < N2; ++f) ws[fbase + task * N2 + f] = sws[le][task][f];
    } else if (task == 6) {
      double v = 0, vn = 0;
      for (int t = 0; t < N3; ++t) {
        v += sWJ[le][t];
        vn += sWJnu[le][t];
      }
      vol[e] = v;
      if (g.nuavg) g.nuavg[e] = vn / v;
    } else {
      // coefficient of L_1(xi_b) L_0 L_0 in the Legendre expansion of coordinate a
      const int q = task - 7, a = q / 3, b = q % 3;
      double s = 0;
      if (N > 2) {   // GLL quadrature is exact for x * xi_b when p >= 2
        for (int t = 0; t < N3; ++t) {
          const int ti = t % N, tj = (t / N) % N, tk = t / N2;
          const int idx[3] = {ti, tj, tk};
          s += w1[ti] * w1[tj] * w1[tk] * sX[le][a][t] * x1[idx[b]];
        }
        s *= 0.375;
      } else {       // p = 1: mean half-difference along b of the trilinear map
        for (int t = 0; t < N3; ++t) {
          const int ti = t % N, tj = (t / N) % N, tk = t / N2;
          const int idx[3] = {ti, tj, tk};
          s += (idx[b] == 1 ? 0.125 : -0.125) * sX[le][a][t];
        }
      }
      lin[(int64_t)e * 9 + q] = s;
    }
  }
}

template <int N>
void launch_geometry(const GeoArgs& g, const double* D, const double* w, const double* x, double nu, hipStream_t st) {
  using S = OpShape<N>;
  const int nb = (g.nel + S::EPB - 1) / S::EPB;
  if (nb > 0) hipLaunchKernelGGL((geometry_kernel<N>), dim3(nb), dim3(S::THREADS), 0, st, g, D, w, x, nu);
}

void geometry(int p, const GeoArgs& g, const double* D, const double* w, const double* x, double nu,
              hipStream_t st) {
  switch (p) {
    case 1: launch_geometry<2>(g, D, w, x, nu, st); break;
    case 2: launch_geometry<3>(g, D, w, x, nu, st); break;
    case 3: launch_geometry<4>(g, D, w, x, nu, st); break;
    case 4: launch_geometry<5>(g, D, w, x, nu, st); break;
    case 5: launch_geometry<6>(g, D, w, x, nu, st); break;
    case 6: launch_geometry<7>(g, D, w, x, nu, st); break;
    case 7: launch_geometry<8>(g, D, w, x, nu, st); break;
    case 8: launch_geometry<9>(g, D, w, x, nu, st); break;
    default: break;
  }
}

// node of face phi at face-node index f (layout of face_node) and normal index t, degree n - 1
__device__ __forceinline__ int face_node_n(int n, int phi, int f, int t) {
  const int a = f / n, b = f % n, ax = phi >> 1;
  if (ax == 0) return (a * n + b) * n + t;
  if (ax == 1) return (a * n + t) * n + b;
  return (t * n + a) * n + b;
}

// Penalty factor per element-face node: interior mu_F max(nu-, nu+) omega s with
// mu_F = mu_star avg(p(p+1)/(2 h_perp)) over the two sides (each with its own degree),
// Dirichlet 2 mu nu omega s, Neumann 0; h_perp = vol / area (eq. helmholtz:dgm).  With a nodal
// nu (one degree), nu- and nu+ are the two sides' values at the face node.
// muf[e][phi] = mu_F nu (Dirichlet: 2 mu nu) for the face integration on mixed-degree faces.
__global__ void penalty_kernel(int E, int p, const int* __restrict__ deg, const int64_t* __restrict__ offF,
                               double mu_star, double nu, const double* __restrict__ nun,
                               const int* __restrict__ nbr, const int8_t* __restrict__ nfo,
                               const int8_t* __restrict__ bc, const double* __restrict__ vol,
                               const double* __restrict__ area, const double* __restrict__ ws,
                               double* __restrict__ pen, double* __restrict__ muf) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)E * 6) return;
  const int e = (int)(t / 6), phi = (int)(t % 6);
  const int pe = deg ? deg[e] : p;
  const int N2 = (pe + 1) * (pe + 1);
  const double own = pe * (pe + 1) / (2.0 * (vol[e] / area[t]));
  const int en = nbr[t];
  // the neighbour's face and the relative orientation (unstructured meshes), else aligned
  const int phio = nfo && en >= 0 ? (nfo[t] & 7) : (phi ^ 1);
  const int ori = nfo && en >= 0 ? (nfo[t] >> 3) : 0;
  double fac = 0.0;
  if (en >= 0) {
    const int pn = deg ? deg[en] : p;
    const double oth = pn * (pn + 1) / (2.0 * (vol[en] / area[(int64_t)en * 6 + phio]));
    fac = mu_star * 0.5 * (own + oth);
  } else if (bc[t] == 1) {
    fac = 2.0 * mu_star * own;
  }
  if (muf) muf[t] = fac * nu;
  const int64_t fb = (offF ? offF[e] : (int64_t)e * 6 * N2) + (int64_t)phi * N2;
  if (!nun) {
    for (int f = 0; f < N2; ++f) pen[fb + f] = fac * nu * ws[fb + f];
    return;
  }
  const int n = pe + 1, N3 = N2 * n;
  const int end = (phi & 1) ? n - 1 : 0, endo = (phio & 1) ? n - 1 : 0;
  for (int f = 0; f < N2; ++f) {
    double nf = nun[(int64_t)e * N3 + face_node_n(n, phi, f, end)];
    if (en >= 0) {
      const int a = f / n, b = f % n;
      const int x = (ori & 1) ? b : a, y = (ori & 1) ? a : b;
      const int fo = ((ori & 2) ? n - 1 - x : x) * n + ((ori & 4) ? n - 1 - y : y);
      nf = fmax(nf, nun[(int64_t)en * N3 + face_node_n(n, phio, fo, endo)]);
    }
    pen[fb + f] = fac * nf * ws[fb + f];
  }
}

void penalty(int E, int p, const int* deg, const int64_t* offF, double mu_star, double nu, const double* nun,
             const int* nbr, const int8_t* nfo, const int8_t* bc, const double* vol, const double* area,
             const double* ws, double* pen, double* muf, hipStream_t st) {
  const int64_t n = (int64_t)E * 6;
  hipLaunchKernelGGL(penalty_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, E, p, deg, offF, mu_star,
                     nu, nun, nbr, nfo, bc, vol, area, ws, pen, muf);
}

}  // namespace dgfas

namespace dgfas {

// Right-hand side of eq. helmholtz:system:
//   b = w J f + Dirichlet faces (2 mu nu omega s u_D at the face node, lifting
//   -nu omega s u_D (n . grad phi_q)) + Neumann faces (omega s q_N).
template <int N>
__global__ void __launch_bounds__(OpShape<N>::THREADS)
rhs_kernel(RhsArgs r, const double* __restrict__ Dg, double inv_wend) {
  using S = OpShape<N>;
  constexpr int N2 = S::N2, N3 = S::N3, EPB = S::EPB;
  const double* __restrict__ f = r.f;
  const double* __restrict__ uD = r.uD;
  const double* __restrict__ qN = r.qN;
  double* __restrict__ b = r.b;
  const double* __restrict__ G = r.G;
  const double* __restrict__ WJ = r.WJ;
  const double* __restrict__ pen = r.pen;
  const double* __restrict__ ws = r.ws;
  const int* __restrict__ nbr = r.nbr;
  const int8_t* __restrict__ bc = r.bc;
  const int lb = blockIdx.x;
  const int tid = threadIdx.x;
  const int le = tid / N3, node = tid - le * N3;
  const int li = lb * EPB + le;
  const bool active = (le < EPB) && (li < r.nel);
  const int e = active ? (r.elist ? r.elist[li] : li) : 0;
  __shared__ double sD[N2];
  __shared__ double sL[EPB][3][N3];
  __shared__ double sRow[EPB][N3];
  for (int t = tid; t < N2; t += S::THREADS) sD[t] = Dg[t];
  const int64_t base = r.off ? r.off[e] : (int64_t)e * N3, ndof = r.ndof;
  const int64_t fbase = r.offF ? r.offF[e] : (int64_t)e * 6 * N2;
  if (active) {
    sL[le][0][node] = sL[le][1][node] = sL[le][2][node] = 0.0;
    sRow[le][node] = 0.0;
  }
  __syncthreads();
  for (int ax = 0; ax < 3; ++ax) {
    if (active) {
      for (int t = node; t < 2 * N2; t += N3) {
        const int s = t / N2, fn = t - s * N2;
        const int phi = 2 * ax + s;
        if (nbr[(int64_t)e * 6 + phi] >= 0) continue;
        const int vi = face_node<N>(phi, fn, (phi & 1) ? N - 1 : 0);
        const int8_t code = bc[(int64_t)e * 6 + phi];
        if (code == 1 && uD) {
          const double ud = uD[base + vi];
          const double sgn = (phi & 1) ? 1.0 : -1.0;
          sRow[le][vi] += pen[fbase + phi * N2 + fn] * ud;
          for (int c = 0; c < 3; ++c) sL[le][c][vi] += -ud * sgn * inv_wend * G[sym_index(ax, c) * ndof + base + vi];
        } else if (code == 2 && qN) {
          sRow[le][vi] += ws[fbase + phi * N2 + fn] * qN[base + vi];
        }
      }
    }
    __syncthreads();
  }
  if (active) {
    const int i = node % N, j = (node / N) % N, k = node / N2;
    double acc = WJ[base + node] * f[base + node] + sRow[le][node];
    for (int m = 0; m < N; ++m) {
      acc += sD[m * N + i] * sL[le][0][(k * N + j) * N + m];
      acc += sD[m * N + j] * sL[le][1][(k * N + m) * N + i];
      acc += sD[m * N + k] * sL[le][2][(m * N + j) * N + i];
    }
    b[base + node] = acc;
  }
}

template <int N>
void launch_rhs(const RhsArgs& r, const double* D, double inv_wend, hipStream_t st) {
  using S = OpShape<N>;
  const int nb = (r.nel + S::EPB - 1) / S::EPB;
  if (nb > 0) hipLaunchKernelGGL((rhs_kernel<N>), dim3(nb), dim3(S::THREADS), 0, st, r, D, inv_wend);
}

void rhs(int p, const RhsArgs& r, const double* D, double inv_wend, hipStream_t st) {
  switch (p) {
    case 1: launch_rhs<2>(r, D, inv_wend, st); break;
    case 2: launch_rhs<3>(r, D, inv_wend, st); break;
    case 3: launch_rhs<4>(r, D, inv_wend, st); break;
    case 4: launch_rhs<5>(r, D, inv_wend, st); break;
    case 5: launch_rhs<6>(r, D, inv_wend, st); break;
    case 6: launch_rhs<7>(r, D, inv_wend, st); break;
    case 7: launch_rhs<8>(r, D, inv_wend, st); break;
    case 8: launch_rhs<9>(r, D, inv_wend, st); break;
    default: break;
  }
}

}  // namespace dgfas
