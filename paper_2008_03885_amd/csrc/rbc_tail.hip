// rbc_tail.hip -- red-black coarsening: the levels from a standard level of side 65 or 33
// down to the 17^2 coarsest one, resident in the LDS of one workgroup.
//
// What bounds these levels is the number of phases between barriers and the latency of one
// phase, so nothing of them touches memory between the top level's first load and its last
// store, and a phase is short: a thread owns the same points on every level (a 2 x 2 cell
// of a standard level; on the rotated level below, the cell's two C points, which are that
// level's F and C point), keeps their values and right-hand sides in registers, and reads
// only its neighbours' from LDS.
//   Standard level of side N, cells (p, k), p, k < M = (N-1)/2: with i = 2p+1, j = 2k+1
//     C1 = (i, j), F1 = (i, j+1), F2 = (i+1, j), C2 = (i+1, j+1)
//   rotated level of the same side: F = (i, j) = C1's place, C = (i+1, j+1) = C2's place.
// One array per kind of point, each with a frame of one cell, so that every neighbour is at
// a constant offset; row and column 0 of the grid are the frame cells before the first (p =
// -1, k = -1), row and column N-1 belong to the last cells.  Each array has two buffers: a
// partial step writes the other one (its same-colour neighbours are read old), so a step
// takes one barrier.
//
// The 17^2 level is solved by sine transforms (its compact symmetric stencil is diagonal in
// the sine modes): four passes over 225 values instead of a product with a 225 x 225
// inverse streamed from L2 (12 us of the 35 us the general tail took from side 33).
//
// Measured (MI355X, kernel trace of solves, G1 V(1,1)): 14.5 us a launch from side 65 with its
// 17^2 solve, in place of the general tail from side 33 (28 to 35 us) and four passes (27 us);
// 257^2 solve 1171 -> 769 us, 4097^2 6.05 -> 5.57 ms.
#include <cmath>
#include <vector>

#include "mg_internal.h"
#include "rbc_passes.h"

namespace mgk {
namespace {

constexpr int kQ = 15, kM0 = kQ * kQ;

template <int N>
struct Dim {
  static constexpr int M = (N - 1) / 2, PW = M + 2, SZ = (M + 2) * PW;
};

// One standard level.
template <int N>
struct Std {
  static constexpr int M = Dim<N>::M, PW = Dim<N>::PW, SZ = Dim<N>::SZ;
  enum { C1, F1, F2, C2 };
  double u[4], f[4];
  double *cell;  // this thread's cell in buffer 0 of the first array
  int wf, wc;    // current buffers of the F and of the C arrays
  bool owner, ki, pi;  // the cell's second column / row is interior
  int p, k;

  __device__ __forceinline__ void init(double *base) {
    const int t = threadIdx.x;
    owner = t < M * M;
    k = t % M;
    p = t / M;
    ki = k < M - 1;
    pi = p < M - 1;
    cell = base + (owner ? (p + 1) * PW + k + 1 : PW + 1);
    wf = wc = 0;
  }
  __device__ __forceinline__ double *arr(int q, int w) const { return cell + (2 * q + w) * SZ; }
  __device__ __forceinline__ const double *cur(int q) const { return arr(q, q == F1 || q == F2 ? wf : wc); }
  __device__ __forceinline__ bool act(int q) const { return (q == C1 || q == F2 || ki) && (q == C1 || q == F1 || pi); }
  __device__ __forceinline__ void store(int q, int w) const { arr(q, w)[0] = u[q]; }

  __device__ __forceinline__ void defect_f(const RbcOp &op, double &r1, double &r2) const {
    const double *c1 = cur(C1), *c2 = cur(C2);
    double l1 = op.c0 * u[F1] + op.a1 * ((c2[-PW] + u[C2]) + (u[C1] + c1[1]));
    double l2 = op.c0 * u[F2] + op.a1 * ((u[C1] + c1[PW]) + (c2[-1] + u[C2]));
    if (op.d1 != 0.0) {
      const double *f1 = cur(F1), *f2 = cur(F2);
      l1 += op.d1 * ((f2[-PW] + f2[-PW + 1]) + (u[F2] + f2[1]));
      l2 += op.d1 * ((f1[-1] + u[F1]) + (f1[PW - 1] + f1[PW]));
    }
    r1 = f[F1] - l1;
    r2 = f[F2] - l2;
  }
  __device__ __forceinline__ void defect_c(const RbcOp &op, double &r1, double &r2) const {
    const double *f1 = cur(F1), *f2 = cur(F2);
    double l1 = op.c0 * u[C1] + op.a1 * ((f2[-PW] + u[F2]) + (f1[-1] + u[F1]));
    double l2 = op.c0 * u[C2] + op.a1 * ((u[F1] + f1[PW]) + (u[F2] + f2[1]));
    if (op.d1 != 0.0) {
      const double *c1 = cur(C1), *c2 = cur(C2);
      l1 += op.d1 * ((c2[-PW - 1] + c2[-PW]) + (c2[-1] + u[C2]));
      l2 += op.d1 * ((u[C1] + c1[1]) + (c1[PW] + c1[PW + 1]));
    }
    r1 = f[C1] - l1;
    r2 = f[C2] - l2;
  }
  // F step (colour 0) or C step (1); zero: the iterate is zero, so the F step needs no
  // neighbours.
  __device__ __forceinline__ void step(const RbcOp &op, double om, int colour, bool zero) {
    if (owner) {
      double r1 = f[colour ? C1 : F1], r2 = f[colour ? C2 : F2];
      if (!zero) {
        if (colour)
          defect_c(op, r1, r2);
        else
          defect_f(op, r1, r2);
      }
      if (colour) {
        u[C1] += om * r1;
        u[C2] = act(C2) ? u[C2] + om * r2 : u[C2];
        store(C1, wc ^ 1);
        store(C2, wc ^ 1);
      } else {
        u[F1] = act(F1) ? u[F1] + om * r1 : u[F1];
        u[F2] = act(F2) ? u[F2] + om * r2 : u[F2];
        store(F1, wf ^ 1);
        store(F2, wf ^ 1);
      }
    }
    if (colour)
      wc ^= 1;
    else
      wf ^= 1;
    __syncthreads();
  }
  // All four values into the current buffers.
  __device__ __forceinline__ void put() const {
    if (owner) {
      store(C1, wc);
      store(F1, wf);
      store(F2, wf);
      store(C2, wc);
    }
    __syncthreads();
  }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int q = 0; q < 4; ++q) u[q] = 0.0;
    put();
  }
  // The defect restricted onto the rotated level below: its F and C right-hand side at this
  // thread's places.
  __device__ __forceinline__ void restrict_to(const RbcOp &op, double &fF, double &fC) const {
    double a1 = 0.0, a2 = 0.0, b1 = 0.0, b2 = 0.0;
    double *s1 = arr(F1, wf ^ 1), *s2 = arr(F2, wf ^ 1);  // the spare buffers
    if (owner) {
      defect_f(op, a1, a2);
      defect_c(op, b1, b2);
      a1 = act(F1) ? a1 : 0.0;
      a2 = act(F2) ? a2 : 0.0;
      s1[0] = a1;
      s2[0] = a2;
    }
    __syncthreads();
    fF = fC = 0.0;
    if (owner) {
      // frame cells hold boundary values of u: the defect there is 0
      const double up = p > 0 ? s2[-PW] : 0.0, lf = k > 0 ? s1[-1] : 0.0;
      fF = (4.0 * b1 + ((up + a2) + (lf + a1))) * 0.125;
      const double v = (4.0 * b2 + ((a1 + s1[PW]) + (a2 + s2[1]))) * 0.125;
      fC = act(C2) ? v : 0.0;
    }
  }
};

// One rotated level.
template <int N>
struct Rot {
  static constexpr int M = Dim<N>::M, PW = Dim<N>::PW, SZ = Dim<N>::SZ;
  double uF, uC, fF, fC;
  double *cell;
  int wf, wc, p, k;
  bool owner, in;  // in: the C point is interior

  __device__ __forceinline__ void init(double *base) {
    const int t = threadIdx.x;
    owner = t < M * M;
    k = t % M;
    p = t / M;
    in = k < M - 1 && p < M - 1;
    cell = base + (owner ? (p + 1) * PW + k + 1 : PW + 1);
    wf = wc = 0;
    uF = uC = fF = fC = 0.0;
  }
  __device__ __forceinline__ double *F(int w) const { return cell + w * SZ; }
  __device__ __forceinline__ double *C(int w) const { return cell + (2 + w) * SZ; }

  __device__ __forceinline__ double defect_f(const RbcOp &op) const {
    const double *c = C(wc);
    double l = op.c0 * uF + op.d1 * ((c[-PW - 1] + c[-PW]) + (c[-1] + uC));
    if (op.a2 != 0.0) {
      const double *f = F(wf);
      const double um = p > 0 ? f[-PW] : -uF, up = p < M - 1 ? f[PW] : -uF;
      const double vm = k > 0 ? f[-1] : -uF, vp = k < M - 1 ? f[1] : -uF;
      l += op.a2 * ((um + up) + (vm + vp));
    }
    return fF - l;
  }
  __device__ __forceinline__ double defect_c(const RbcOp &op) const {
    const double *f = F(wf);
    double l = op.c0 * uC + op.d1 * ((uF + f[1]) + (f[PW] + f[PW + 1]));
    if (op.a2 != 0.0) {
      const double *c = C(wc);
      l += op.a2 * ((c[-PW] + c[PW]) + (c[-1] + c[1]));
    }
    return fC - l;
  }
  __device__ __forceinline__ void step(const RbcOp &op, double om, int colour, bool zero) {
    if (owner) {
      if (colour) {
        const double r = zero ? fC : defect_c(op);
        uC = in ? uC + om * r : 0.0;
        C(wc ^ 1)[0] = uC;
      } else {
        const double r = zero ? fF : defect_f(op);
        uF += om * r;
        F(wf ^ 1)[0] = uF;
      }
    }
    if (colour)
      wc ^= 1;
    else
      wf ^= 1;
    __syncthreads();
  }
  __device__ __forceinline__ void put() const {
    if (owner) {
      F(wf)[0] = uF;
      C(wc)[0] = uC;
    }
    __syncthreads();
  }
  __device__ __forceinline__ void zero() {
    uF = uC = 0.0;
    put();
  }
  // The defect restricted onto the standard level below (side M + 1), its point (P+1, K+1)
  // into the spare C buffer's cell (P, K).
  __device__ __forceinline__ void restrict_down(const RbcOp &op) const {
    double a = 0.0, b = 0.0;
    double *s = F(wf ^ 1);
    if (owner) {
      a = defect_f(op);
      b = defect_c(op);
      s[0] = a;
    }
    __syncthreads();
    if (owner) {
      const double v = (4.0 * b + ((a + s[1]) + (s[PW] + s[PW + 1]))) * 0.125;
      C(wc ^ 1)[0] = in ? v : 0.0;
    }
    __syncthreads();
  }
};

constexpr int std_elems(int N) { return 8 * ((N - 1) / 2 + 2) * ((N - 1) / 2 + 2); }
constexpr int rot_elems(int N) { return std_elems(N) / 2; }
// The 17^2 level: the solution with its zero boundary, two work arrays, the sine table.
constexpr int kE17 = 17 * 17, kWork = kM0;
constexpr int coarse_elems() { return kE17 + 2 * kWork + kM0 + 1; }

template <int TOP>
constexpr int lds_elems() {
  return (TOP == 65 ? std_elems(65) + rot_elems(65) : 0) + std_elems(33) + rot_elems(33) + coarse_elems();
}
template <int TOP>
constexpr int threads_of() {
  return Dim<TOP>::M * Dim<TOP>::M;
}

template <int TOP>
struct Tail {
  const RbcTailArgs &a;
  Std<65> s65;
  Rot<65> r65;
  Std<33> s33;
  Rot<33> r33;
  double *b33, *e17, *w0, *w1, *tab;
  double scale;  // of this thread's mode on the 17^2 level
  __device__ Tail(const RbcTailArgs &args) : a(args) {}

  __device__ __forceinline__ const RbcOp &op(int i) const { return a.op[i]; }  // 65, r65, 33, r33
  __device__ __forceinline__ double om(int i) const { return a.om[i]; }

  // e = A^{-1} g on the 17^2 level by sine transforms along both axes and back; g in the
  // spare C buffer of r33.
  __device__ __forceinline__ void coarsest() {
    const int t = threadIdx.x;
    const int P = t / kQ, K = t % kQ;
    const bool on = t < kM0;
    constexpr int PW = Rot<33>::PW;
    if (on) {
      const double *g = r33.C(r33.wc ^ 1) - (r33.owner ? (r33.p + 1) * PW + r33.k + 1 : PW + 1) + (P + 1) * PW + 1;
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < kQ; ++i) s += tab[i * kQ + K] * g[i];
      w0[t] = s;
    }
    __syncthreads();
    if (on) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < kQ; ++i) s += tab[i * kQ + P] * w0[i * kQ + K];
      w1[t] = s * scale;
    }
    __syncthreads();
    if (on) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < kQ; ++i) s += tab[i * kQ + K] * w1[P * kQ + i];
      w0[t] = s;
    }
    __syncthreads();
    if (on) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < kQ; ++i) s += tab[i * kQ + P] * w0[i * kQ + K];
      e17[(P + 1) * 17 + K + 1] = s;
    }
    __syncthreads();
  }

  template <typename L>
  __device__ __forceinline__ void sweeps(L &l, int i, int nu, bool zero) {
    if (zero && nu == 0) l.zero();
    for (int s = 0; s < nu; ++s) {
      l.step(op(i), om(i), 0, zero && s == 0);
      l.step(op(i), om(i), 1, false);
    }
  }
  // A level entered with the zero iterate: values in registers and current buffers.
  template <int N>
  __device__ __forceinline__ void start(Std<N> &l, int nu) {
#pragma unroll
    for (int q = 0; q < 4; ++q) l.u[q] = 0.0;
    if (nu > 0) l.put();  // the C points (and same-colour neighbours) read by the first steps
  }
  template <int N>
  __device__ __forceinline__ void start(Rot<N> &l, int nu) {
    l.uF = l.uC = 0.0;
    if (nu > 0) l.put();
  }

  __device__ __forceinline__ void visit_r33(bool zero) {
    if (zero) start(r33, a.nu1);
    sweeps(r33, 3, a.nu1, zero);
    r33.restrict_down(op(3));
    coarsest();
    if (r33.owner) {
      const double *e = e17 + r33.p * 17 + r33.k;  // (P, K)
      r33.uC = r33.in ? r33.uC + e[18] : 0.0;
      r33.uF += 0.25 * ((e[0] + e[1]) + (e[17] + e[18]));
    }
    r33.put();
    sweeps(r33, 3, a.nu2, false);
  }
  // The correction of a rotated level onto the standard level of its side.
  template <int N>
  __device__ __forceinline__ void correct(Std<N> &s, const Rot<N> &r) {
    if (s.owner) {
      using S = Std<N>;
      constexpr int PW = S::PW;
      const double *F = r.F(r.wf), *C = r.C(r.wc);
      const double e1 = r.uF, e2 = r.uC;
      const double d1 = 0.25 * ((C[-PW] + e2) + (e1 + F[1])), d2 = 0.25 * ((e1 + F[PW]) + (C[-1] + e2));
      s.u[S::C1] += e1;
      s.u[S::C2] = s.act(S::C2) ? s.u[S::C2] + e2 : s.u[S::C2];
      s.u[S::F1] = s.act(S::F1) ? s.u[S::F1] + d1 : s.u[S::F1];
      s.u[S::F2] = s.act(S::F2) ? s.u[S::F2] + d2 : s.u[S::F2];
    }
    s.put();
  }
  __device__ __forceinline__ void visit_s33(bool zero) {
    if (zero) start(s33, a.nu1);
    sweeps(s33, 2, a.nu1, zero);
    s33.restrict_to(op(2), r33.fF, r33.fC);
    for (int g = 0; g < a.gamma; ++g) visit_r33(g == 0);
    correct(s33, r33);
    sweeps(s33, 2, a.nu2, false);
  }
  __device__ __forceinline__ void visit_r65(bool zero) {
    if (zero) start(r65, a.nu1);
    sweeps(r65, 1, a.nu1, zero);
    r65.restrict_down(op(1));
    if (s33.owner) {
      constexpr int PW = Rot<65>::PW;
      const double *g = r65.C(r65.wc ^ 1) - ((r65.p + 1) * PW + r65.k + 1) + (2 * s33.p + 1) * PW + 2 * s33.k + 1;
      s33.f[Std<33>::C1] = g[0];
      s33.f[Std<33>::F1] = g[1];
      s33.f[Std<33>::F2] = g[PW];
      s33.f[Std<33>::C2] = g[PW + 1];
    }
    for (int g = 0; g < a.gamma; ++g) visit_s33(g == 0);
    if (r65.owner) {
      // e(i, j), i = P or P+1, j = K or K+1, out of the arrays of s33
      auto e = [&](int i, int j) {
        using S = Std<33>;
        const int q = (i & 1) ? ((j & 1) ? S::C1 : S::F1) : ((j & 1) ? S::F2 : S::C2);
        const int w = (q == S::F1 || q == S::F2) ? s33.wf : s33.wc;
        return b33[(2 * q + w) * S::SZ + ((i + 1) >> 1) * S::PW + ((j + 1) >> 1)];
      };
      const int P = r65.p, K = r65.k;
      const double e00 = e(P, K), e01 = e(P, K + 1), e10 = e(P + 1, K), e11 = e(P + 1, K + 1);
      r65.uC = r65.in ? r65.uC + e11 : 0.0;
      r65.uF += 0.25 * ((e00 + e01) + (e10 + e11));
    }
    r65.put();
    sweeps(r65, 1, a.nu2, false);
  }
  __device__ __forceinline__ void visit_s65(bool zero) {
    if (zero) start(s65, a.nu1);
    sweeps(s65, 0, a.nu1, zero);
    s65.restrict_to(op(0), r65.fF, r65.fC);
    for (int g = 0; g < a.gamma; ++g) visit_r65(g == 0);
    correct(s65, r65);
    sweeps(s65, 0, a.nu2, false);
  }
};

template <int TOP>
__global__ __launch_bounds__(threads_of<TOP>()) void k_rbc_tail_lds(RbcTailArgs a) {
  extern __shared__ __align__(16) double rbc_lds[];
  constexpr int NT = threads_of<TOP>(), M = Dim<TOP>::M, PW = Dim<TOP>::PW;
  using S = Std<TOP>;
  const int t = threadIdx.x, p = t / M, k = t % M;
  // the top level's data, loaded before anything waits: cell (p, k) and, for the first row
  // and column of cells, the boundary values beside them
  const double *fg = a.f + (2 * p + 1) * TOP + 2 * k + 1;
  const double *ug = a.u + (2 * p + 1) * TOP + 2 * k + 1;
  const double f0 = fg[0], f1 = fg[1], f2 = fg[TOP], f3 = fg[TOP + 1];
  double v0 = 0.0, v1 = 0.0, v2 = 0.0, v3 = 0.0;
  double t0 = 0.0, t1 = 0.0, l0 = 0.0, l1 = 0.0, c0 = 0.0;
  if (!a.zero) {
    v0 = ug[0];
    v1 = ug[1];
    v2 = ug[TOP];
    v3 = ug[TOP + 1];
    if (p == 0) {
      t0 = ug[-TOP];
      t1 = ug[-TOP + 1];
    }
    if (k == 0) {
      l0 = ug[-1];
      l1 = ug[TOP - 1];
    }
    if (t == 0) c0 = a.u[0];
  }
  const double sc = a.dst[kM0 + min(t, kM0 - 1)];
  const double tb = a.dst[min(t, kM0 - 1)];
  if (a.done != nullptr && *a.done != 0) return;
  // every frame cell and the 17^2 solution's boundary start at zero
  for (int e = t; e < lds_elems<TOP>(); e += NT) rbc_lds[e] = 0.0;
  Tail<TOP> T(a);
  double *q = rbc_lds;
  if constexpr (TOP == 65) {
    T.s65.init(q);
    q += std_elems(65);
    T.r65.init(q);
    q += rot_elems(65);
  }
  T.b33 = q;
  T.s33.init(q);
  q += std_elems(33);
  T.r33.init(q);
  q += rot_elems(33);
  T.e17 = q;
  T.w0 = q + kE17;
  T.w1 = T.w0 + kWork;
  T.tab = T.w1 + kWork;
  T.scale = sc;
  __syncthreads();
  if (t < kM0) T.tab[t] = tb;
  S *top;
  if constexpr (TOP == 65)
    top = &T.s65;
  else
    top = &T.s33;
  S &l = *top;
  l.f[S::C1] = f0;
  l.f[S::F1] = f1;
  l.f[S::F2] = f2;
  l.f[S::C2] = f3;
  l.u[S::C1] = v0;
  l.u[S::F1] = v1;
  l.u[S::F2] = v2;
  l.u[S::C2] = v3;
  if (!a.zero) {
    // boundary values: row and column 0 in the frame, and every own value, in both buffers
#pragma unroll
    for (int w = 0; w < 2; ++w) {
#pragma unroll
      for (int i = 0; i < 4; ++i) l.store(i, w);
      if (p == 0) {
        l.arr(S::F2, w)[-PW] = t0;
        l.arr(S::C2, w)[-PW] = t1;
      }
      if (k == 0) {
        l.arr(S::F1, w)[-1] = l0;
        l.arr(S::C2, w)[-1] = l1;
      }
      if (t == 0) l.arr(S::C2, w)[-PW - 1] = c0;
    }
  }
  __syncthreads();
  for (int r = 0; r < a.visits; ++r) {
    if constexpr (TOP == 65)
      T.visit_s65(r == 0 && a.zero != 0);
    else
      T.visit_s33(r == 0 && a.zero != 0);
  }
  double *uo = a.u + (2 * p + 1) * TOP + 2 * k + 1;
  uo[0] = l.u[S::C1];
  if (l.act(S::F1)) uo[1] = l.u[S::F1];
  if (l.act(S::F2)) uo[TOP] = l.u[S::F2];
  if (l.act(S::C2)) uo[TOP + 1] = l.u[S::C2];
}

}  // namespace

std::vector<double> rbc_tail_table(const RbcOp &op) {
  const int N = kQ + 1;
  const double pi = 3.14159265358979323846;
  std::vector<double> tab(2 * kM0);
  for (int i = 0; i < kQ; ++i)
    for (int k = 0; k < kQ; ++k) {
      tab[i * kQ + k] = std::sin(pi * (i + 1) * (k + 1) / N);
      const double ci = std::cos(pi * (i + 1) / N), ck = std::cos(pi * (k + 1) / N);
      tab[kM0 + i * kQ + k] = (2.0 / N) * (2.0 / N) / (op.c0 + 2.0 * op.a1 * (ci + ck) + 4.0 * op.d1 * ci * ck);
    }
  return tab;
}

hipError_t rbc_tail_prepare(int top) {
  if (top == 65)
    return hipFuncSetAttribute((const void *)k_rbc_tail_lds<65>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               lds_elems<65>() * (int)sizeof(double));
  if (top == 33)
    return hipFuncSetAttribute((const void *)k_rbc_tail_lds<33>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               lds_elems<33>() * (int)sizeof(double));
  return hipErrorInvalidValue;
}

size_t rbc_tail_lds(int top) {
  return (size_t)(top == 65 ? lds_elems<65>() : lds_elems<33>()) * sizeof(double);
}

hipError_t launch_rbc_tail(int top, const RbcTailArgs &a, hipStream_t s) {
  if (top == 65)
    hipLaunchKernelGGL(k_rbc_tail_lds<65>, dim3(1), dim3(threads_of<65>()), rbc_tail_lds(65), s, a);
  else if (top == 33)
    hipLaunchKernelGGL(k_rbc_tail_lds<33>, dim3(1), dim3(threads_of<33>()), rbc_tail_lds(33), s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mgk
