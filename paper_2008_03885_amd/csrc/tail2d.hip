// tail2d.hip -- the coarse end of a 2D cycle in one workgroup, for the hierarchy that ends
// 65^2, 33^2, 17^2, 9^2 (any suffix of it with at least two levels).
//
// The work of such a level is a few microseconds of launches per pass and a few hundred
// nanoseconds of arithmetic, so what bounds it is the number of phases between barriers
// and what one phase costs.  Against the general tail (tail.hip) a phase here has
// - compile-time sides: every offset is a constant, a thread owns the same points for the
//   whole launch (a column of rows_of points) and keeps their iterate and right-hand side
//   in registers;
// - no integer division, no level table in LDS, no walk over stencil entries: the cross
//   reads 4 / rows + 4 neighbours a point from a frame with odd ghost images, the
//   separable radius-3 operator takes its y sums from the thread's column and its x sums
//   through slots private to the wavefront (a row of a level is at most one wavefront, so
//   the exchange needs no barrier);
// - the restriction straight into the registers of the coarse point's owner, who stores
//   the first sweep from the zero iterate at once;
// - the 9^2 level as one product with the 49 x 49 inverse, held in the registers of the
//   workgroup (four to thirteen entries a thread), summed across lanes by DPP.
//
// Measured (MI355X, back-to-back launches, FP64 V(2,1) cross): 15.7 us from 65^2, 8.3 us
// from 33^2; two visits of a W(2,1) cycle 42 us from 65^2; a separable red-black V(2,1) 16 us
// from 33^2.  The general tail took 16-25 us from 33^2, 52 us for the two W visits from
// 33^2 and 57 us separable red-black.  In clocks (2.1 GHz): a sweep over 65^2 3000 (FP32 1900),
// over 33^2 1450, over 17^2 720, the 9^2 solve 1200 with its restriction, about 6000 for the
// launch's first loads, LDS set-up and first instructions.  Inside solves (kernel trace, working
// launches): FP64 V(2,1) from 65^2 17.0 us, FP32 10.2, the two visits of a W(2,1) cycle
// 39.5, separable red-black from 33^2 15.9.  Solves: 2D 65^2 999 -> 739 us,
// 2049^2 W(2,1) 28.4 -> 12.1 ms, 513^2 mixed 1.75 -> 1.31 ms.
#include <cmath>
#include <cstdint>

#include "mg_internal.h"

namespace mgk {
namespace {

constexpr int kCoarse = 9, kQ = kCoarse - 2, kM = kQ * kQ;

// Frames of a level of side N.
template <int N>
struct Geo {
  static constexpr int W = N - 1;  // lanes of a row: x = 1 .. N-1, the last one idle
  static constexpr int P = N + 4;  // pitch of a frame: two ghost points on every side
  static constexpr int SZ = P * P + 1;
  static constexpr int XS = W + 8;  // slots of a row in the wavefront's exchange buffer
};

// Points per thread (a column) on a level of side N.  65^2: eight rows by 512 threads for
// the FP64 cross, which spills at four by 1024 (22.4 against 16.8 us a V(2,1) visit); four
// by 1024 in FP32 (12.4 against 13.4 us).
template <typename T, int N, bool SEP>
constexpr int rows_of() {
  return N == 65 ? (sizeof(T) == 8 && !SEP ? 8 : 4) : N == 33 ? 2 : 1;
}

constexpr int kXchg = 96;  // slots per exchange buffer: 64 / W rows of W + 8 slots

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The level's operator, read from the kernel's arguments once per half of a visit: an
// offset the compiler cannot see through keeps it from holding the values of all three
// levels at once (it spilled them).
template <typename T, bool SEP>
__device__ __forceinline__ Tail2dOp<T> fetch(const Tail2dOp<T> &op) {
  if (!SEP) return op;
  int zero;
  asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
  return (&op)[zero];
}

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
// Sum over groups of G = 4, 8 or 16 consecutive lanes, left in every lane of the group.
template <int G>
__device__ __forceinline__ double group_sum(double v) {
  v += dpp<0xB1>(v);                // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);                // quad_perm [2,3,0,1]
  if (G > 4) v += dpp<0x141>(v);    // row_half_mirror
  if (G > 8) v += dpp<0x140>(v);    // row_mirror
  return v;
}

// One level's points of this thread, its two frames and the steps on them.
template <typename T, int N, bool SEP>
struct Lvl {
  using G = Geo<N>;
  static constexpr int ROWS = rows_of<T, N, SEP>(), P = G::P, W = G::W;
  static constexpr int OWNERS = W * (W / ROWS);
  static constexpr int BR = ROWS == 2 ? 2 : 1;  // rows per x exchange
  T u[ROWS], f[ROWS];
  T *cur, *oth;    // this thread's first point in the current and the other frame
  static constexpr int GL = W / ROWS - 1;  // the last thread of a column
  int x, y0, g;
  bool owner, xin;
  int gx;          // offset of the point's image across a vertical side, 0: none
  bool gx1;        // that image is next to the side (distance 1)
  int gy, gxy;     // one row a thread: offsets of the other images, 0: none
  T sx, sy;        // and the signs of the x and y images (1: none)

  // Point r is interior: the last row of the last thread is the boundary line.
  __device__ __forceinline__ bool act(int r) const { return xin && (r < ROWS - 1 || g != GL); }

  __device__ __forceinline__ void init(T *frame0, T *frame1) {
    const int t = threadIdx.x;
    owner = t < OWNERS;
    x = 1 + (t & (W - 1));
    g = N == 65 ? __builtin_amdgcn_readfirstlane(t / W) : t / W;
    y0 = 1 + ROWS * g;
    xin = owner && x <= N - 2;
    const int id = owner ? (y0 + 2) * P + x + 2 : 2 * P + 2;
    cur = frame0 + id;
    oth = frame1 + id;
    gx = x == 1 ? -2 : x == N - 2 ? 2 : 0;
    gx1 = gx != 0;
    if (SEP) gx = x == 2 ? -4 : x == N - 3 ? 4 : gx;
    if constexpr (ROWS == 1) {
      gy = g == 0 ? -2 * P : g == GL - 1 ? 2 * P : 0;
      gxy = gx1 && gy != 0 ? gx + gy : 0;
      if (SEP) gy = g == 1 ? -4 * P : g == GL - 2 ? 4 * P : gy;
      sx = gx != 0 ? T(-1) : T(1);
      sy = gy != 0 ? T(-1) : T(1);
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) u[r] = f[r] = T(0);
  }
  // Zero the boundary lines of both frames with their ghost cells; every other cell is
  // stored before it is read.
  static __device__ __forceinline__ void clear(T *frame0, T *frame1, int nt) {
    for (int e = threadIdx.x; e < 8 * P; e += nt) {
      T *fr = (e & 1) ? frame1 : frame0;
      const int k = (e >> 1) / 4, side = (e >> 1) & 3;
      const int b = (side & 1) ? N + 1 : 2;
      fr[side < 2 ? b * P + k : k * P + b] = T(0);
    }
  }
  // Stores the thread's points with their odd images (corner images at distance 1 only:
  // interpolation reads no other).  Boundary points hold u = 0 and are stored as well.
  __device__ __forceinline__ void put_all(T *fr) const {
    if (!owner) return;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) fr[r * P] = u[r];
    if constexpr (ROWS == 1) {
      // no branches: a point without an image stores its own value once more
      fr[gx] = sx * u[0];
      fr[gy] = sy * u[0];
      fr[gxy] = u[0];
    } else {
      if (gx != 0) {
        T *q = fr + gx;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) q[r * P] = -u[r];
      }
      // rows 1 and 2 are the first thread's, row N-2 the last one's last but one
      if (g == 0) {
        fr[-2 * P] = -u[0];
        if (SEP) fr[-3 * P] = -u[1];
        if (gx1) fr[gx - 2 * P] = u[0];
      }
      if (g == GL) {
        fr[ROWS * P] = -u[ROWS - 2];
        if (SEP && ROWS > 2) fr[(ROWS + 1) * P] = -u[ROWS > 2 ? ROWS - 3 : 0];
        if (gx1) fr[gx + ROWS * P] = u[ROWS - 2];
      }
      if (SEP && ROWS == 2 && g == GL - 1) fr[(ROWS + 3) * P] = -u[1];
    }
  }
  // r = f - L u at the thread's points, u the current frame (and registers).
  __device__ __forceinline__ void defect(const Tail2dOp<T> &op, T *xa, T *xb, T (&res)[ROWS]) const {
    if (!SEP || op.cross) {
      T c[ROWS + 4];
      c[0] = cur[-2 * P];
      c[1] = cur[-P];
      c[ROWS + 2] = cur[ROWS * P];
      c[ROWS + 3] = cur[(ROWS + 1) * P];
#pragma unroll
      for (int r = 0; r < ROWS; ++r) c[2 + r] = u[r];
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        const T *q = cur + r * P;
        const T v = u[r];
        const T d1 = ((v - q[-1]) + (v - q[1])) + ((v - c[r + 1]) + (v - c[r + 3]));
        const T d2 = ((v - q[-2]) + (v - q[2])) + ((v - c[r]) + (v - c[r + 4]));
        res[r] = f[r] - (op.w1 * d1 + op.w2 * d2);
      }
    } else {
      T c[ROWS + 6];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        c[k] = cur[(k - 3) * P];
        c[ROWS + 3 + k] = cur[(ROWS + k) * P];
      }
#pragma unroll
      for (int r = 0; r < ROWS; ++r) c[3 + r] = u[r];
      // this row's slots: x at xa[x + 2], ghost images at -2, -1, N, N + 1
      const int g = (threadIdx.x & 63) / W;
      T *pa = xa + g * G::XS + 2 + x, *pb = xb + g * G::XS + 2 + x;
#pragma unroll
      for (int r0 = 0; r0 < ROWS; r0 += BR) {
        T A[BR], B[BR];
#pragma unroll
        for (int d = 0; d < BR; ++d) {
          const int r = r0 + d;
          const T v = u[r];
          A[d] = T(0);
          B[d] = op.b[0] * v;
#pragma unroll
          for (int k = 1; k <= 3; ++k) {
            A[d] += op.a[k - 1] * ((c[3 + r - k] - v) + (c[3 + r + k] - v));
            B[d] += op.b[k] * (c[3 + r - k] + c[3 + r + k]);
          }
        }
        wave_fence();
#pragma unroll
        for (int d = 0; d < BR; ++d) {
          T *qa = pa + d * 2 * kXchg, *qb = pb + d * 2 * kXchg;
          qa[0] = A[d];
          qb[0] = B[d];
          if (gx != 0) {
            qa[gx] = -A[d];
            qb[gx] = -B[d];
          }
          if (x == 1) qa[-1] = qb[-1] = T(0);  // the slot may hold another level's sum
        }
        wave_fence();
#pragma unroll
        for (int d = 0; d < BR; ++d) {
          const T *qa = pa + d * 2 * kXchg, *qb = pb + d * 2 * kXchg;
          T lu = op.b[0] * A[d];
#pragma unroll
          for (int k = 1; k <= 3; ++k) {
            lu += op.a[k - 1] * ((qb[-k] - B[d]) + (qb[k] - B[d]));
            lu += op.b[k] * (qa[-k] + qa[k]);
          }
          res[r0 + d] = f[r0 + d] - lu;
        }
        // a wavefront runs one batch of rows after the other: all at once would hold every
        // row's sums in registers
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // One partial step (colour 0: every point, 1 red, 2 black) into the other frame.
  __device__ __forceinline__ void relax(T om, int colour, const T (&res)[ROWS]) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      const T w = (colour == 0 || ((x + y0 + r) & 1) == (colour & 1)) ? om : T(0);
      u[r] = act(r) ? u[r] + w * res[r] : T(0);
    }
    put_all(oth);
    T *t = cur;
    cur = oth;
    oth = t;
    __syncthreads();
  }
  __device__ __forceinline__ void step(const Tail2dOp<T> &op, int colour, T *xa, T *xb) {
    T res[ROWS];
    if (owner) defect(op, xa, xb, res);
    relax(op.om, colour, res);
  }
  // nu sweeps, the first `from` partial steps already done.
  __device__ __forceinline__ void sweeps(const Tail2dOp<T> &op, int nu, int rb, int from, T *xa, T *xb) {
    const int steps = rb ? 2 * nu : nu;
    for (int s = from; s < steps; ++s) step(op, rb ? 1 + (s & 1) : 0, xa, xb);
  }
  // The first partial step from a zero iterate (u = omega/a0 f on its points), or the zero
  // iterate itself when there are no sweeps; returns the partial steps done.
  __device__ __forceinline__ int start_zero(const Tail2dOp<T> &op, int nu, int rb) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      const bool on = nu > 0 && (!rb || ((x + y0 + r) & 1) == 1);
      u[r] = (on && act(r)) ? op.om * f[r] : T(0);
    }
    put_all(cur);
    __syncthreads();
    return nu > 0 ? 1 : 0;
  }
  // The defect into the other frame (interior points; no images).
  __device__ __forceinline__ void store_defect(const Tail2dOp<T> &op, T *xa, T *xb) const {
    if (owner) {
      T res[ROWS];
      defect(op, xa, xb, res);
#pragma unroll
      for (int r = 0; r < ROWS; ++r)
        if (act(r)) oth[r * P] = res[r];
    }
    __syncthreads();
  }
  // u += I_H^h v, v in the coarse level's frame (origin at coarse point (0, 0)).
  template <int PC>
  __device__ __forceinline__ void prolong(const T *v, int order) {
    if (owner) {
      constexpr int CR = ROWS == 1 ? 4 : ROWS / 2 + 3;
      const int b = y0 >> 1;  // rows b-1 .. b+CR-2 of the coarse frame
      const T *q = v + (b - 1) * PC + (x >> 1);
      const bool ox = x & 1;
      // 9/16 and -1/16 (the sums round as 9 s - t does), or 1/2 and 0
      const T w1 = order == 3 ? T(0.5625) : T(0.5), w3 = order == 3 ? T(-0.0625) : T(0);
      T h[CR];
#pragma unroll
      for (int j0 = 0; j0 < CR; j0 += 4) {  // four rows of loads at a time (registers)
        T m[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (j0 + j < CR) m[j][i] = q[(j0 + j) * PC + i - 1];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (j0 + j < CR) h[j0 + j] = ox ? w1 * (m[j][1] + m[j][2]) + w3 * (m[j][0] + m[j][3]) : m[j][1];
        if (CR > 4) __builtin_amdgcn_sched_barrier(0);
      }
      // thread rows start at an odd fine row when ROWS > 1
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        // fine row 2 (b + r') (even) takes coarse row b + r', odd rows the mean below and above
        const int j = ROWS == 1 ? 1 : 1 + (r + 1) / 2;  // h index of coarse row floor(y/2)
        const bool oy = ROWS == 1 ? (y0 & 1) : (r & 1) == 0;
        const T e = oy ? w1 * (h[j] + h[j + 1]) + w3 * (h[j - 1] + h[j + 2 < CR ? j + 2 : j]) : h[j];
        u[r] = act(r) ? cur[r * P] + e : T(0);
      }
      put_all(cur);
    }
    __syncthreads();
  }
};

// Full weighting of the defect in a fine frame (pitch PF, origin at fine point (0, 0)) at
// coarse point (X, Y).
template <typename T, int PF>
__device__ __forceinline__ T full_weight(const T *r, int X, int Y) {
  const T *q = r + 2 * Y * PF + 2 * X;
  const T ym = T(0.25) * q[-PF - 1] + T(0.5) * q[-PF] + T(0.25) * q[-PF + 1];
  const T y0 = T(0.25) * q[-1] + T(0.5) * q[0] + T(0.25) * q[1];
  const T yp = T(0.25) * q[PF - 1] + T(0.5) * q[PF] + T(0.25) * q[PF + 1];
  return T(0.25) * ym + T(0.5) * y0 + T(0.25) * yp;
}

template <typename T, int TOP, bool SEP>
constexpr int tail2d_threads() {
  return Lvl<T, TOP, SEP>::OWNERS;
}

// LDS elements before each part: frames of the levels TOP .. 17 (two each), the 9^2 frame,
// the exchange buffers.
template <int TOP>
constexpr int frames_elems() {
  return 2 * ((TOP >= 65 ? Geo<65>::SZ : 0) + (TOP >= 33 ? Geo<33>::SZ : 0) + Geo<17>::SZ) + Geo<9>::SZ + Geo<65>::P;
}

template <typename T, int TOP, bool SEP>
struct Engine {
  static constexpr int NT = tail2d_threads<T, TOP, SEP>();
  static constexpr int PARTS = NT / 64, ENT = (kM + PARTS - 1) / PARTS;
  const Tail2dArgs<T> &a;
  Lvl<T, 65, SEP> l65;
  Lvl<T, 33, SEP> l33;
  Lvl<T, 17, SEP> l17;
  T *frame9;
  T *xa, *xb;
  double *fvec;        // the 9^2 right-hand side, 49 values
  double inv[ENT];     // this thread's entries of the 9^2 inverse: row t / PARTS, columns t % PARTS + PARTS k

  __device__ Engine(const Tail2dArgs<T> &args) : a(args) {}

  template <int N>
  __device__ __forceinline__ const Tail2dOp<T> &op() const {
    return a.op[N == 65 ? 0 : N == 33 ? 1 : 2];
  }
  // Offset of a frame's coarse/fine point (0, 0).
  template <int N>
  static __device__ __forceinline__ int origin() {
    return 2 * Geo<N>::P + 2;
  }
  // frame base of the level's other / current frame, uniform over threads
  template <int N>
  __device__ __forceinline__ T *frame_of(const Lvl<T, N, SEP> &l, bool other) const {
    const int id = l.owner ? (l.y0 + 2) * Geo<N>::P + l.x + 2 : 2 * Geo<N>::P + 2;
    return (other ? l.oth : l.cur) - id;
  }

  __device__ __forceinline__ void coarsest() {
    const int t = threadIdx.x;
    if (t < 64) {
      const int X = 1 + (t & 7), Y = 1 + (t >> 3);
      if (X <= kQ && Y <= kQ)
        fvec[(Y - 1) * kQ + X - 1] =
            (double)full_weight<T, Geo<17>::P>(frame_of<17>(l17, true) + origin<17>(), X, Y);
    }
    __syncthreads();
    const int row = t / PARTS, p = t % PARTS;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < ENT; ++k) {
      const int c = p + PARTS * k;
      s += inv[k] * fvec[c < kM ? c : 0];
    }
    s = group_sum<PARTS>(s);
    if (p == 0 && row < kM) {
      constexpr int P = Geo<9>::P;
      const int X = 1 + row % kQ, Y = 1 + row / kQ;
      const T v = (T)s;
      T *q = frame9 + (Y + 2) * P + X + 2;
      q[0] = v;
      const int gx = X == 1 ? -2 : X == kQ ? 2 : 0, gy = Y == 1 ? -2 : Y == kQ ? 2 : 0;
      if (gx != 0) q[gx] = -v;
      if (gy != 0) q[gy * P] = -v;
      if (gx != 0 && gy != 0) q[gy * P + gx] = v;
    }
    __syncthreads();
  }

  // One visit: pre-smoothing (from the zero iterate, or the current one with `from`
  // partial steps already done), defect, coarse visits, correction, post-smoothing.
  __device__ __forceinline__ void visit17(bool zero, int from) {
    Tail2dOp<T> o = fetch<T, SEP>(op<17>());
    if (zero) from = l17.start_zero(o, a.nu1, a.rb);
    l17.sweeps(o, a.nu1, a.rb, from, xa, xb);
    l17.store_defect(o, xa, xb);
    coarsest();
    o = fetch<T, SEP>(op<17>());
    l17.template prolong<Geo<9>::P>(frame9 + origin<9>(), a.prolong);
    l17.sweeps(o, a.nu2, a.rb, 0, xa, xb);
  }
  __device__ __forceinline__ void visit33(bool zero, int from) {
    Tail2dOp<T> o = fetch<T, SEP>(op<33>());
    if (zero) from = l33.start_zero(o, a.nu1, a.rb);
    l33.sweeps(o, a.nu1, a.rb, from, xa, xb);
    l33.store_defect(o, xa, xb);
    if (l17.act(0))
      l17.f[0] = full_weight<T, Geo<33>::P>(frame_of<33>(l33, true) + origin<33>(), l17.x, l17.y0);
    for (int g = 0; g < a.gamma; ++g) visit17(g == 0, 0);
    o = fetch<T, SEP>(op<33>());
    l33.template prolong<Geo<17>::P>(frame_of<17>(l17, false) + origin<17>(), a.prolong);
    l33.sweeps(o, a.nu2, a.rb, 0, xa, xb);
  }
  __device__ __forceinline__ void visit65(bool zero, int from) {
    Tail2dOp<T> o = fetch<T, SEP>(op<65>());
    if (zero) from = l65.start_zero(o, a.nu1, a.rb);
    l65.sweeps(o, a.nu1, a.rb, from, xa, xb);
    l65.store_defect(o, xa, xb);
    if (l33.owner) {
      const T *r = frame_of<65>(l65, true) + origin<65>();
#pragma unroll
      for (int k = 0; k < Lvl<T, 33, SEP>::ROWS; ++k)
        if (l33.act(k)) l33.f[k] = full_weight<T, Geo<65>::P>(r, l33.x, l33.y0 + k);
    }
    for (int g = 0; g < a.gamma; ++g) visit33(g == 0, 0);
    o = fetch<T, SEP>(op<65>());
    l65.template prolong<Geo<33>::P>(frame_of<33>(l33, false) + origin<33>(), a.prolong);
    l65.sweeps(o, a.nu2, a.rb, 0, xa, xb);
  }
};

template <typename T, int TOP, bool SEP>
__device__ __forceinline__ auto &top_level(Engine<T, TOP, SEP> &e) {
  if constexpr (TOP == 65)
    return e.l65;
  else if constexpr (TOP == 33)
    return e.l33;
  else
    return e.l17;
}
template <typename T, int TOP, bool SEP>
__device__ __forceinline__ void visit_top(Engine<T, TOP, SEP> &e, bool zero, int from) {
  if constexpr (TOP == 65)
    e.visit65(zero, from);
  else if constexpr (TOP == 33)
    e.visit33(zero, from);
  else
    e.visit17(zero, from);
}

// The frames, carved from `lds`, with their boundary lines cleared.
template <typename T, int TOP, bool SEP>
__device__ __forceinline__ void setup(Engine<T, TOP, SEP> &e, unsigned char *lds) {
  constexpr int NT = tail2d_threads<T, TOP, SEP>();
  e.fvec = reinterpret_cast<double *>(lds);
  T *const frames = reinterpret_cast<T *>(e.fvec + 64);
  T *p = frames;
  if constexpr (TOP >= 65) {
    Lvl<T, 65, SEP>::clear(p, p + Geo<65>::SZ, NT);
    e.l65.init(p, p + Geo<65>::SZ);
    p += 2 * Geo<65>::SZ;
  }
  if constexpr (TOP >= 33) {
    Lvl<T, 33, SEP>::clear(p, p + Geo<33>::SZ, NT);
    e.l33.init(p, p + Geo<33>::SZ);
    p += 2 * Geo<33>::SZ;
  }
  Lvl<T, 17, SEP>::clear(p, p + Geo<17>::SZ, NT);
  e.l17.init(p, p + Geo<17>::SZ);
  p += 2 * Geo<17>::SZ;
  e.frame9 = p;
  Lvl<T, 9, SEP>::clear(p, p, NT);
  T *x = frames + frames_elems<TOP>();
  e.xa = x + (threadIdx.x >> 6) * 4 * kXchg;
  e.xb = e.xa + kXchg;
  if (SEP)
    for (int k = threadIdx.x & 63; k < 4 * kXchg; k += 64) e.xa[k] = T(0);
}

template <typename T, int TOP, bool SEP>
constexpr size_t lds_bytes() {
  return (frames_elems<TOP>() + (SEP ? tail2d_threads<T, TOP, SEP>() / 64 * 4 * kXchg : 0)) * sizeof(T) +
         64 * sizeof(double);
}

// Stores the top level's iterate with its zero boundary.
template <typename T, int N, bool SEP>
__device__ __forceinline__ void store_top(const Lvl<T, N, SEP> &l, T *ug) {
  if (!l.owner) return;
#pragma unroll
  for (int r = 0; r < Lvl<T, N, SEP>::ROWS; ++r) {
    const int y = l.y0 + r;
    ug[y * N + l.x] = l.act(r) ? l.u[r] : T(0);
    if (l.x == 1) ug[y * N] = T(0);
  }
  if (l.y0 == 1) {
    ug[l.x] = T(0);
    if (l.x == 1) ug[0] = T(0);
  }
}

// The top level's values of a thread, loaded ahead of the set-up of the frames.
template <typename T, int N, bool SEP>
struct TopData {
  using L = Lvl<T, N, SEP>;
  T f[L::ROWS], u[L::ROWS];
  __device__ __forceinline__ void load(const T *fg, const T *ug, bool zero) {
    const int x = 1 + threadIdx.x % L::W, y0 = 1 + L::ROWS * (threadIdx.x / L::W);
#pragma unroll
    for (int r = 0; r < L::ROWS; ++r) {
      f[r] = fg[(y0 + r) * N + x];
      u[r] = T(0);
    }
    if (!zero) {
#pragma unroll
      for (int r = 0; r < L::ROWS; ++r) u[r] = ug[(y0 + r) * N + x];
    }
  }
  __device__ __forceinline__ void put(L &l) const {
#pragma unroll
    for (int r = 0; r < L::ROWS; ++r) {
      l.f[r] = l.act(r) ? f[r] : T(0);
      l.u[r] = l.act(r) ? u[r] : T(0);
    }
  }
};

// This thread's entries of the 9^2 inverse.
template <typename T, int TOP, bool SEP>
__device__ __forceinline__ void load_inverse(Engine<T, TOP, SEP> &e) {
  const int row = threadIdx.x / e.PARTS, part = threadIdx.x % e.PARTS;
#pragma unroll
  for (int k = 0; k < e.ENT; ++k) {
    const int c = part + e.PARTS * k;
    const double v = e.a.ainv_t[min(c, kM - 1) * kM + min(row, kM - 1)];
    e.inv[k] = c < kM ? v : 0.0;  // rows past the last one are not stored
  }
}

template <typename T, int TOP, bool SEP>
__global__ __launch_bounds__((tail2d_threads<T, TOP, SEP>())) void k_tail2d(Tail2dArgs<T> a) {
  extern __shared__ __align__(16) unsigned char tail2d_lds[];
  const int *done = slot_done(a.done);
  const T *fg = slot_ptr(static_cast<const T *>(a.f_top), (size_t)TOP * TOP);
  T *ug = slot_ptr(static_cast<T *>(a.u_top), (size_t)TOP * TOP);
  Engine<T, TOP, SEP> e(a);
  auto &l = top_level(e);
  // the flag, the right-hand side and the inverse are loaded before anything waits
  TopData<T, TOP, SEP> d;
  d.load(fg, ug, a.zero_init != 0);
  const int stop = done != nullptr ? *done : 0;
  load_inverse(e);
  if (stop != 0) return;
  setup(e, tail2d_lds);
  d.put(l);
  if (!a.zero_init) l.put_all(l.cur);
  __syncthreads();
  for (int r = 0; r < a.repeats; ++r) visit_top(e, r == 0 && a.zero_init != 0, 0);
  store_top(l, ug);
}

template <typename T, int TOP, bool SEP>
hipError_t launch_top(const Tail2dArgs<T> &args, hipStream_t s, int slots) {
  hipLaunchKernelGGL((k_tail2d<T, TOP, SEP>), dim3(1, 1, slots), dim3(tail2d_threads<T, TOP, SEP>()),
                     (lds_bytes<T, TOP, SEP>()), s, args);
  return hipGetLastError();
}

template <typename T, int TOP, bool SEP>
hipError_t prepare_top() {
  return hipFuncSetAttribute((const void *)k_tail2d<T, TOP, SEP>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)lds_bytes<T, TOP, SEP>());
}

// The FP64 separable instance starts at 33^2: from 65^2 it holds more than 128 registers a
// thread and spills (a 65^2 sweep took 9 us, one V(2,1) visit 31 us against 11 us from
// 33^2 and two launches).
template <typename T>
constexpr bool has65_sep() {
  return sizeof(T) == 4;
}

template <typename T, int TOP>
size_t lds_of(bool sep) {
  return sep ? lds_bytes<T, TOP, true>() : lds_bytes<T, TOP, false>();
}

}  // namespace

template <typename T>
size_t tail2d_lds_bytes(int top, bool sep) {
  if (top == 65 && sep && !has65_sep<T>()) return SIZE_MAX;  // no such instance
  return top == 65 ? lds_of<T, 65>(sep) : top == 33 ? lds_of<T, 33>(sep) : lds_of<T, 17>(sep);
}

template <typename T>
hipError_t tail2d_prepare(int top, bool sep) {
  switch (top) {
    case 65:
      if (!sep) return prepare_top<T, 65, false>();
      if constexpr (has65_sep<T>()) return prepare_top<T, 65, true>();
      return hipErrorInvalidValue;
    case 33: return sep ? prepare_top<T, 33, true>() : prepare_top<T, 33, false>();
    case 17: return sep ? prepare_top<T, 17, true>() : prepare_top<T, 17, false>();
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_tail2d(int top, const Tail2dArgs<T> &args, bool sep, hipStream_t s, int slots) {
  switch (top) {
    case 65:
      if (!sep) return launch_top<T, 65, false>(args, s, slots);
      if constexpr (has65_sep<T>()) return launch_top<T, 65, true>(args, s, slots);
      return hipErrorInvalidValue;
    case 33: return sep ? launch_top<T, 33, true>(args, s, slots) : launch_top<T, 33, false>(args, s, slots);
    case 17: return sep ? launch_top<T, 17, true>(args, s, slots) : launch_top<T, 17, false>(args, s, slots);
    default: return hipErrorInvalidValue;
  }
}

template size_t tail2d_lds_bytes<double>(int, bool);
template size_t tail2d_lds_bytes<float>(int, bool);
template hipError_t tail2d_prepare<double>(int, bool);
template hipError_t tail2d_prepare<float>(int, bool);
template hipError_t launch_tail2d<double>(int, const Tail2dArgs<double> &, bool, hipStream_t, int);
template hipError_t launch_tail2d<float>(int, const Tail2dArgs<float> &, bool, hipStream_t, int);

}  // namespace mgk
