// rbc_passes.hip -- red-black coarsening: a level's half cycles in one pass each.
//
// The partial steps, restriction and interpolation of a red-black coarsening level are
// stencils of one row and one column each, so a level that runs them one launch after the
// other moves its iterate through HBM six times per V(1,1) visit.  These kernels run the
// whole half of a visit in one pass: every wavefront owns a strip of columns (64 lanes with
// a halo of H on each side that is computed but not written) and marches down a band of
// rows with the stages pipelined, stage s a row or two behind stage s-1, so that the
// stages of one row step are independent.  Neighbours in a row come by DPP wavefront
// shifts, neighbours across rows from register windows: no LDS, no barriers.
//   pre:  F step, C step, defect, restriction (reads u and f, writes u and f_coarse);
//   post: interpolation and correction, F step, C step (reads u, f and e, writes u).
// A rotated level (packed rows) is marched two storage rows at a time: row pair p holds
// the C points (2p, 2k), which are the next level's points (p, k), and the F points
// (2p+1, 2k+1), so every coupling is to row pairs p-1, p, p+1 and columns k-1, k, k+1.
//
// Bound: HBM on the large levels.  Measured (MI355X, kernel trace of a 4097^2 G1 V(1,1)
// solve), against four partial steps of 92 us, a restriction of 117 us and an interpolation
// of 93 us on level 0: pre 100 to 105 us by card (28 B a point, 4.5 TB/s; a 256 MB device copy
// runs at 5.5 TB/s; 547 MB counted, 1.16x), post 102 to 113 us (561 MB counted); rotated
// level 1 (8.4e6 points) pre from zero 45 us, post 57 to 59 us (4 x 48, 84 and 42 us); a level of side 513 or less
// 4.5 to 8 us a pass, its launch and the latency of one band.  A cycle moves 1.22 times its
// algorithmic bytes.  Solve 14.0 -> 6.05 ms (257^2: 1.71 -> 1.17 ms).
#include <algorithm>

#include "mg_internal.h"
#include "rbc_passes.h"

namespace mgk {
namespace {

constexpr int kWave = 64, kWaves = kBlock / kWave;
constexpr int kAhead = 4;  // rows of every array in flight
constexpr int kTurn = 8;   // row steps per unrolled loop turn: the length of the rings

__device__ __forceinline__ int dpp_prev(int v) { return __builtin_amdgcn_mov_dpp(v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int dpp_next(int v) { return __builtin_amdgcn_mov_dpp(v, 0x130, 0xf, 0xf, true); }
// The value of lane L-1 / L+1 in lane L (0 where there is none).
__device__ __forceinline__ double left(double v) {
  return __hiloint2double(dpp_prev(__double2hiint(v)), dpp_prev(__double2loint(v)));
}
__device__ __forceinline__ double right(double v) {
  return __hiloint2double(dpp_next(__double2hiint(v)), dpp_next(__double2loint(v)));
}

__host__ __device__ constexpr int ring(int a) { return ((a % kTurn) + kTurn) % kTurn; }

template <typename F, int... I>
__device__ __forceinline__ void turn_impl(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <typename F>
__device__ __forceinline__ void turn(F &&f) {
  turn_impl(f, std::make_integer_sequence<int, kTurn>{});
}

__device__ double block_sum(double v) {
  __shared__ double ws[kWaves];
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < kWaves; ++i) t += ws[i];
  return t;
}

struct PassArgs {
  const double *f, *u;  // u: the input iterate (pre: null for zero)
  const double *e;      // post: the next level's correction
  double *uout, *fc, *uc;
  int m, chunk;         // storage side; rows (standard) or row pairs (rotated) per block
  RbcOp op;
  double om;            // omega / c0
  double *partials;
  const int *done;
};

// The strip and band of a wavefront.
struct Place {
  int x;        // column of this lane (rotated: packed column)
  bool active, useful;
  int ra, rb;   // rows [ra, rb) belong to this block
};
template <int H>
__device__ __forceinline__ Place place(int cols, int rows, int chunk) {
  constexpr int S = kWave - 2 * H;
  const int lane = threadIdx.x & (kWave - 1);
  const Block2 blk = block2();
  const int strip = blk.x * kWaves + (threadIdx.x >> 6);
  Place p;
  p.x = strip * S - H + lane;
  p.active = strip * S < cols;
  p.useful = lane >= H && lane < H + S && p.x < cols;
  p.ra = blk.y * chunk;
  p.rb = min(p.ra + chunk, rows);
  return p;
}

// Pins a value loaded ahead in a register before its slot is loaded again.
__device__ __forceinline__ void pin(double &v) { asm volatile("" : "+v"(v)); }

// ----------------------------------------------------------------- standard levels ----
// L u at the centre of three rows of a column; NINE: with diagonal neighbours.
template <bool NINE>
__device__ __forceinline__ double lap_std(double up, double c, double dn, const RbcOp &op) {
  const double s = up + dn;
  double v = op.c0 * c + op.a1 * (s + (left(c) + right(c)));
  if (NINE) v += op.d1 * (left(s) + right(s));
  return v;
}

template <bool NINE, bool HAS_U, bool RESTRICT>
__global__ __launch_bounds__(kBlock) void k_rbc_pre_std(PassArgs a) {
  constexpr int H = RESTRICT ? 4 : 2;
  if (a.done != nullptr && *a.done != 0) return;
  const int m = a.m, wc = (m + 1) / 2;
  const Place pl = place<H>(m, m, a.chunk);
  const int x = pl.x;
  const bool xin = x > 0 && x < m - 1;
  const int xs = min(max(x, 0), m - 1);
  // F at row t, C at t-2, the defect at t-4, the restriction at t-6
  const int ts = pl.ra - (RESTRICT ? 3 : 1), te = pl.rb - 1 + (RESTRICT ? 6 : 2);
  double acc = 0.0;
  if (pl.active) {
    const RbcOp op = a.op;
    auto at = [&](const double *p, int y) { return p[(size_t)min(max(y, 0), m - 1) * m + xs]; };
    double w0[kTurn], w1[kTurn], w2[kTurn], fr[kTurn], dr[kTurn], uq[kAhead], fq[kAhead];
#pragma unroll
    for (int k = 0; k < kTurn; ++k) w0[k] = w1[k] = w2[k] = fr[k] = dr[k] = 0.0;
    if (HAS_U) {
      w0[ring(-1)] = at(a.u, ts - 1);
      w0[ring(0)] = at(a.u, ts);
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (HAS_U) uq[k] = at(a.u, ts + 1 + k);
      fq[k] = at(a.f, ts + k);
    }
    auto inside = [&](int y) { return xin && y > 0 && y < m - 1; };
    auto step = [&](const int t, auto pc) {
      constexpr int P = decltype(pc)::value, Q = P % kAhead;
      double unew = HAS_U ? uq[Q] : 0.0, fnew = fq[Q];
      pin(unew);
      pin(fnew);
      __builtin_amdgcn_sched_barrier(0);
      if (HAS_U) uq[Q] = at(a.u, t + 1 + kAhead);
      fq[Q] = at(a.f, t + kAhead);
      w0[ring(P + 1)] = unew;
      fr[ring(P)] = fnew;
      // F points (odd x + y) at row t
      const bool odd_t = ((x + t) & 1) != 0;  // the same for rows t-2, t-4, t-6
      const double r1 = HAS_U ? fnew - lap_std<NINE>(w0[ring(P - 1)], w0[ring(P)], w0[ring(P + 1)], op) : fnew;
      const bool in1 = inside(t);
      if (a.partials != nullptr && in1 && pl.useful && t >= pl.ra && t < pl.rb) acc += r1 * r1;
      const double n1 = (in1 && odd_t) ? w0[ring(P)] + a.om * r1 : w0[ring(P)];
      // C points (even x + y) at row t-2
      const double r2 = fr[ring(P - 2)] - lap_std<NINE>(w1[ring(P - 3)], w1[ring(P - 2)], w1[ring(P - 1)], op);
      const double n2 = (inside(t - 2) && !odd_t) ? w1[ring(P - 2)] + a.om * r2 : w1[ring(P - 2)];
      if constexpr (RESTRICT) {
        const int y3 = t - 4, y4 = t - 6;
        double r3 = fr[ring(P - 4)] - lap_std<NINE>(w2[ring(P - 5)], w2[ring(P - 4)], w2[ring(P - 3)], op);
        if (!inside(y3)) r3 = 0.0;
        if (pl.useful && y3 >= pl.ra && y3 < pl.rb) a.uout[(size_t)y3 * m + x] = w2[ring(P - 4)];
        const double d0 = dr[ring(P - 6)];
        const double v = (4.0 * d0 + ((dr[ring(P - 7)] + dr[ring(P - 5)]) + (left(d0) + right(d0)))) * 0.125;
        if (pl.useful && y4 >= pl.ra && y4 < pl.rb && !odd_t) {
          const size_t id = (size_t)y4 * wc + (x >> 1);
          a.fc[id] = inside(y4) ? v : 0.0;
          if (a.uc != nullptr) a.uc[id] = 0.0;
        }
        dr[ring(P - 4)] = r3;
      } else {
        if (pl.useful && t - 2 >= pl.ra && t - 2 < pl.rb) a.uout[(size_t)(t - 2) * m + x] = n2;
      }
      w1[ring(P)] = n1;
      w2[ring(P - 2)] = n2;
    };
    for (int t = ts; t <= te; t += kTurn)
      turn([&](auto pc) { step(t + decltype(pc)::value, pc); });
  }
  if (a.partials != nullptr) {
    const double tot = block_sum(acc);
    if (threadIdx.x == 0) a.partials[blockIdx.y * gridDim.x + blockIdx.x] = tot;
  }
}

template <bool NINE>
__global__ __launch_bounds__(kBlock) void k_rbc_post_std(PassArgs a) {
  constexpr int H = 3;
  if (a.done != nullptr && *a.done != 0) return;
  const int m = a.m, wc = (m + 1) / 2;
  const Place pl = place<H>(m, m, a.chunk);
  if (!pl.active) return;
  const int x = pl.x;
  const bool xin = x > 0 && x < m - 1;
  const int xs = min(max(x, 0), m - 1), xe = min(max(x >> 1, 0), wc - 1);
  // the corrected iterate at row t, F at t-2, C at t-4
  const int ts = pl.ra - 2, te = pl.rb - 1 + 4;
  const RbcOp op = a.op;
  auto row = [&](int y) { return (size_t)min(max(y, 0), m - 1); };
  auto at = [&](const double *p, int y) { return p[row(y) * m + xs]; };
  // row y of the rotated level below: its entry x >> 1 is the point of column x or the one
  // beside it
  auto ent = [&](int y) { return a.e[row(y) * wc + xe]; };
  double g0[kTurn], w1[kTurn], fr[kTurn], er[kTurn], uq[kAhead], fq[kAhead], eq[kAhead];
#pragma unroll
  for (int k = 0; k < kTurn; ++k) g0[k] = w1[k] = fr[k] = er[k] = 0.0;
  er[ring(-1)] = ent(ts - 1);
  er[ring(0)] = ent(ts);
#pragma unroll
  for (int k = 0; k < kAhead; ++k) {
    uq[k] = at(a.u, ts + k);
    fq[k] = at(a.f, ts + k);
    eq[k] = ent(ts + 1 + k);
  }
  auto inside = [&](int y) { return xin && y > 0 && y < m - 1; };
  auto step = [&](const int t, auto pc) {
    constexpr int P = decltype(pc)::value, Q = P % kAhead;
    double unew = uq[Q], fnew = fq[Q], enew = eq[Q];
    pin(unew);
    pin(fnew);
    pin(enew);
    __builtin_amdgcn_sched_barrier(0);
    uq[Q] = at(a.u, t + kAhead);
    fq[Q] = at(a.f, t + kAhead);
    eq[Q] = ent(t + 1 + kAhead);
    er[ring(P + 1)] = enew;
    fr[ring(P)] = fnew;
    const bool odd_t = ((x + t) & 1) != 0;
    const double e0 = er[ring(P)];
    const double side = (t & 1) == 0 ? e0 + right(e0) : left(e0) + e0;
    const double ef = 0.25 * ((er[ring(P - 1)] + er[ring(P + 1)]) + side);
    const double g = inside(t) ? unew + (odd_t ? ef : e0) : unew;
    const double r1 = fr[ring(P - 2)] - lap_std<NINE>(g0[ring(P - 3)], g0[ring(P - 2)], g0[ring(P - 1)], op);
    const double n1 = (inside(t - 2) && odd_t) ? g0[ring(P - 2)] + a.om * r1 : g0[ring(P - 2)];
    const double r2 = fr[ring(P - 4)] - lap_std<NINE>(w1[ring(P - 5)], w1[ring(P - 4)], w1[ring(P - 3)], op);
    const double n2 = (inside(t - 4) && !odd_t) ? w1[ring(P - 4)] + a.om * r2 : w1[ring(P - 4)];
    if (pl.useful && t - 4 >= pl.ra && t - 4 < pl.rb) a.uout[(size_t)(t - 4) * m + x] = n2;
    g0[ring(P)] = g;
    w1[ring(P - 2)] = n1;
  };
  for (int t = ts; t <= te; t += kTurn)
    turn([&](auto pc) { step(t + decltype(pc)::value, pc); });
}

// ------------------------------------------------------------------ rotated levels ----
// Column access of a packed rotated level: the C point (2p, 2k) and the F point
// (2p+1, 2k+1) of row pair p, extended oddly about the boundary lines (zero boundary).
struct RotColumn {
  int w;        // pitch = side of the C grid; the F grid has w - 1
  int kc, kf;   // folded columns
  double sc, sf;  // their signs (C: 0 on the boundary columns)
  __device__ __forceinline__ void init(int k, int w_) {
    w = w_;
    int c = k < 0 ? -k : k > w - 1 ? 2 * (w - 1) - k : k;
    c = min(max(c, 0), w - 1);
    kc = c;
    sc = c == 0 || c == w - 1 ? 0.0 : c == k ? 1.0 : -1.0;
    int f = k < 0 ? -1 - k : k > w - 2 ? 2 * w - 3 - k : k;
    f = min(max(f, 0), w - 2);
    kf = f;
    sf = f == k ? 1.0 : -1.0;
  }
  // row pair of the C / F row p after folding, and whether it is a mirror image
  __device__ __forceinline__ int rc(int p, bool &neg) const {
    const int q = p < 0 ? -p : p > w - 1 ? 2 * (w - 1) - p : p;
    neg = q != p;
    return min(max(q, 0), w - 1);
  }
  __device__ __forceinline__ int rf(int p, bool &neg) const {
    const int q = p < 0 ? -1 - p : p > w - 2 ? 2 * w - 3 - p : p;
    neg = q != p;
    return min(max(q, 0), w - 2);
  }
  // raw loads; sign_* turn a value into the extension's
  __device__ __forceinline__ double load_c(const double *a, int p) const {
    bool neg;
    return a[(size_t)(2 * rc(p, neg)) * w + kc];
  }
  __device__ __forceinline__ double load_f(const double *a, int p) const {
    bool neg;
    return a[(size_t)(2 * rf(p, neg) + 1) * w + kf];
  }
  __device__ __forceinline__ double sign_c(double v, int p) const {
    bool neg;
    const int q = rc(p, neg);
    return (q == 0 || q == w - 1) ? 0.0 : v * (neg ? -sc : sc);
  }
  __device__ __forceinline__ double sign_f(double v, int p) const {
    bool neg;
    (void)rf(p, neg);
    return v * (neg ? -sf : sf);
  }
  // the next (standard) level's point (p, k): the same grid as the C points
  __device__ __forceinline__ double load_e(const double *a, int p) const {
    bool neg;
    return a[(size_t)rc(p, neg) * w + kc];
  }
};

// L u at F row p from the C rows p, p+1 and the F rows p-1, p, p+1.
template <bool A2>
__device__ __forceinline__ double lap_f(double c0, double c1, double fm, double f, double fp, const RbcOp &op) {
  const double s = c0 + c1;
  double v = op.c0 * f + op.d1 * (s + right(s));
  if (A2) v += op.a2 * ((fm + fp) + (left(f) + right(f)));
  return v;
}
// L u at C row p from the F rows p-1, p and the C rows p-1, p, p+1.
template <bool A2>
__device__ __forceinline__ double lap_c(double f0, double f1, double cm, double c, double cp, const RbcOp &op) {
  const double s = f0 + f1;
  double v = op.c0 * c + op.d1 * (left(s) + s);
  if (A2) v += op.a2 * ((cm + cp) + (left(c) + right(c)));
  return v;
}

template <bool A2, bool HAS_U, bool RESTRICT>
__global__ __launch_bounds__(kBlock) void k_rbc_pre_rot(PassArgs a) {
  constexpr int H = RESTRICT ? 4 : 2;
  if (a.done != nullptr && *a.done != 0) return;
  const int w = (a.m + 1) / 2;
  const Place pl = place<H>(w, w, a.chunk);
  if (!pl.active) return;
  const int k = pl.x;
  RotColumn col;
  col.init(k, w);
  const bool kin = k > 0 && k < w - 1, fin = k < w - 1;
  // F at row pair t, C at t-1, the defect at t-3, the restriction at t-4
  const int ts = pl.ra - (RESTRICT ? 2 : 1), te = pl.rb - 1 + (RESTRICT ? 4 : 1);
  const RbcOp op = a.op;
  double C0[kTurn], F0[kTurn], C1[kTurn], F1[kTurn], gc[kTurn], gf[kTurn], dc[kTurn], df[kTurn];
  double cq[kAhead], fq[kAhead], gcq[kAhead], gfq[kAhead];
#pragma unroll
  for (int i = 0; i < kTurn; ++i) C0[i] = F0[i] = C1[i] = F1[i] = gc[i] = gf[i] = dc[i] = df[i] = 0.0;
  if (HAS_U) {
    C0[ring(0)] = col.sign_c(col.load_c(a.u, ts), ts);
    F0[ring(-1)] = col.sign_f(col.load_f(a.u, ts - 1), ts - 1);
    F0[ring(0)] = col.sign_f(col.load_f(a.u, ts), ts);
  }
#pragma unroll
  for (int i = 0; i < kAhead; ++i) {
    if (HAS_U) {
      cq[i] = col.load_c(a.u, ts + 1 + i);
      fq[i] = col.load_f(a.u, ts + 1 + i);
    }
    gcq[i] = col.load_c(a.f, ts + i);
    gfq[i] = col.load_f(a.f, ts + i);
  }
  auto cin = [&](int p) { return kin && p > 0 && p < w - 1; };
  auto step = [&](const int t, auto pc) {
    constexpr int P = decltype(pc)::value, Q = P % kAhead;
    double cn = HAS_U ? col.sign_c(cq[Q], t + 1) : 0.0, fn = HAS_U ? col.sign_f(fq[Q], t + 1) : 0.0;
    double gcn = col.sign_c(gcq[Q], t), gfn = col.sign_f(gfq[Q], t);
    pin(cn);
    pin(fn);
    pin(gcn);
    pin(gfn);
    __builtin_amdgcn_sched_barrier(0);
    if (HAS_U) {
      cq[Q] = col.load_c(a.u, t + 1 + kAhead);
      fq[Q] = col.load_f(a.u, t + 1 + kAhead);
    }
    gcq[Q] = col.load_c(a.f, t + kAhead);
    gfq[Q] = col.load_f(a.f, t + kAhead);
    C0[ring(P + 1)] = cn;
    F0[ring(P + 1)] = fn;
    gc[ring(P)] = gcn;
    gf[ring(P)] = gfn;
    const double f_ = F0[ring(P)];
    const double n1 = HAS_U ? f_ + a.om * (gfn - lap_f<A2>(C0[ring(P)], C0[ring(P + 1)], F0[ring(P - 1)], f_,
                                                         F0[ring(P + 1)], op))
                            : a.om * gfn;
    const double c_ = C0[ring(P - 1)];
    const double r2 = gc[ring(P - 1)] - lap_c<A2>(F1[ring(P - 2)], F1[ring(P - 1)], C0[ring(P - 2)], c_, C0[ring(P)], op);
    const double n2 = c_ + a.om * r2;  // 0 on the boundary lines: every term is odd about them
    if constexpr (RESTRICT) {
      const int q = t - 3, s = t - 4;
      const double rf = gf[ring(P - 3)] - lap_f<A2>(C1[ring(P - 3)], C1[ring(P - 2)], F1[ring(P - 4)], F1[ring(P - 3)],
                                                    F1[ring(P - 2)], op);
      const double rc = gc[ring(P - 3)] - lap_c<A2>(F1[ring(P - 4)], F1[ring(P - 3)], C1[ring(P - 4)], C1[ring(P - 3)],
                                                    C1[ring(P - 2)], op);
      if (pl.useful && q >= pl.ra && q < pl.rb) {
        a.uout[(size_t)(2 * q) * w + k] = cin(q) ? C1[ring(P - 3)] : 0.0;
        if (fin && q < w - 1) a.uout[(size_t)(2 * q + 1) * w + k] = F1[ring(P - 3)];
      }
      const double sf = df[ring(P - 5)] + df[ring(P - 4)];
      const double v = (4.0 * dc[ring(P - 4)] + (left(sf) + sf)) * 0.125;
      if (pl.useful && s >= pl.ra && s < pl.rb) {
        a.fc[(size_t)s * w + k] = cin(s) ? v : 0.0;
        if (a.uc != nullptr) a.uc[(size_t)s * w + k] = 0.0;
      }
      dc[ring(P - 3)] = rc;
      df[ring(P - 3)] = rf;
    } else {
      const int q = t - 1;
      if (pl.useful && q >= pl.ra && q < pl.rb) {
        a.uout[(size_t)(2 * q) * w + k] = cin(q) ? n2 : 0.0;
        if (fin && q < w - 1) a.uout[(size_t)(2 * q + 1) * w + k] = F1[ring(P - 1)];
      }
    }
    F1[ring(P)] = n1;
    C1[ring(P - 1)] = n2;
  };
  for (int t = ts; t <= te; t += kTurn)
    turn([&](auto pc) { step(t + decltype(pc)::value, pc); });
}

template <bool A2>
__global__ __launch_bounds__(kBlock) void k_rbc_post_rot(PassArgs a) {
  constexpr int H = 3;
  if (a.done != nullptr && *a.done != 0) return;
  const int w = (a.m + 1) / 2;
  const Place pl = place<H>(w, w, a.chunk);
  if (!pl.active) return;
  const int k = pl.x;
  RotColumn col;
  col.init(k, w);
  const bool kin = k > 0 && k < w - 1, fin = k < w - 1;
  // the corrected iterate at row pair t, F at t-2, C at t-3
  const int ts = pl.ra - 3, te = pl.rb - 1 + 3;
  const RbcOp op = a.op;
  double C0[kTurn], F0[kTurn], F1[kTurn], gc[kTurn], gf[kTurn], er[kTurn];
  double cq[kAhead], fq[kAhead], gcq[kAhead], gfq[kAhead], eq[kAhead];
#pragma unroll
  for (int i = 0; i < kTurn; ++i) C0[i] = F0[i] = F1[i] = gc[i] = gf[i] = er[i] = 0.0;
  er[ring(0)] = col.sign_c(col.load_e(a.e, ts), ts);
#pragma unroll
  for (int i = 0; i < kAhead; ++i) {
    cq[i] = col.load_c(a.u, ts + i);
    fq[i] = col.load_f(a.u, ts + i);
    gcq[i] = col.load_c(a.f, ts + i);
    gfq[i] = col.load_f(a.f, ts + i);
    eq[i] = col.load_e(a.e, ts + 1 + i);
  }
  auto step = [&](const int t, auto pc) {
    constexpr int P = decltype(pc)::value, Q = P % kAhead;
    double cn = col.sign_c(cq[Q], t), fn = col.sign_f(fq[Q], t);
    double gcn = col.sign_c(gcq[Q], t), gfn = col.sign_f(gfq[Q], t), en = col.sign_c(eq[Q], t + 1);
    pin(cn);
    pin(fn);
    pin(gcn);
    pin(gfn);
    pin(en);
    __builtin_amdgcn_sched_barrier(0);
    cq[Q] = col.load_c(a.u, t + kAhead);
    fq[Q] = col.load_f(a.u, t + kAhead);
    gcq[Q] = col.load_c(a.f, t + kAhead);
    gfq[Q] = col.load_f(a.f, t + kAhead);
    eq[Q] = col.load_e(a.e, t + 1 + kAhead);
    er[ring(P + 1)] = en;
    gc[ring(P)] = gcn;
    gf[ring(P)] = gfn;
    const double e0 = er[ring(P)];
    const double cc = cn + e0;
    const double ff = fn + 0.25 * ((e0 + right(e0)) + (en + right(en)));
    const double f_ = F0[ring(P - 2)];
    const double n1 = f_ + a.om * (gf[ring(P - 2)] - lap_f<A2>(C0[ring(P - 2)], C0[ring(P - 1)], F0[ring(P - 3)], f_,
                                                               F0[ring(P - 1)], op));
    const double c_ = C0[ring(P - 3)];
    const double n2 = c_ + a.om * (gc[ring(P - 3)] - lap_c<A2>(F1[ring(P - 4)], F1[ring(P - 3)], C0[ring(P - 4)], c_,
                                                               C0[ring(P - 2)], op));
    const int q = t - 3;
    if (pl.useful && q >= pl.ra && q < pl.rb) {
      a.uout[(size_t)(2 * q) * w + k] = (kin && q > 0 && q < w - 1) ? n2 : 0.0;
      if (fin && q < w - 1) a.uout[(size_t)(2 * q + 1) * w + k] = F1[ring(P - 3)];
    }
    C0[ring(P)] = cc;
    F0[ring(P)] = ff;
    F1[ring(P - 2)] = n1;
  };
  for (int t = ts; t <= te; t += kTurn)
    turn([&](auto pc) { step(t + decltype(pc)::value, pc); });
}

int cdiv(int a, int b) { return (a + b - 1) / b; }

// Rows per band.  A band of r rows marches r + extra row steps in turns of kTurn, so r =
// kTurn j - extra; the band with the fewest turns times rounds of resident blocks, and of
// those the one with the least work in all.  (One round in bands of at least four rows took
// 8.4 us for a post pass over a 129^2 rotated level, 16 steps; two rows, 8 steps, 6.6 us.)
int pass_rows(int rows, int across, int capacity, int extra) {
  int best = 0;
  long cost0 = 0, work0 = 0;
  for (int r = kTurn - extra % kTurn; r < rows + kTurn; r += kTurn) {
    if (r < 2) continue;
    const long blocks = (long)across * cdiv(rows, r), steps = r + extra;
    const long cost = (blocks + capacity - 1) / capacity * steps, work = blocks * steps;
    if (best == 0 || cost < cost0 || (cost == cost0 && work < work0)) {
      best = r;
      cost0 = cost;
      work0 = work;
    }
  }
  return best;
}

// Blocks across and bands; extra: row steps of a band beyond its rows.
template <typename K>
hipError_t launch(K kernel, PassArgs &a, int cols, int H, int extra, int *np, hipStream_t s) {
  dim3 grid(cdiv(cdiv(cols, kWave - 2 * H), kWaves));
  a.chunk = pass_rows(cols, grid.x, resident_blocks((const void *)kernel, kBlock, 0), extra);
  grid.y = cdiv(cols, a.chunk);
  if (np) *np = grid.x * grid.y;
  hipLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

}  // namespace

// Bands of a standard level have at least five rows (pass_rows with extra 3 or 9).
int rbc_pre_partials(int m) { return cdiv(cdiv(m, kWave - 8), kWaves) * cdiv(m, 5); }

hipError_t launch_rbc_pre(bool odd, const RbcOp &op, double omega, const double *f, const double *u,
                          double *uout, double *fc, double *uc, int m, double *partials, int *np,
                          const int *done, hipStream_t s) {
  if (m < kRbcPassSide || uout == u || uout == nullptr || f == nullptr) return hipErrorInvalidValue;
  PassArgs a{f, u, nullptr, uout, fc, uc, m, 0, op, omega / op.c0, odd ? nullptr : partials, done};
  const int cols = odd ? (m + 1) / 2 : m, H = fc != nullptr ? 4 : 2;
  const int extra = fc != nullptr ? (odd ? 6 : 9) : (odd ? 2 : 3);
  const bool wide = odd ? op.a2 != 0.0 : op.d1 != 0.0;
#define RBC_PRE(K, W)                                                                                        \
  return fc != nullptr ? (u != nullptr ? launch(K<W, true, true>, a, cols, H, extra, np, s)                         \
                                       : launch(K<W, false, true>, a, cols, H, extra, np, s))                       \
                       : (u != nullptr ? launch(K<W, true, false>, a, cols, H, extra, np, s)                        \
                                       : launch(K<W, false, false>, a, cols, H, extra, np, s))
  if (odd) {
    if (wide) RBC_PRE(k_rbc_pre_rot, true);
    RBC_PRE(k_rbc_pre_rot, false);
  }
  if (wide) RBC_PRE(k_rbc_pre_std, true);
  RBC_PRE(k_rbc_pre_std, false);
#undef RBC_PRE
}

hipError_t launch_rbc_post(bool odd, const RbcOp &op, double omega, const double *e, const double *uin,
                           const double *f, double *uout, int m, const int *done, hipStream_t s) {
  if (m < kRbcPassSide || uout == uin || uin == nullptr || e == nullptr || f == nullptr || uout == nullptr)
    return hipErrorInvalidValue;
  PassArgs a{f, uin, e, uout, nullptr, nullptr, m, 0, op, omega / op.c0, nullptr, done};
  const int cols = odd ? (m + 1) / 2 : m;
  if (odd)
    return op.a2 != 0.0 ? launch(k_rbc_post_rot<true>, a, cols, 3, 6, nullptr, s)
                        : launch(k_rbc_post_rot<false>, a, cols, 3, 6, nullptr, s);
  return op.d1 != 0.0 ? launch(k_rbc_post_std<true>, a, cols, 3, 6, nullptr, s)
                      : launch(k_rbc_post_std<false>, a, cols, 3, 6, nullptr, s);
}

}  // namespace mgk
