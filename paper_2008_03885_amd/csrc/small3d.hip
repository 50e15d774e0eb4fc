// small3d.hip -- the rediscretized (radius-2 cross) 3D levels of few points: one point, one
// defect or one pair of points per thread, every input loaded at once.
//
// The marching kernels of kernels3d.hip reuse each plane from registers and LDS, which is
// what a level needs whose planes come from memory.  A level of up to kSmallSide points per
// side lies in the caches whole and has too few columns to fill the chip: there a march of
// eight planes is a chain of eight loads, barriers and stores behind the launch.  Here all
// threads of the level run at once and wait for one set of loads; the neighbours' lines
// come from L1 and L2.
//
// Measured (FP64, from -> to, us): sweep 65^3 7.3 -> 5.6, 33^3 6.7 -> 4.0; defect and full
// weighting 65^3 6.4 -> 6.2, 33^3 6.3 -> 4.6; interpolation 65^3 8.0 -> 5.9, 33^3 7.6 -> 4.8;
// a 65^3 V(2,1) solve 2328 -> 1840.
//
// The odd extension across the Dirichlet boundary (u(-i) = -u(i), boundary values zero) and
// the order of the sums are those of the marching kernels.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "mg_internal.h"

namespace mgk {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ bool stopped(const int *done) { return done != nullptr && *done != 0; }

// Row and column of point e of a plane of n^2 points (exact: e < 2^22 here).
__device__ __forceinline__ int row_of(int e, float rn) { return (int)(((float)e + 0.5f) * rn); }

// Sum over the block (valid in thread 0).
__device__ double block_sum(double v) {
  __shared__ double ws[kThreads / 64];
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < kThreads / 64; ++w) t += ws[w];
  return t;
}

// The neighbours of an interior point along one axis: coordinate x, stride st.  A
// neighbour past the boundary is read as the point itself and negated, one on it is 0.
template <typename T>
struct Axis {
  T m2, m1, p1, p2;
  __device__ __forceinline__ void load(const T *u, size_t id, int x, int n, size_t st) {
    m1 = u[x > 1 ? id - st : id];
    p1 = u[x < n - 2 ? id + st : id];
    m2 = u[x > 2 ? id - 2 * st : id];
    p2 = u[x < n - 3 ? id + 2 * st : id];
  }
  __device__ __forceinline__ void extend(int x, int n) {
    m1 = x > 1 ? m1 : T(0);
    p1 = x < n - 2 ? p1 : T(0);
    m2 = x > 2 ? m2 : (x == 1 ? -m2 : T(0));
    p2 = x < n - 3 ? p2 : (x == n - 2 ? -p2 : T(0));
  }
  __device__ __forceinline__ void scale(T s) {
#pragma clang fp contract(off)
    m1 = m1 * s;
    p1 = p1 * s;
    m2 = m2 * s;
    p2 = p2 * s;
  }
};

// c and L u at the interior point (x, y, z); scaled: u is scale * (the array), rounded as a
// stored iterate would be.
template <typename T, bool SCALED>
__device__ __forceinline__ T cross_lu(const T *u, int x, int y, int z, int n, const KOp<T> &op, T &c) {
#pragma clang fp contract(off)
  const size_t st = (size_t)n * n, id = (size_t)z * st + (size_t)y * n + x;
  Axis<T> ax, ay, az;
  c = u[id];
  ax.load(u, id, x, n, 1);
  ay.load(u, id, y, n, n);
  az.load(u, id, z, n, st);
  ax.extend(x, n);
  ay.extend(y, n);
  az.extend(z, n);
  if (SCALED) {
    c = c * op.om_d;
    ax.scale(op.om_d);
    ay.scale(op.om_d);
    az.scale(op.om_d);
  }
  const T d1 = ((c - ax.m1) + (c - ax.p1)) + ((c - ay.m1) + (c - ay.p1)) + ((c - az.m1) + (c - az.p1));
  const T d2 = ((c - ax.m2) + (c - ax.p2)) + ((c - ay.m2) + (c - ay.p2)) + ((c - az.m2) + (c - az.p2));
  return fma(op.w2, d2, op.w1 * d1);
}

// One sweep, defect or norm (SweepMode); grid (blocks of a plane, planes).
template <typename T, typename TO, int MODE>
__global__ __launch_bounds__(kThreads) void k_ssweep3d(const T *__restrict__ f, const T *__restrict__ u,
                                                       TO *__restrict__ out, int n, float rn, KOp<T> op,
                                                       double *__restrict__ partials,
                                                       const int *__restrict__ done) {
  if (stopped(done)) return;
  const Block2 blk = block2();
  const int e = blk.x * kThreads + threadIdx.x, z = blk.y;
  const int y = row_of(e, rn), x = e - y * n;
  const bool inside = x > 0 && x < n - 1 && y > 0 && y < n - 1 && z > 0 && z < n - 1;
  const size_t id = (size_t)z * n * n + e;
  double acc = 0.0;
  if (inside) {
    T c;
    const T fz = f[id];
    const T lu = cross_lu<T, MODE == kSweepZ2>(MODE == kSweepZ2 ? f : u, x, y, z, n, op, c);
    const T r = fz - lu;
    if (partials != nullptr) acc = (double)r * (double)r;
    if (MODE == kSweep || MODE == kSweepZ2) out[id] = (TO)(c + op.om_d * r);
    if (MODE == kSweepRB) out[id] = (TO)(c + colour_om(op, x + y + z) * r);
    if (MODE == kResidual) out[id] = (TO)r;
    if (MODE == kSweepCorr) {  // out is the FP64 iterate: add the sweep's result as stored
      T e1 = c + op.om_d * r;
      asm volatile("" : "+v"(e1));
      out[id] += (TO)e1;
    }
  } else if (MODE != kNormOnly && MODE != kSweepCorr && y < n) {
    out[id] = (TO)0;
  }
  if (partials != nullptr) {
    const double tot = block_sum(acc);
    if (threadIdx.x == 0) partials[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = tot;
  }
}

// Defect and full weighting: the block's CX x CY x CZ coarse points, one defect of their
// support (765 points) per thread, weighted from LDS.  Two coarse planes per block: with
// four (1377 points, three passes of 512 threads) 33^3 takes 5.7 us and not 4.6.
constexpr int kCX = 8, kCY = 4, kCZ = 2, kRrThreads = 768;
template <typename T, bool HAS_U>
__global__ __launch_bounds__(kRrThreads) void k_srr3d(const T *__restrict__ f, const T *__restrict__ u,
                                                      T *__restrict__ fc, int n, KOp<T> op,
                                                      const int *__restrict__ done) {
  constexpr int DX = 2 * kCX + 1, DY = 2 * kCY + 1, DZ = 2 * kCZ + 1, DS = DX * DY * DZ;
  __shared__ T d[DS];
  if (stopped(done)) return;
  const int nc = (n - 1) / 2 + 1;
  const Block3 blk = block3();
  const int I0 = 1 + blk.x * kCX, J0 = 1 + blk.y * kCY, K0 = 1 + blk.z * kCZ;
  static_assert(DS <= kRrThreads, "one defect per thread");
  const int e = threadIdx.x;
  if (e < DS) {
    const int x = 2 * I0 - 1 + e % DX, y = 2 * J0 - 1 + e / DX % DY, z = 2 * K0 - 1 + e / (DX * DY);
    T r = T(0);
    if (x < n - 1 && y < n - 1 && z < n - 1) {
      T c;
      r = f[((size_t)z * n + y) * n + x];
      if (HAS_U) r -= cross_lu<T, false>(u, x, y, z, n, op, c);
    }
    d[e] = r;
  }
  __syncthreads();
  // the first tiles also store the boundary plane, row and column 0
  constexpr int SX = kCX + 1, SY = kCY + 1, SZ = kCZ + 1;
  static_assert(SX * SY * SZ <= kRrThreads, "one coarse point per thread");
  const int t = threadIdx.x;
  const int i = t % SX - 1, j = t / SX % SY - 1, k = t / (SX * SY) - 1;
  const int I = I0 + i, J = J0 + j, K = K0 + k;
  if (k >= kCZ || I >= nc || J >= nc || K >= nc) return;
  if ((i < 0 && blk.x != 0) || (j < 0 && blk.y != 0) || (k < 0 && blk.z != 0)) return;
  T v = T(0);
  if (I > 0 && I < nc - 1 && J > 0 && J < nc - 1 && K > 0 && K < nc - 1) {
    const T *q = d + ((2 * k + 1) * DY + 2 * j + 1) * DX + 2 * i + 1;
    T p[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      T s[3];
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const T *w = q + ((c - 1) * DY + b - 1) * DX;
        s[b] = T(0.25) * w[-1] + T(0.5) * w[0] + T(0.25) * w[1];
      }
      p[c] = T(0.25) * s[0] + T(0.5) * s[1] + T(0.25) * s[2];
    }
    v = T(0.25) * p[0] + T(0.5) * p[1] + T(0.25) * p[2];
  }
  fc[((size_t)K * nc + J) * nc + I] = v;
}

// Interpolation of order P and correction.  A thread takes the fine points 2I and 2I+1 of
// one row; blockIdx.y is the parity of the row and the plane, so that a block's threads read
// the same 1, 4 or 16 coarse rows each (the class with 16 first).  uout may be uin.
template <typename T, int P>
__global__ __launch_bounds__(kThreads) void k_sprolong3d(const T *__restrict__ v, const T *uin, T *uout, int n,
                                                         float rnc1, float rnc, const int *__restrict__ done) {
  if (stopped(done)) return;
  const int nc = (n - 1) / 2 + 1;
  const int py = (blockIdx.y & 1) ^ 1, pz = (blockIdx.y >> 1) ^ 1;
  const int e = blockIdx.x * kThreads + threadIdx.x;
  const int jk = row_of(e, rnc1), I = e - jk * (nc - 1);
  const int K = row_of(jk, rnc), J = jk - K * nc;
  const int y = 2 * J + py, z = 2 * K + pz;
  if (y > n - 1 || z > n - 1) return;
  const size_t row = ((size_t)z * n + y) * n;
  T *o = uout + row + 2 * I;
  if (I == nc - 2) o[2] = T(0);
  if (y == 0 || y == n - 1 || z == 0 || z == n - 1) {
    o[0] = T(0);
    o[1] = T(0);
    return;
  }
  const T u0 = uin[row + 2 * I], u1 = uin[row + 2 * I + 1];
  // coarse index i of the odd extension: address and sign (0 on the boundary)
  auto fold1 = [&](int i, T &s) {
    s = (i <= 0 || i >= nc - 1) ? (i == 0 || i == nc - 1 ? T(0) : T(-1)) : T(1);
    return i < 0 ? -i : (i > nc - 1 ? 2 * (nc - 1) - i : i);
  };
  constexpr int A0 = P == 3 ? 0 : 1, A1 = P == 3 ? 4 : 3;  // taps of an odd point
  const T wt[4] = {P == 3 ? T(-0.0625) : T(0), P == 3 ? T(0.5625) : T(0.5), P == 3 ? T(0.5625) : T(0.5),
                   P == 3 ? T(-0.0625) : T(0)};
  int xi[4];
  T xs[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) xi[a] = fold1(I - 1 + a, xs[a]);
  auto rows = [&](auto ny, auto nz) {  // taps in y and z: 1 or all
    constexpr bool OY = decltype(ny)::value, OZ = decltype(nz)::value;
    constexpr int B0 = OY ? A0 : 1, B1 = OY ? A1 : 2, C0 = OZ ? A0 : 1, C1 = OZ ? A1 : 2;
    T g[4][4][4];
    T ys[4], zs[4];
    int yi[4], zi[4];
#pragma unroll
    for (int b = B0; b < B1; ++b) yi[b] = fold1(J - 1 + b, ys[b]) * nc;
#pragma unroll
    for (int c = C0; c < C1; ++c) zi[c] = fold1(K - 1 + c, zs[c]) * nc * nc;
#pragma unroll
    for (int c = C0; c < C1; ++c)
#pragma unroll
      for (int b = B0; b < B1; ++b)
#pragma unroll
        for (int a = A0; a < A1; ++a) g[c][b][a] = v[zi[c] + yi[b] + xi[a]];
    T he = T(0), ho = T(0);
#pragma unroll
    for (int c = C0; c < C1; ++c) {
      T pe = T(0), po = T(0);
#pragma unroll
      for (int b = B0; b < B1; ++b) {
        T re = xs[1] * g[c][b][1], ro = T(0);
#pragma unroll
        for (int a = A0; a < A1; ++a) ro += wt[a] * (xs[a] * g[c][b][a]);
        const T w = OY ? wt[b] * ys[b] : ys[b];
        pe += w * re;
        po += w * ro;
      }
      const T w = OZ ? wt[c] * zs[c] : zs[c];
      he += w * pe;
      ho += w * po;
    }
    o[0] = I > 0 ? u0 + he : T(0);
    o[1] = u1 + ho;
  };
  if (py && pz)
    rows(std::true_type{}, std::true_type{});
  else if (py)
    rows(std::true_type{}, std::false_type{});
  else if (pz)
    rows(std::false_type{}, std::true_type{});
  else
    rows(std::false_type{}, std::false_type{});
}

int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

template <typename T>
KOp<T> to_kop(const LevelOp &op, double omega, int colour) {
  KOp<T> k = {};
  k.w1 = (T)(-op.a[2]);
  k.w2 = (T)(-op.a[1]);
  k.om_d = (T)(omega / op.diag);
  k.colour = colour;
  return k;
}

}  // namespace

int small3d_partials(int n) { return cdiv((long)n * n, kThreads) * n; }

template <typename T, typename TO>
hipError_t launch_small_sweep_3d(int mode, const LevelOp &op, double omega, const T *f, const T *u, TO *out,
                                 int n, double *partials, int *nparts, const int *done, hipStream_t s,
                                 int colour) {
  const dim3 grid(cdiv((long)n * n, kThreads), n);
  if (nparts) *nparts = grid.x * grid.y;
  const KOp<T> k = to_kop<T>(op, omega, colour);
  const float rn = 1.0f / (float)n;
#define MG_SS(MODE) \
  hipLaunchKernelGGL((k_ssweep3d<T, TO, MODE>), grid, dim3(kThreads), 0, s, f, u, out, n, rn, k, partials, done)
  if (mode == kResidual) {
    MG_SS(kResidual);
    return hipGetLastError();
  }
  if constexpr (std::is_same_v<T, TO>) {  // FP64 in, FP32 out: the defect of a refinement step only
    if (mode == kSweep) MG_SS(kSweep);
    else if (mode == kSweepRB) MG_SS(kSweepRB);
    else if (mode == kSweepZ2) MG_SS(kSweepZ2);
    else if (mode == kNormOnly) MG_SS(kNormOnly);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
#undef MG_SS
}

hipError_t launch_small_sweep_corr_3d(const LevelOp &op, double omega, const float *f, const float *e,
                                      double *u64, int n, const int *done, hipStream_t s) {
  const dim3 grid(cdiv((long)n * n, kThreads), n);
  hipLaunchKernelGGL((k_ssweep3d<float, double, kSweepCorr>), grid, dim3(kThreads), 0, s, f, e, u64, n,
                     1.0f / (float)n, to_kop<float>(op, omega, 0), nullptr, done);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_small_resid_restrict_3d(const LevelOp &op, const T *f, const T *u, T *fc, int n,
                                          const int *done, hipStream_t s) {
  const int nc = (n - 1) / 2 + 1;
  const dim3 grid(cdiv(nc - 1, kCX), cdiv(nc - 1, kCY), cdiv(nc - 1, kCZ));
  const KOp<T> k = to_kop<T>(op, 1.0, 0);
  if (u != nullptr)
    hipLaunchKernelGGL((k_srr3d<T, true>), grid, dim3(kRrThreads), 0, s, f, u, fc, n, k, done);
  else
    hipLaunchKernelGGL((k_srr3d<T, false>), grid, dim3(kRrThreads), 0, s, f, u, fc, n, k, done);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_small_prolong_3d(int prolong, const T *v, const T *uin, T *uout, int n, const int *done,
                                   hipStream_t s) {
  const int nc = (n - 1) / 2 + 1;
  const dim3 grid(cdiv((long)(nc - 1) * nc * nc, kThreads), 4);
  const float rnc1 = 1.0f / (float)(nc - 1), rnc = 1.0f / (float)nc;
  if (prolong == 3)
    hipLaunchKernelGGL((k_sprolong3d<T, 3>), grid, dim3(kThreads), 0, s, v, uin, uout, n, rnc1, rnc, done);
  else
    hipLaunchKernelGGL((k_sprolong3d<T, 1>), grid, dim3(kThreads), 0, s, v, uin, uout, n, rnc1, rnc, done);
  return hipGetLastError();
}

#define MG_INST(T, TO)                                                                                     \
  template hipError_t launch_small_sweep_3d<T, TO>(int, const LevelOp &, double, const T *, const T *, TO *, \
                                                   int, double *, int *, const int *, hipStream_t, int);
MG_INST(double, double)
MG_INST(float, float)
MG_INST(double, float)
#undef MG_INST
template hipError_t launch_small_resid_restrict_3d<double>(const LevelOp &, const double *, const double *,
                                                           double *, int, const int *, hipStream_t);
template hipError_t launch_small_resid_restrict_3d<float>(const LevelOp &, const float *, const float *,
                                                          float *, int, const int *, hipStream_t);
template hipError_t launch_small_prolong_3d<double>(int, const double *, const double *, double *, int,
                                                    const int *, hipStream_t);
template hipError_t launch_small_prolong_3d<float>(int, const float *, const float *, float *, int,
                                                   const int *, hipStream_t);

}  // namespace mgk
