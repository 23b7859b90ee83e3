// Multigrid with sparse-approximate-inverse (SPAI) smoothing on compact
// radius-1 stencils and Galerkin coarse operators (Section 2.1.3: the
// preconditioned Richardson iteration, the radius-1 smoother stencil M, the
// Galerkin operator R A P), on natural-layout level arrays.
//
// Every operator here is a cubically symmetric 27-point stencil given by its
// centre, face, edge and corner weights.  The kernels that sweep a level
// (smoothing step, residual norm, residual with full weighting) are marching
// wavefronts: lane l holds a column of a few rows in registers, x-neighbours
// come from the lanes beside by lane shifts, y-neighbours from the lane's own
// rows, and along z only two partial sums per row are carried.  No LDS and no
// barrier: the LDS-staged kernels before them waited at two barriers per plane
// and spent as long on LDS reads (27 per node) as on memory.  Measured at
// 511^3 / 255^3 / 127^3, FP64, us (before): step 804 (990) / 108 (134) / 20
// (27), residual and full weighting 545 (1159) / 61 (147) / 13 (18), norm 387
// (662, the rate of a plain read) / 47 (85) / 10 (12).
#include <algorithm>

#include "internal.h"
#include "reduce.h"

namespace psn {
namespace {

constexpr int BX = 64, BY = 4, KZ = 8;

// planes per block of the stored residual and the prolongation
inline int nkz(const NGeom& G) { return G.n >= 512 ? 32 : G.n >= 128 ? KZ : 1; }
inline dim3 ngrid(const NGeom& G) {
  const int e = G.n - 1;
  const int kz = nkz(G);
  return dim3((e + BX - 1) / BX, (e + BY - 1) / BY, (e + kz - 1) / kz);
}

struct Plane {
  double c, f, e;
};

// in-plane sums in FP64 whatever the storage type
template <typename T>
__device__ inline Plane plane_sums(const T* __restrict__ u, long long idx, int W) {
  auto v = [&](long long q) { return (double)u[q]; };
  Plane p;
  p.c = v(idx);
  p.f = (v(idx - 1) + v(idx + 1)) + (v(idx - W) + v(idx + W));
  p.e = (v(idx - W - 1) + v(idx - W + 1)) + (v(idx + W - 1) + v(idx + W + 1));
  return p;
}

__device__ inline double apply_sums(const W4& w, const Plane& m, const Plane& z, const Plane& p) {
  return w.c * z.c + w.f * (z.f + m.c + p.c) + w.e * (z.e + m.f + p.f) + w.k * (m.e + p.e);
}

// r = f - A u, stored, the squares summed into one partial per block (the
// residual operator; the cycles use k_nres_w).  A thread owns one (i, j) column
// and keeps the in-plane sums c = u(i, j), f = the 4 in-plane face neighbours,
// e = the 4 in-plane corners of three planes.
template <typename T>
__global__ __launch_bounds__(BX* BY) void k_n27(const T* __restrict__ src, const T* __restrict__ f,
                                                T* __restrict__ dst, NGeom G, W4 w, double* __restrict__ partial) {
  int bx, by, bz;
  xcd_block(bx, by, bz);
  const int i = 1 + bx * BX + (int)threadIdx.x;
  const int j = 1 + by * BY + (int)threadIdx.y;
  const int kz = (G.n - 1 + (int)gridDim.z - 1) / (int)gridDim.z;
  const int k0 = 1 + bz * kz;
  const int k1 = min(k0 + kz - 1, G.n - 1);
  double acc = 0.0;
  if (i < G.n && j < G.n && k0 <= k1) {
    Plane m = plane_sums(src, G.at(i, j, k0 - 1), G.W);
    Plane z = plane_sums(src, G.at(i, j, k0), G.W);
    for (int k = k0; k <= k1; ++k) {
      const long long idx = G.at(i, j, k);
      const Plane p = plane_sums(src, idx + G.P, G.W);
      const double s = apply_sums(w, m, z, p);
      const double r = (double)f[idx] - s;
      dst[idx] = (T)r;
      acc += r * r;
      m = z;
      z = p;
    }
  }
  const double b = block_sum(acc);
  if (threadIdx.x == 0 && threadIdx.y == 0) partial[linear_block()] = b;
}

// ---- marching wavefronts: rows in registers, x-neighbours from the lanes beside
// The value of the lane to the left (DIR < 0) or right; the wavefront's edge
// lane gets zero.
template <int DIR>
__device__ inline double lane_shift(double v) {
  constexpr int ctrl = DIR < 0 ? 0x138 : 0x130;  // wave_shr:1, wave_shl:1
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), ctrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), ctrl, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ inline double beside(double v) { return lane_shift<-1>(v) + lane_shift<1>(v); }

// One fused Richardson step out of place: out = u - M (f - A u) at the unknowns
// (Eq. richardson).  A wavefront owns SX = 60 columns and R rows and marches
// the planes of its run with no LDS and no barrier: lane l holds column
// x0 - 2 + l of R + 4 rows of u (loaded one plane ahead), forms r on 62 columns
// and R + 2 rows and the output on 60 and R, x-neighbours by lane shifts and
// y-neighbours from its own rows.  Along z a stencil applied to plane q is split into what
// it gives to its own plane, a = w_c c + w_f f + w_e e, and to the two beside,
// b = w_f c + w_e f + w_k e, so two partial sums per row are all the state.
// Four wavefronts stacked in y share their halo rows through the cache.
// ZG: u is zero (a coarse level's first step): it is not read.
constexpr int SX = 60;
template <typename T, int R, bool ZG>
__global__ __launch_bounds__(256) void k_nspai_w(const T* __restrict__ u, const T* __restrict__ f,
                                                 T* __restrict__ out, NGeom G, W4 A, W4 M) {
  int bx, by, bz;
  xcd_block(bx, by, bz);
  const int n = G.n, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int gx = 1 + bx * SX - 2 + lane;
  const int y0 = 1 + (by * 4 + wave) * R;  // first output row
  const int kz = (n - 1 + (int)gridDim.z - 1) / (int)gridDim.z;
  const int kb = 1 + bz * kz, ke = min(kb + kz - 1, n - 1);
  if (y0 > n - 1 || kb > ke) return;
  const bool xin = gx >= 1 && gx <= n - 1;
  const bool mine = xin && lane >= 2 && lane < 2 + SX;
  const int cx = min(max(gx, 0), n);  // loads stay in the array
  const bool ux = gx >= 0 && gx <= n;
  double un[R + 4], fn[R + 2];         // the next plane's rows
  auto load_u = [&](int q) {
    if (ZG) return;
    const T* p = u + (long long)min(max(q, 0), n) * G.P + cx;
#pragma unroll
    for (int i = 0; i < R + 4; ++i) un[i] = (double)p[(long long)min(max(y0 - 2 + i, 0), n) * G.W];
  };
  auto load_f = [&](int q) {
    const T* p = f + (long long)min(max(q, 1), n - 1) * G.P + cx;
#pragma unroll
    for (int i = 0; i < R + 2; ++i) fn[i] = (double)p[(long long)min(max(y0 - 1 + i, 1), n - 1) * G.W];
  };
  double rp[R + 2], rb[R + 2];  // r: sum so far for the plane before, its b
  double op[R], ob[R], u1[R], u2[R];
#pragma unroll
  for (int i = 0; i < R + 2; ++i) rp[i] = rb[i] = 0.0;
#pragma unroll
  for (int i = 0; i < R; ++i) op[i] = ob[i] = u1[i] = u2[i] = 0.0;
  load_u(kb - 2);
  load_f(kb - 1);
  for (int q = kb - 2; q <= ke + 2; ++q) {
    double c[R + 4], h[R + 4];
    const bool qin = q >= 0 && q <= n;
#pragma unroll
    for (int i = 0; i < R + 4; ++i) {
      const int y = y0 - 2 + i;
      c[i] = !ZG && qin && y >= 0 && y <= n && ux ? un[i] : 0.0;
    }
    double fc[R + 2];
#pragma unroll
    for (int i = 0; i < R + 2; ++i) fc[i] = fn[i];
    if (q < ke + 2) load_u(q + 1);
    if (q >= kb && q <= ke + 1) load_f(q);
#pragma unroll
    for (int i = 0; i < R + 4; ++i) h[i] = ZG ? 0.0 : beside(c[i]);
    // r on plane q - 1
    double r[R + 2];
    const bool rin = q - 1 >= 1 && q - 1 <= n - 1;
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {
      const double fs = h[i + 1] + (c[i] + c[i + 2]), es = h[i] + h[i + 2];
      const double b = A.f * c[i + 1] + A.e * fs + A.k * es;
      const int y = y0 - 1 + i;
      r[i] = rin && xin && y >= 1 && y <= n - 1 ? fc[i] - (rp[i] + b) : 0.0;
      rp[i] = A.c * c[i + 1] + A.f * fs + A.e * es + rb[i];
      rb[i] = b;
    }
    double g[R + 2];
#pragma unroll
    for (int i = 0; i < R + 2; ++i) g[i] = beside(r[i]);
    // output on plane q - 2
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const double fs = g[i + 1] + (r[i] + r[i + 2]), es = g[i] + g[i + 2];
      const double b = M.f * r[i + 1] + M.e * fs + M.k * es;
      const int y = y0 + i;
      if (q >= kb + 2 && mine && y <= n - 1)
        __builtin_nontemporal_store((T)(u2[i] - (op[i] + b)), out + G.at(gx, y, q - 2));
      op[i] = M.c * r[i + 1] + M.f * fs + M.e * es + ob[i];
      ob[i] = b;
      u2[i] = u1[i];
      u1[i] = c[i + 2];
    }
  }
}

// r = f - A u, marching as k_nspai_w: R rows and 62 columns of r per wavefront.
// NORM: one partial sum of r^2 per block.  Otherwise the residual is fully
// weighted onto the coarse grid without being stored (Gf.n even, R odd: the
// fine rows 2 J0 - 1 .. 2 J0 + R - 2 of (R - 1) / 2 coarse rows; 30 coarse columns on the even
// fine ones): weights 1, 2, 1 along each axis, over 64.
template <typename T, typename TC, int R, bool NORM>
__global__ __launch_bounds__(256) void k_nres_w(const T* __restrict__ u, const T* __restrict__ f, NGeom G, W4 A,
                                                TC* __restrict__ fc, NGeom Gc, double* __restrict__ partial) {
  constexpr int RC = (R - 1) / 2;          // coarse rows per wavefront
  constexpr int RX = NORM ? 62 : 60;       // columns a wavefront advances
  constexpr int RY = NORM ? R : R - 1;     // rows
  int bx, by, bz;
  xcd_block(bx, by, bz);
  const int n = G.n, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int gx = bx * RX + lane;                 // lanes 1 .. 62 hold r
  const int y0 = 1 + (by * 4 + wave) * RY;       // first row of r
  const int runs = (int)gridDim.z;
  // planes of r: kb .. ke (restriction: from an odd plane to an odd plane)
  int kb, ke;
  if (NORM) {
    const int kz = (n - 1 + runs - 1) / runs;
    kb = 1 + bz * kz;
    ke = min(kb + kz - 1, n - 1);
  } else {
    const int kz = (Gc.n - 1 + runs - 1) / runs, K0 = 1 + bz * kz;
    kb = 2 * K0 - 1;
    ke = 2 * min(K0 + kz - 1, Gc.n - 1) + 1;
  }
  const bool work = y0 <= n - 1 && kb <= ke;
  double acc = 0.0;
  if (work) {
    const bool xin = gx >= 1 && gx <= n - 1 && lane >= 1 && lane <= 62;
    const int cx = min(gx, n);
    double un[R + 2], fn[R];
    auto load_u = [&](int q) {
      const T* p = u + (long long)min(q, n) * G.P + cx;
#pragma unroll
      for (int i = 0; i < R + 2; ++i) un[i] = (double)p[(long long)min(y0 - 1 + i, n) * G.W];
    };
    auto load_f = [&](int q) {
      const T* p = f + (long long)min(max(q, 1), n - 1) * G.P + cx;
#pragma unroll
      for (int i = 0; i < R; ++i) fn[i] = (double)p[(long long)min(y0 + i, n - 1) * G.W];
    };
    double rp[R], rb[R], z0[RC > 0 ? RC : 1];
#pragma unroll
    for (int i = 0; i < R; ++i) rp[i] = rb[i] = 0.0;
#pragma unroll
    for (int i = 0; i < RC; ++i) z0[i] = 0.0;
    load_u(kb - 1);
    load_f(kb);
    // plane q of u completes r on plane q - 1
    for (int q = kb - 1; q <= ke + 1; ++q) {
      double c[R + 2], h[R + 2], fr[R];
#pragma unroll
      for (int i = 0; i < R + 2; ++i) c[i] = gx <= n && y0 - 1 + i <= n ? un[i] : 0.0;
#pragma unroll
      for (int i = 0; i < R; ++i) fr[i] = fn[i];
      if (q <= ke) load_u(q + 1);
      if (q > kb && q <= ke) load_f(q);
#pragma unroll
      for (int i = 0; i < R + 2; ++i) h[i] = beside(c[i]);
      const int k = q - 1;
      double r[R];
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const double fs = h[i + 1] + (c[i] + c[i + 2]), es = h[i] + h[i + 2];
        const double b = A.f * c[i + 1] + A.e * fs + A.k * es;
        r[i] = xin && y0 + i <= n - 1 && k >= kb && k <= n - 1 ? fr[i] - (rp[i] + b) : 0.0;
        if (NORM && k >= kb) acc += r[i] * r[i];
        rp[i] = A.c * c[i + 1] + A.f * fs + A.e * es + rb[i];
        rb[i] = b;
      }
      if constexpr (!NORM) {
        double x[R];
#pragma unroll
        for (int i = 0; i < R; ++i) x[i] = 2.0 * r[i] + beside(r[i]);
#pragma unroll
        for (int i = 0; i < RC; ++i) {
          const double p = x[2 * i] + 2.0 * x[2 * i + 1] + x[2 * i + 2];
          if (k & 1) {  // closes coarse plane (k - 1) / 2 and opens the next
            const int J = (y0 + 1) / 2 + i, I = gx >> 1;
            if (k > kb && !(gx & 1) && lane >= 2 && lane <= 60 && I >= 1 && I < Gc.n && J < Gc.n)
              fc[Gc.at(I, J, (k - 1) >> 1)] = (TC)((z0[i] + p) * (1.0 / 64.0));
            z0[i] = p;
          } else {
            z0[i] += 2.0 * p;
          }
        }
      }
    }
  }
  if constexpr (NORM) {
    const double s = block_sum(acc);
    if (threadIdx.x == 0) partial[linear_block()] = s;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_ncopy(const T* __restrict__ a, T* __restrict__ b, long long count) {
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < count; i += (long long)gridDim.x * 256) b[i] = a[i];
}

// fine u += trilinear interpolation of the coarse correction (P = 8 R^T).
// A thread owns a fine (i, j) column and marches k: b_K, the sum of the four
// coarse values around (i, j) on coarse plane K (each counted twice when i or
// j is even), is formed once per coarse plane; fine plane 2K takes 2 b_K,
// plane 2K+1 takes b_K + b_{K+1}, both times 1/8.
template <typename TC, typename TF>
__global__ __launch_bounds__(BX* BY) void k_nprolong(const TC* __restrict__ uc, NGeom Gc, TF* __restrict__ uf,
                                                     NGeom Gf) {
  int bx, by, bz;
  xcd_block(bx, by, bz);
  const int i = 1 + bx * BX + (int)threadIdx.x;
  const int j = 1 + by * BY + (int)threadIdx.y;
  const int kz = (Gf.n - 1 + (int)gridDim.z - 1) / (int)gridDim.z;
  const int k0 = 1 + bz * kz;
  const int k1 = min(k0 + kz - 1, Gf.n - 1);
  if (i >= Gf.n || j >= Gf.n || k0 > k1) return;
  const int i0 = i >> 1, j0 = j >> 1;
  const int i1 = i0 + (i & 1), j1 = j0 + (j & 1);
  auto bsum = [&](int K) {
    return ((double)uc[Gc.at(i0, j0, K)] + (double)uc[Gc.at(i1, j0, K)]) +
           ((double)uc[Gc.at(i0, j1, K)] + (double)uc[Gc.at(i1, j1, K)]);
  };
  int Kc = k0 >> 1;
  double bc = bsum(Kc), bn = bsum(Kc + 1);
  for (int k = k0; k <= k1; ++k) {
    if ((k >> 1) != Kc) {
      Kc = k >> 1;
      bc = bn;
      bn = bsum(Kc + 1);
    }
    const double s = (k & 1) ? (bc + bn) : 2.0 * bc;
    const long long q = Gf.at(i, j, k);
    uf[q] = (TF)((double)uf[q] + 0.125 * s);
  }
}

// coarsest level: u = A^-1 f with the dense inverse, one wavefront per row;
// add (here and below): u += A^-1 f
template <typename T>
__global__ __launch_bounds__(256) void k_ncoarse(const double* __restrict__ inv, const T* __restrict__ f,
                                                 T* __restrict__ u, NGeom G, int add) {
  const int E = G.n - 1;
  const int N = E * E * E;
  const int row = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= N) return;
  double acc = 0.0;
  for (int col = lane; col < N; col += 64) {
    const int i = col % E, j = (col / E) % E, k = col / (E * E);
    acc += inv[(long long)row * N + col] * (double)f[G.at(i + 1, j + 1, k + 1)];
  }
  acc = wave_sum(acc);
  if (lane == 0) {
    const int i = row % E, j = (row / E) % E, k = row / (E * E);
    T* x = u + G.at(i + 1, j + 1, k + 1);
    *x = (T)(add ? (double)*x + acc : acc);
  }
}

// coarsest level by conjugate gradients on A = -L (SPD) from a zero guess,
// one block, everything in LDS: p with a zero ghost layer, x, r, q.  Stops
// once ||r|| <= rtol ||f|| or after maxit steps (Section 2.1.2's CG as the
// coarsest solve of Section 2.1.3).  Sums are block reductions in a fixed
// order.
template <typename T>
__global__ __launch_bounds__(1024) void k_ncg(const T* __restrict__ f, T* __restrict__ u, NGeom G, W4 A,
                                              double rtol, int maxit, int add) {
  extern __shared__ double sh[];
  __shared__ double bc;
  const int E = G.n - 1, EP = E + 2, N = E * E * E;
  double* pp = sh;
  double* x = pp + EP * EP * EP;
  double* r = x + N;
  double* q = r + N;
  const int tid = threadIdx.x, nt = blockDim.x;
  auto pad = [&](int c) {
    const int i = c % E, j = (c / E) % E, k = c / (E * E);
    return ((k + 1) * EP + (j + 1)) * EP + (i + 1);
  };
  auto at = [&](int c) {
    const int i = c % E, j = (c / E) % E, k = c / (E * E);
    return G.at(i + 1, j + 1, k + 1);
  };
  for (int c = tid; c < EP * EP * EP; c += nt) pp[c] = 0.0;
  __syncthreads();
  double part = 0.0;
  for (int c = tid; c < N; c += nt) {
    const double v = (double)f[at(c)];
    x[c] = 0.0;
    r[c] = v;
    pp[pad(c)] = v;
    part += v * v;
  }
  auto allsum = [&](double v) {
    const double s = block_sum(v);
    if (tid == 0) bc = s;
    __syncthreads();
    const double out = bc;
    __syncthreads();
    return out;
  };
  double rr = allsum(part);
  const double stop = rtol * rtol * rr;
  for (int it = 0; it < maxit && rr > stop; ++it) {
    part = 0.0;
    for (int c = tid; c < N; c += nt) {
      const int o = pad(c);
      const double* b = pp + o;
      double fc = 0.0, ec = 0.0, kc = 0.0;
      for (int dz = -1; dz <= 1; ++dz)
        for (int dy = -1; dy <= 1; ++dy)
          for (int dx = -1; dx <= 1; ++dx) {
            const int nz = (dx != 0) + (dy != 0) + (dz != 0);
            const double v = b[(dz * EP + dy) * EP + dx];
            if (nz == 1) fc += v;
            else if (nz == 2) ec += v;
            else if (nz == 3) kc += v;
          }
      const double qv = -(A.c * b[0] + A.f * fc + A.e * ec + A.k * kc);
      q[c] = qv;
      part += b[0] * qv;
    }
    const double alpha = rr / allsum(part);
    part = 0.0;
    for (int c = tid; c < N; c += nt) {
      x[c] -= alpha * pp[pad(c)];
      r[c] -= alpha * q[c];
      part += r[c] * r[c];
    }
    const double rr_new = allsum(part);
    const double beta = rr_new / rr;
    for (int c = tid; c < N; c += nt) pp[pad(c)] = r[c] + beta * pp[pad(c)];
    __syncthreads();
    rr = rr_new;
  }
  for (int c = tid; c < N; c += nt) u[at(c)] = (T)(add ? (double)u[at(c)] + x[c] : x[c]);
}

// caller node array (one ghost layer, pitches p0, p1) -> level array;
// interior zeroed when zero_inner
__global__ __launch_bounds__(BX* BY) void k_nin(const double* __restrict__ src, long long p0, long long p1,
                                                double* __restrict__ u, NGeom G, int zero_inner) {
  const int i = blockIdx.x * BX + (int)threadIdx.x;
  const int j = blockIdx.y * BY + (int)threadIdx.y;
  const int k = blockIdx.z;
  if (i > G.n || j > G.n || k > G.n) return;
  const bool inner = i > 0 && i < G.n && j > 0 && j < G.n && k > 0 && k < G.n;
  u[G.at(i, j, k)] = (zero_inner && inner) ? 0.0 : src[k * p1 + j * p0 + i];
}

// right-hand side at the unknowns: scale * B rho, with B
//   order 2: the identity;
//   order 4: (6 rho_n + sum of the 6 face neighbours) / 12;
//   order 6: (402 rho_n + 40 (6 face neighbours) - 3 (6 axis nodes at
//            distance 2) + 8 (12 in-plane diagonals)) / 720, i.e.
//            rho + D/12 - D^2/240 + (mixed D_d D_e)/90 collected per node
//            (D the unit-spacing second differences); reads rho two nodes
//            beyond the unknowns.
__global__ __launch_bounds__(BX* BY) void k_nrhs(const double* __restrict__ rho, long long p0, long long p1,
                                                 double* __restrict__ f, NGeom G, int order, double scale) {
  const int i = 1 + blockIdx.x * BX + (int)threadIdx.x;
  const int j = 1 + blockIdx.y * BY + (int)threadIdx.y;
  const int k = 1 + blockIdx.z;
  if (i >= G.n || j >= G.n || k >= G.n) return;
  const long long q = k * p1 + j * p0 + i;
  double v = rho[q];
  if (order == 4) {
    v = (6.0 * v + ((rho[q - 1] + rho[q + 1]) + (rho[q - p0] + rho[q + p0]) + (rho[q - p1] + rho[q + p1]))) *
        (1.0 / 12.0);
  } else if (order == 6) {
    const double f1 = (rho[q - 1] + rho[q + 1]) + (rho[q - p0] + rho[q + p0]) + (rho[q - p1] + rho[q + p1]);
    const double f2 =
        (rho[q - 2] + rho[q + 2]) + (rho[q - 2 * p0] + rho[q + 2 * p0]) + (rho[q - 2 * p1] + rho[q + 2 * p1]);
    const double exy = (rho[q - p0 - 1] + rho[q - p0 + 1]) + (rho[q + p0 - 1] + rho[q + p0 + 1]);
    const double exz = (rho[q - p1 - 1] + rho[q - p1 + 1]) + (rho[q + p1 - 1] + rho[q + p1 + 1]);
    const double eyz = (rho[q - p1 - p0] + rho[q - p1 + p0]) + (rho[q + p1 - p0] + rho[q + p1 + p0]);
    v = (402.0 * v + 40.0 * f1 - 3.0 * f2 + 8.0 * (exy + exz + eyz)) * (1.0 / 720.0);
  }
  f[G.at(i, j, k)] = scale * v;
}

__global__ __launch_bounds__(BX* BY) void k_nout(const double* __restrict__ u, NGeom G, double* __restrict__ dst,
                                                 long long p0, long long p1) {
  const int i = 1 + blockIdx.x * BX + (int)threadIdx.x;
  const int j = 1 + blockIdx.y * BY + (int)threadIdx.y;
  const int k = 1 + blockIdx.z;
  if (i >= G.n || j >= G.n || k >= G.n) return;
  dst[k * p1 + j * p0 + i] = u[G.at(i, j, k)];
}

inline dim3 inner_grid(const NGeom& G) { return dim3((G.n - 1 + BX - 1) / BX, (G.n - 1 + BY - 1) / BY, G.n - 1); }

}  // namespace

NGeom make_ngeom(int n, double h) {
  NGeom G{};
  G.n = n;
  G.W = (n + 1 + 31) / 32 * 32;
  G.P = (long long)(n + 1) * G.W;
  G.h = h;
  return G;
}

long long n27_blocks(const NGeom& G) {
  const dim3 g = ngrid(G);
  return (long long)g.x * g.y * g.z;
}

void n27_residual(const double* u, const double* f, double* r, const NGeom& G, const W4& A, double* partial,
                  hipStream_t st) {
  k_n27<double><<<ngrid(G), dim3(BX, BY), 0, st>>>(u, f, r, G, A, partial);
}

// Rows per wavefront R and planes per run kz of the marching kernels: more
// rows share more of a row's loads, fewer and shorter runs give a small level
// enough wavefronts.  Step at 127^3 20 us with (R, kz) = (4, 4), 23 with (2, 4), 29
// with (4, 16); at 255^3 108 with (4, 16), 125 with (4, 4), 125 with (2, 16);
// at 511^3 804 with (4, 32), 888 with (2, 32), 956 with (4, 256); at 31^3 5.8
// with (2, 1), 7.8 with (2, 4); at 63^3 8.2 with (2, 4), 11 with (2, 1).  The
// lines at 48, 96, 160 and 384 lie between tuned sizes; a step there is 1.14
// (48), 1.21 (96), 1.29 (160) and 1.19 (384) times as fast as the LDS tiles were.
struct March {
  int R, kz;
};
static March step_march(int n) {
  return n < 48 ? March{2, 1} : n < 96 ? March{2, 4} : n < 160 ? March{4, 4} : n < 384 ? March{4, 16} : March{4, 32};
}

template <typename T, int R>
static void spai_step_go(const T* u, const T* f, T* out, const NGeom& G, const W4& A, const W4& M, int kz,
                         hipStream_t st) {
  const int e = G.n - 1;
  const dim3 gr((e + SX - 1) / SX, (e + 4 * R - 1) / (4 * R), (e + kz - 1) / kz);
  if (u)
    k_nspai_w<T, R, false><<<gr, 256, 0, st>>>(u, f, out, G, A, M);
  else
    k_nspai_w<T, R, true><<<gr, 256, 0, st>>>(u, f, out, G, A, M);
}
template <typename T>
static void spai_step_t(const T* u, const T* f, T* out, const NGeom& G, const W4& A, const W4& M, hipStream_t st) {
  const March m = step_march(G.n);
  if (m.R == 2)
    spai_step_go<T, 2>(u, f, out, G, A, M, m.kz, st);
  else
    spai_step_go<T, 4>(u, f, out, G, A, M, m.kz, st);
}

void n_spai_step(const void* u, const void* f, void* out, bool f32, const NGeom& G, const W4& A, const W4& M,
                 hipStream_t st) {
  if (f32)
    spai_step_t<float>((const float*)u, (const float*)f, (float*)out, G, A, M, st);
  else
    spai_step_t<double>((const double*)u, (const double*)f, (double*)out, G, A, M, st);
}

// As the step's rule: norm at 63^3 4.7 us with (4, 2), 5.2 with (4, 1); at 127^3 9.8
// with (4, 4), 11.7 with (4, 2); at 255^3 47 with (4, 16), 52 with (4, 4).
static March norm_march(int n) {
  return n < 48 ? March{2, 1} : n < 96 ? March{4, 2} : n < 160 ? March{4, 4} : n < 384 ? March{4, 16} : March{4, 32};
}
int n27_norm(const double* u, const double* f, const NGeom& G, const W4& A, double* partial, hipStream_t st) {
  const March m = norm_march(G.n);
  const int e = G.n - 1;
  const dim3 gr((e + 61) / 62, (e + 4 * m.R - 1) / (4 * m.R), (e + m.kz - 1) / m.kz);
  if (m.R == 2)
    k_nres_w<double, double, 2, true><<<gr, 256, 0, st>>>(u, f, G, A, nullptr, G, partial);
  else
    k_nres_w<double, double, 4, true><<<gr, 256, 0, st>>>(u, f, G, A, nullptr, G, partial);
  return (int)(gr.x * gr.y * gr.z);
}

// Rows of r (2 or 4 fine rows advance, R - 1) and coarse planes per run: 4.5 us at
// 31^3 with (3, 1), 5.3 with (5, 1); at 127^3 12.6 with (5, 2), 14.0 with (3,
// 4); at 255^3 61 with (5, 8), 69 with (5, 16); at 511^3 545 with (5, 16), 578 with (5, 2).
template <typename T, typename TC>
static void resrestrict_t(const T* u, const T* f, const NGeom& G, const W4& A, TC* fc, const NGeom& Gc,
                          hipStream_t st) {
  const March m = G.n < 96 ? March{3, 1} : G.n < 160 ? March{5, 2} : G.n < 384 ? March{5, 8} : March{5, 16};
  const int e = Gc.n - 1, rc = (m.R - 1) / 2;
  const dim3 gr((e + 29) / 30, (e + 4 * rc - 1) / (4 * rc), (e + m.kz - 1) / m.kz);
  if (m.R == 3)
    k_nres_w<T, TC, 3, false><<<gr, 256, 0, st>>>(u, f, G, A, fc, Gc, nullptr);
  else
    k_nres_w<T, TC, 5, false><<<gr, 256, 0, st>>>(u, f, G, A, fc, Gc, nullptr);
}

void n_resrestrict(const void* u, const void* f, bool f32, const NGeom& G, const W4& A, void* fc, bool f32_coarse,
                   const NGeom& Gc, hipStream_t st) {
  if (f32)  // the levels below an FP32 level are FP32
    resrestrict_t((const float*)u, (const float*)f, G, A, (float*)fc, Gc, st);
  else if (f32_coarse)
    resrestrict_t((const double*)u, (const double*)f, G, A, (float*)fc, Gc, st);
  else
    resrestrict_t((const double*)u, (const double*)f, G, A, (double*)fc, Gc, st);
}

void n_copy(const void* a, void* b, bool f32, const NGeom& G, hipStream_t st) {
  const long long count = G.total();
  const long long blocks = std::min<long long>((count + 255) / 256, 65536);
  if (f32)
    k_ncopy<float><<<(unsigned)blocks, 256, 0, st>>>((const float*)a, (float*)b, count);
  else
    k_ncopy<double><<<(unsigned)blocks, 256, 0, st>>>((const double*)a, (double*)b, count);
}

void n_prolong_add(const void* uc, bool f32_coarse, const NGeom& Gc, void* uf, bool f32_fine, const NGeom& Gf,
                   hipStream_t st) {
  const dim3 gr = ngrid(Gf), bl(BX, BY);
  if (f32_coarse && f32_fine)
    k_nprolong<float, float><<<gr, bl, 0, st>>>((const float*)uc, Gc, (float*)uf, Gf);
  else if (f32_coarse && !f32_fine)
    k_nprolong<float, double><<<gr, bl, 0, st>>>((const float*)uc, Gc, (double*)uf, Gf);
  else if (!f32_coarse && !f32_fine)
    k_nprolong<double, double><<<gr, bl, 0, st>>>((const double*)uc, Gc, (double*)uf, Gf);
  else
    k_nprolong<double, float><<<gr, bl, 0, st>>>((const double*)uc, Gc, (float*)uf, Gf);
}

void n_coarse(const double* inv, const void* f, void* u, bool f32, const NGeom& G, hipStream_t st, bool add) {
  const int E = G.n - 1;
  const int N = E * E * E;
  if (f32)
    k_ncoarse<float><<<(N + 3) / 4, 256, 0, st>>>(inv, (const float*)f, (float*)u, G, add);
  else
    k_ncoarse<double><<<(N + 3) / 4, 256, 0, st>>>(inv, (const double*)f, (double*)u, G, add);
}

size_t n_cg_lds_bytes(const NGeom& G) {
  const size_t E = G.n - 1, EP = E + 2;
  return sizeof(double) * (EP * EP * EP + 3 * E * E * E);
}

void n_coarse_cg(const void* f, void* u, bool f32, const NGeom& G, const W4& A, double rtol, hipStream_t st,
                 bool add) {
  const int E = G.n - 1;
  const int maxit = 2 * E * E * E;
  const size_t lds = n_cg_lds_bytes(G);
  if (f32)
    k_ncg<float><<<1, 1024, lds, st>>>((const float*)f, (float*)u, G, A, rtol, maxit, add);
  else
    k_ncg<double><<<1, 1024, lds, st>>>((const double*)f, (double*)u, G, A, rtol, maxit, add);
}

// Caller arrays hold `ghost` layers; node 0 of the level (the first ghost
// layer) sits ghost - 1 nodes in along every axis.
static long long node0(int ghost, long long p0, long long p1) { return (long long)(ghost - 1) * (p1 + p0 + 1); }

void n_from_caller(const double* src, long long p0, long long p1, int ghost, double* u, const NGeom& G,
                   bool zero_inner, hipStream_t st) {
  k_nin<<<dim3((G.n + 1 + BX - 1) / BX, (G.n + 1 + BY - 1) / BY, G.n + 1), dim3(BX, BY), 0, st>>>(
      src + node0(ghost, p0, p1), p0, p1, u, G, zero_inner ? 1 : 0);
}

void n_rhs(const double* rho, long long p0, long long p1, int ghost, double* f, const NGeom& G, int order,
           double scale, hipStream_t st) {
  k_nrhs<<<inner_grid(G), dim3(BX, BY), 0, st>>>(rho + node0(ghost, p0, p1), p0, p1, f, G, order, scale);
}

void n_to_caller(const double* u, const NGeom& G, double* dst, long long p0, long long p1, int ghost,
                 hipStream_t st) {
  k_nout<<<inner_grid(G), dim3(BX, BY), 0, st>>>(u, G, dst + node0(ghost, p0, p1), p0, p1);
}

}  // namespace psn
