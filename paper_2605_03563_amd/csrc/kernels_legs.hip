// One leg of a 7-point V-cycle level in one launch, for levels of up to
// kLegMax intervals: the way down (nu1 red-black sweeps, residual, full
// weighting) and the way up (correction, nu2 sweeps, residual norm).
//
// What bounds these levels is launches: at 31^3 and 63^3 a colour pass takes
// 2.7-4.2 us whatever it moves, and a leg is five or six of them.  Here a
// block stages the 19^3 nodes around its own 8^3 in LDS and sweeps them there;
// each pass is valid on a region one node narrower per side than the one
// before, so the passes of one leg need no exchange between blocks.  The
// recomputed halo costs up to (17/8)^3 of the arithmetic, which LDS and the
// vector units do in less time than a launch takes; above kLegMax intervals
// it would cost more than the launches.  Blocks of 8^3 own nodes rather than
// 16^3, so that the 31^3 level still has 64 of them.
//
// Measured, V(2,2) with FP64: 31^3 down 10 us and up 10 us (five and six
// launches: 17 and 20 us), 63^3 with FP32 9 and 13 us (26 and 28 us).
//
// A leg reads one array and writes another, since neighbouring blocks read the
// values that a block replaces.
#include <type_traits>

#include "internal.h"
#include "reduce.h"

namespace psn {

namespace {

constexpr int kLegThreads = 1024;
constexpr int CB = 4;            // coarse nodes per block and axis
constexpr int OB = 2 * CB;       // fine nodes a block owns per axis
constexpr int D = OB + 11;       // staged nodes per axis: local x is array index 8 bx - 4 + x
constexpr int W = (D + 1) / 2;   // compact columns of a staged row
constexpr int P = D * W;         // a staged plane of one colour
constexpr int CS = D * P;        // a colour
constexpr int lo = 5, hi = lo + OB - 1;  // own nodes
constexpr int Q = (D - 1) / 2;   // nodes of one colour in a row, staged edge nodes excluded
constexpr int DI = D - 2;        // rows and planes without the staged edge
constexpr int SLOTS = Q * DI * DI;
constexpr int NR = (SLOTS + kLegThreads - 1) / kLegThreads;
constexpr int DC = (D + 1) / 2 + 1;  // coarse nodes per axis under the staged ones

// a block's place in the level (array offsets fit 32 bits: n <= kLegMax)
struct Place {
  int a, b, k;   // array indices of its local node (0, 0, 0); even
  int n, W, M, cs;
  __device__ Place(int bx, int by, int bz, const Geom& G)
      : a(OB * bx - 4), b(OB * by - 4), k(OB * bz - 4), n(G.n), W(G.W), M(G.M), cs((int)G.cs) {}
  __device__ bool in_x(int x) const { return (unsigned)(a + x - 1) < (unsigned)(n - 1); }  // unknowns
  __device__ bool in_row(int y, int z) const {
    return (unsigned)(b + y - 1) < (unsigned)(n - 1) && (unsigned)(k + z - 1) < (unsigned)(n - 1);
  }
  __device__ bool in(int x, int y, int z) const { return in_x(x) && in_row(y, z); }
  __device__ bool array(int x, int y, int z) const {  // a node of the level, ghosts included
    return (unsigned)(a + x) <= (unsigned)n && (unsigned)(b + y) <= (unsigned)n && (unsigned)(k + z) <= (unsigned)n;
  }
  // offset of compact column 0 of a local row in a colour's array
  __device__ int row(int y, int z) const { return ((k + z) * M + b + y) * W + (a >> 1); }
};

// The thread's nodes: slot tid + i 1024 is the t-th node of either colour in a
// local row (y, z) without the staged edge.  The colour of a local node is
// (x + y + z) & 1, as the block's first array index is even along every axis.
// What the passes need of a node is formed once: its LDS index, its array
// offset, on which side its second x-neighbour lies, and its distance from the
// middle of the own nodes, |2 x - lo - hi| at most over the axes (kFar where
// there is no unknown).  A pass is then one comparison and six LDS reads at
// constant offsets per node, and little code: these kernels run for so short a
// time that fetching their instructions is part of it.
constexpr int kFar = 1 << 20;
__device__ inline int off_middle(int x) { return abs(2 * x - lo - hi); }
template <typename T>
struct Own {
  int adr[2][NR], at[2][NR], dist[2][NR], odd[NR];
  T f[2][NR];
  __device__ Own(const Place& p, const T* __restrict__ F) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int slot = (int)threadIdx.x + i * kLegThreads;
      const int line = slot / Q, t = slot - line * Q;
      const int z = 1 + line / DI, y = 1 + line % DI;
      const bool row = z < D - 1 && p.in_row(y, z);
      const int far = row ? max(off_middle(y), off_middle(z)) : kFar;
      const int first = z * P + y * W, array = p.row(y, z);
      odd[i] = (y + z) & 1;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int x = 1 + ((c ^ odd[i]) ^ 1) + 2 * t;
        adr[c][i] = c * CS + first + (x >> 1);
        at[c][i] = array + (x >> 1);
        const bool ok = x < D - 1 && p.in_x(x);
        dist[c][i] = ok ? max(far, off_middle(x)) : kFar;
        f[c][i] = ok && row ? F[c * p.cs + at[c][i]] : (T)0;
      }
    }
  }
  // fn(i) for the unknowns of colour c at most d from the middle
  template <typename Fn>
  __device__ void each(int c, int d, Fn&& fn) const {
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (dist[c][i] <= d) fn(i);
  }
  // sum over the neighbours of node i of colour c: an even x has its second
  // x-neighbour one compact column to the left, an odd one to the right
  __device__ T neighbours(const T* u, int c, int i) const {
    const T* o = u + adr[c][i] + (c ? -CS : CS);
    return o[0] + o[2 * (c ^ odd[i]) - 1] + o[-W] + o[W] + o[-P] + o[P];
  }
  __device__ void relax(T* u, int c, int d, T h2) const {
    each(c, d, [&](int i) { u[adr[c][i]] = (neighbours(u, c, i) - h2 * f[c][i]) * (T)(1.0 / 6.0); });
    __syncthreads();
  }
  __device__ T residual(const T* u, int c, int i, T ih2) const {
    return f[c][i] - (neighbours(u, c, i) - (T)6 * u[adr[c][i]]) * ih2;
  }
  // the block's own nodes to X
  __device__ void store(const T* u, T* __restrict__ X, const Place& p) const {
#pragma unroll
    for (int c = 0; c < 2; ++c) each(c, OB - 1, [&](int i) { X[c * p.cs + at[c][i]] = u[adr[c][i]]; });
  }
};

// staged nodes of one colour per thread
constexpr int NS = (CS + kLegThreads - 1) / kLegThreads;
__device__ inline bool staged(int i, int c, int& x, int& y, int& z) {
  z = i / P;
  y = (i / W) % D;
  x = 2 * (i % W) + ((c - y - z) & 1);
  return i < CS && x < D;
}

// Stages colour c of X (the values a first pass over the other colour reads),
// all loads in flight together; nodes outside the level become zero.
template <typename T>
__device__ inline void stage(T* u, int c, const T* __restrict__ X, const Place& p) {
  T v[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    int x, y, z;
    const bool ok = staged((int)threadIdx.x + s * kLegThreads, c, x, y, z) && p.array(x, y, z);
    v[s] = ok ? X[c * p.cs + p.row(y, z) + (x >> 1)] : (T)0;
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = (int)threadIdx.x + s * kLegThreads;
    if (i < CS) u[c * CS + i] = v[s];
  }
}

// the ghost values of colour c, zero at its unknowns
template <typename T>
__device__ inline void stage_ghosts(T* u, int c, const T* __restrict__ X, const Place& p) {
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = (int)threadIdx.x + s * kLegThreads;
    int x, y, z;
    const bool ok = staged(i, c, x, y, z) && p.array(x, y, z) && !p.in(x, y, z);
    const T v = ok ? X[c * p.cs + p.row(y, z) + (x >> 1)] : (T)0;
    if (i < CS) u[c * CS + i] = v;
  }
}

// Way down: passes of colours 0, 1, ..., valid on the local nodes 4 - left ..
// 14 + left (left: passes still to come), then the residuals of colour 0 (the
// other colour's vanish) on 5 .. 13 and their full weighting.  The regions
// taken are symmetric about the own nodes, one node wider below; what those
// nodes get does not reach the valid ones.  ZG: zero guess and zero
// ghosts, Xin is not read.
template <typename T, bool ZG>
__global__ __launch_bounds__(kLegThreads) void k_down7(const T* __restrict__ Xin, T* __restrict__ X,
                                                       const T* __restrict__ F, Geom G, T* __restrict__ Fc, Geom Gc,
                                                       int nu, T h2, T ih2) {
  __shared__ T u[2 * CS];
  constexpr int R = OB + 2;  // from local node lo - 1
  __shared__ T r[R * R * R];
  int bx, by, bz;
  xcd_block(bx, by, bz);
  const int tid = threadIdx.x;
  const Place p(bx, by, bz, G);
  const Own<T> own(p, F);
  if constexpr (ZG) {
    for (int i = tid; i < 2 * CS; i += kLegThreads) u[i] = (T)0;
  } else {
    stage(u, 1, Xin, p);
    stage_ghosts(u, 0, Xin, p);
  }
  if (tid < R * R * R) r[tid] = (T)0;
  __syncthreads();
  for (int left = 2 * nu - 1; left > 0; left -= 2) {
    own.relax(u, 0, OB + 3 + 2 * left, h2);
    own.relax(u, 1, OB + 1 + 2 * left, h2);
  }
  own.each(0, OB + 1, [&](int i) {
    const int q = own.adr[0][i], z = q / P, y = (q / W) % D, x = 2 * (q % W) + own.odd[i];
    r[((z - lo + 1) * R + y - lo + 1) * R + x - lo + 1] = own.residual(u, 0, i, ih2);
  });
  own.store(u, X, p);
  __syncthreads();
  if (tid < CB * CB * CB) {
    const int I = tid % CB, J = (tid / CB) % CB, K = tid / (CB * CB);
    const int A = CB * bx + 1 + I, B = CB * by + 1 + J, C = CB * bz + 1 + K;
    if (A < Gc.n && B < Gc.n && C < Gc.n) {
      const T q = (T)0.25, hf = (T)0.5;
      const T* w = r + ((2 * K + 2) * R + 2 * J + 2) * R + 2 * I + 2;
      auto rx = [&](int dy, int dz) -> T {
        const T* x = w + (dz * R + dy) * R;
        return hf * x[0] + q * (x[-1] + x[1]);
      };
      auto ry = [&](int dz) -> T { return hf * rx(0, dz) + q * (rx(-1, dz) + rx(1, dz)); };
      T acc = q * ry(-1);
      acc += hf * ry(0);
      Fc[Gc.at(A, B, C)] = acc + q * ry(1);
    }
  }
}

// Way up: colour 0 of Xin corrected by the interpolated coarse potential, then
// passes of colours 1, 0, ... (the first reads no colour-1 unknown), the last
// one over the own nodes -- widened by one where the norm of colour 1's
// residuals (colour 0's vanish) is wanted, one partial sum per block.  Ghost:
// array holding the level's ghost values (nullptr: they are zero).
template <typename T, bool NORM>
__global__ __launch_bounds__(kLegThreads) void k_up7(const T* __restrict__ Xin, T* __restrict__ X,
                                                     const T* __restrict__ Ghost, const T* __restrict__ F, Geom G,
                                                     const T* __restrict__ Ec, Geom Gc, int nu, T h2, T ih2,
                                                     double* __restrict__ partial) {
  __shared__ T u[2 * CS];
  __shared__ T e[DC * DC * DC];
  int bx, by, bz;
  xcd_block(bx, by, bz);
  const int tid = threadIdx.x;
  const Place p(bx, by, bz, G);
  const Own<T> own(p, F);
  T ev[(DC * DC * DC + kLegThreads - 1) / kLegThreads];
#pragma unroll
  for (int i = tid, s = 0; s < (int)(sizeof ev / sizeof(T)); ++s, i += kLegThreads) {
    const int A = p.a / 2 + i % DC, B = p.b / 2 + (i / DC) % DC, C = p.k / 2 + i / (DC * DC);
    const bool in = (unsigned)(A - 1) < (unsigned)(Gc.n - 1) && (unsigned)(B - 1) < (unsigned)(Gc.n - 1) &&
                    (unsigned)(C - 1) < (unsigned)(Gc.n - 1);
    ev[s] = in ? Ec[Gc.at(A, B, C)] : (T)0;
  }
  // colour 0 of the iterate, or the level's ghost values
  T v[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    int x, y, z;
    const bool ok = staged(tid + s * kLegThreads, 0, x, y, z) && p.array(x, y, z);
    const bool in = p.in(x, y, z);
    v[s] = (T)0;
    if (ok && in) v[s] = Xin[p.row(y, z) + (x >> 1)];
    if (ok && !in && Ghost) v[s] = Ghost[p.row(y, z) + (x >> 1)];
  }
  if (Ghost) {
    stage_ghosts(u, 1, Ghost, p);
  } else {
    for (int i = tid; i < CS; i += kLegThreads) u[CS + i] = (T)0;
  }
#pragma unroll
  for (int i = tid, s = 0; s < (int)(sizeof ev / sizeof(T)); ++s, i += kLegThreads)
    if (i < DC * DC * DC) e[i] = ev[s];
  __syncthreads();
  const T half = (T)0.5;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = tid + s * kLegThreads;
    int x, y, z;
    if (staged(i, 0, x, y, z) && p.in(x, y, z)) {
      // the two coarse nodes of an even index coincide: the mean is exact
      const T* w = e + ((z >> 1) * DC + (y >> 1)) * DC + (x >> 1);
      const int dx = x & 1, dy = (y & 1) * DC, dz = (z & 1) * DC * DC;
      auto col = [&](const T* l) -> T {
        return half * (half * (l[0] + l[dy]) + half * (l[dz] + l[dz + dy]));
      };
      v[s] += half * (col(w) + col(w + dx));
    }
    if (i < CS) u[i] = v[s];
  }
  __syncthreads();
  constexpr int wide = NORM ? 2 : 0;
  for (int left = 2 * nu - 1; left > 0; left -= 2) {
    own.relax(u, 1, OB - 1 + wide + 2 * left, h2);
    own.relax(u, 0, OB - 3 + wide + 2 * left, h2);
  }
  own.store(u, X, p);
  if constexpr (NORM) {
    double acc = 0.0;
    own.each(1, OB - 1, [&](int i) {
      const T res = own.residual(u, 1, i, ih2);
      acc += (double)res * (double)res;
    });
    const double sum = block_sum(acc);
    if (tid == 0) partial[linear_block()] = sum;
  }
}

dim3 leg_grid(const Geom& G) {
  const unsigned nb = (unsigned)((G.n - 1 + OB - 1) / OB);
  return dim3(nb, nb, nb);
}

}  // namespace

bool legs_ok(const Geom& G, int nu1, int nu2) {
  return G.C == 2 && G.g == 1 && G.n >= 4 && G.n % 2 == 0 && G.n <= kLegMax && nu1 >= 1 && nu1 <= 2 && nu2 >= 1 &&
         nu2 <= 2;
}

int leg_blocks(const Geom& G) {
  const dim3 g = leg_grid(G);
  return (int)(g.x * g.y * g.z);
}

template <typename T>
static void down_t(const T* xin, T* x, const T* f, const Geom& G, T* fc, const Geom& Gc, int nu, hipStream_t st) {
  const T h2 = (T)(G.h * G.h), ih2 = (T)(1.0 / (G.h * G.h));
  if (xin)
    k_down7<T, false><<<leg_grid(G), kLegThreads, 0, st>>>(xin, x, f, G, fc, Gc, nu, h2, ih2);
  else
    k_down7<T, true><<<leg_grid(G), kLegThreads, 0, st>>>(xin, x, f, G, fc, Gc, nu, h2, ih2);
}

void leg_down(const void* xin, void* x, const void* f, bool f32, const Geom& G, void* fc, const Geom& Gc, int nu,
              hipStream_t st) {
  if (f32)
    down_t((const float*)xin, (float*)x, (const float*)f, G, (float*)fc, Gc, nu, st);
  else
    down_t((const double*)xin, (double*)x, (const double*)f, G, (double*)fc, Gc, nu, st);
}

template <typename T>
static void up_t(const T* xin, T* x, const T* ghost, const T* f, const Geom& G, const T* e, const Geom& Gc, int nu,
                 double* partial, hipStream_t st) {
  const T h2 = (T)(G.h * G.h), ih2 = (T)(1.0 / (G.h * G.h));
  if (partial)
    k_up7<T, true><<<leg_grid(G), kLegThreads, 0, st>>>(xin, x, ghost, f, G, e, Gc, nu, h2, ih2, partial);
  else
    k_up7<T, false><<<leg_grid(G), kLegThreads, 0, st>>>(xin, x, ghost, f, G, e, Gc, nu, h2, ih2, partial);
}

void leg_up(const void* xin, void* x, const void* ghost, const void* f, bool f32, const Geom& G, const void* e,
            const Geom& Gc, int nu, double* partial, hipStream_t st) {
  if (f32)
    up_t((const float*)xin, (float*)x, (const float*)ghost, (const float*)f, G, (const float*)e, Gc, nu, partial, st);
  else
    up_t((const double*)xin, (double*)x, (const double*)ghost, (const double*)f, G, (const double*)e, Gc, nu, partial,
         st);
}

}  // namespace psn
