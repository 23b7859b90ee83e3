// The small levels of a Cartesian V-cycle in one workgroup (Section 2.1.3):
// every level from the tail's top level down to the coarsest one is smoothed,
// restricted, solved and prolonged inside one launch, with the potentials in
// LDS.
//
// What bounds these levels is latency: a colour pass over 15^3 unknowns moves
// 30 KB, but as a launch of its own it takes 2.5-3.5 us plus the gap to the
// next one, and a V(2,2) cycle on a 16- and an 8-interval level needs 12 such
// launches (21 on four-colour levels).  Here a pass is a few hundred LDS
// reads per wavefront and one barrier.  One workgroup of 1024 threads, because
// a barrier inside a workgroup costs ~0.1 us and one across workgroups
// several; no level above 24 intervals or 160 KB of LDS, where a pass by one
// compute unit costs as much as a launch.
//
// Measured, FP64, levels of 16 and 8 intervals: 15 us (7-point) and 29 us
// (star) for one V(2,2) cycle, of which 3 us wait for the right-hand side and
// the blocks, 0.7 / 1 us are one pass, 4 us the coarsest solve; launched one by
// one the same kernels took 41 and 95 us.  A register spill in this kernel
// costs more than anything else: unrolled code (28 KB) was no faster than
// loops (15 KB).
//
// The coarsest solve is the exact inverse in the basis of even and odd
// functions along each axis.  The operators commute with the three mirror
// images of the box, so the inverse splits into eight blocks, and with the
// exchange of axes, so blocks with equally many odd axes are alike: 343
// unknowns need 8425 matrix entries (67 KB, read into LDS while the levels
// above are smoothed) instead of 117.6 thousand (0.94 MB).
#include <math.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "reduce.h"

namespace psn {

namespace {

constexpr int kTailThreads = 1024;
constexpr size_t kTailLds = 160 * 1024;  // LDS of one compute unit
constexpr int kTailCoarseMax = 1024;     // coarsest unknowns: one thread per row of the inverse

constexpr double kC0 = -49.0 / 18.0, kC1 = 1.5, kC2 = -3.0 / 20.0, kC3 = 1.0 / 90.0;  // 19-point star

// sectors of the coarsest inverse: bit d of s set = odd along axis d; E / 2 odd
// functions per axis and E - E / 2 even ones
inline int sector_odd(int s) { return (s & 1) + ((s >> 1) & 1) + (s >> 2); }
inline int sector_size(int E, int s) {
  int n = 1;
  for (int d = 0; d < 3; ++d) n *= (s >> d) & 1 ? E / 2 : E - E / 2;
  return n;
}

// A level inside the tail, sized for NT intervals at compile time so that a
// node's neighbours are LDS reads at constant offsets from one address (with
// runtime pitches the address arithmetic, not LDS, bounds a pass).  The layout
// is the colour-split one of Geom with the row pitch cut to the compact
// columns: rows of nine FP64 columns for 16 intervals, so 64 lanes reading
// consecutive nodes of a colour rarely meet on a bank.  Levels of fewer
// intervals use the same arrays partly.
template <typename T, int C, int NT>
struct Lev {
  static constexpr int lc = C == 2 ? 1 : 2;
  static constexpr int g = C == 2 ? 1 : 3;
  static constexpr int M = NT + 1 + 2 * (g - 1);
  static constexpr int W = (M + C - 1) / C;
  static constexpr int P = M * W;
  static constexpr int CS = M * P;
  static constexpr int ED = NT - 1;                       // pitch of natural-order arrays
  static constexpr int Q = (ED + C - 1) / C;              // nodes of one colour per row, at most
  static constexpr int SLOTS = Q * ED * ED;               // (node, row, plane) triples of one colour
  static constexpr int NR = (SLOTS + kTailThreads - 1) / kTailThreads;
  static constexpr int U = C * CS;
  static constexpr int off = ((-3 * (g - 1)) % C + C) % C;  // as make_geom
  // row and plane of a slot, counted from 0, and the number of its node
  __device__ static void decode(int slot, int& t, int& j, int& k) {
    const int line = slot / Q;
    t = slot - line * Q;
    k = line / ED;
    j = line - k * ED;
  }
  __device__ static int row(int j, int k) { return (k + g) * P + (j + g) * W; }
  __device__ static int shift(int j, int k) { return j + k + 2 * g + off; }
  // the t-th unknown of colour c in a row of shift s
  __device__ static int node(int c, int s, int t) { return g + ((c - s - g) & (C - 1)) + C * t; }
  // u at the grid node (i, j, k), counted from the box face
  __device__ static T at(const T* u, int i, int j, int k) {
    const int a = i + g - 1, b = j + g - 1, kk = k + g - 1;
    return u[((a + b + kk + off) & (C - 1)) * CS + kk * P + b * W + (a >> lc)];
  }
  // sums over the neighbours of the colour-c node a of the row at u: the six
  // nearest (two colours), or those at distance 1, 2 and 3 (four)
  __device__ static void sums(const T* u, int c, int a, T* s) {
    const int m = a >> lc;
    if constexpr (C == 2) {
      const T* o = u + (c ^ 1) * CS + m;
      s[0] = o[0] + o[2 * (a & 1) - 1] + o[-W] + o[W] + o[-P] + o[P];
    } else {
      const int q = a & 3;
      const T* o1 = u + ((c + 1) & 3) * CS + m;
      const T* o2 = u + ((c + 2) & 3) * CS + m;
      const T* o3 = u + ((c + 3) & 3) * CS + m;
      s[0] = o1[q == 3 ? 1 : 0] + o3[q == 0 ? -1 : 0] + o1[W] + o3[-W] + o1[P] + o3[-P];
      s[1] = o2[q >= 2 ? 1 : 0] + o2[q <= 1 ? -1 : 0] + o2[2 * W] + o2[-2 * W] + o2[2 * P] + o2[-2 * P];
      s[2] = o3[q >= 1 ? 1 : 0] + o1[q <= 2 ? -1 : 0] + o3[3 * W] + o1[-3 * W] + o3[3 * P] + o1[-3 * P];
    }
  }
  __device__ static T relaxed(const T* u, int c, int a, T f, T h2) {
    T s[3];
    sums(u, c, a, s);
    if constexpr (C == 2)
      return (s[0] - h2 * f) * (T)(1.0 / 6.0);
    else
      return (h2 * f - ((T)kC1 * s[0] + (T)kC2 * s[1] + (T)kC3 * s[2])) * (T)(1.0 / (3.0 * kC0));
  }
  __device__ static T residual(const T* u, int c, int a, T f, T ih2) {
    T s[3];
    sums(u, c, a, s);
    const T uc = u[c * CS + (a >> lc)];
    if constexpr (C == 2)
      return f - (s[0] - (T)6 * uc) * ih2;
    else
      return f - ((T)(3.0 * kC0) * uc + (T)kC1 * s[0] + (T)kC2 * s[1] + (T)kC3 * s[2]) * ih2;
  }
};

// LDS offsets (elements) of a tail sized for NT intervals whose lowest level
// holds at least kTailLow intervals: every level's potential, then the
// right-hand sides below the top, then the residual and coarsest vectors
constexpr int kTailLow = 4;
template <typename T, int C, int NT, int L>
struct Arena {
  static constexpr int u = Arena<T, C, NT * 2, L - 1>::u + Lev<T, C, NT * 2>::U;
  static constexpr int f = Arena<T, C, NT * 2, L - 1>::f + (L > 1 ? (NT * 2 - 1) * (NT * 2 - 1) * (NT * 2 - 1) : 0);
};
template <typename T, int C, int NT>
struct Arena<T, C, NT, 0> {
  static constexpr int u = 0, f = 0;
};

// Trilinear interpolation at fine grid node (i, j, k) of the coarse values
// val(I, J, K).  The two coarse nodes of an even index coincide and their mean
// is exact, so no lane takes another path than its neighbours.
template <typename T, typename Val>
__device__ inline T interpolate(int i, int j, int k, Val&& val) {
  const T half = (T)0.5;
  const int I = i >> 1, J = j >> 1, K = k >> 1, I1 = (i + 1) >> 1, J1 = (j + 1) >> 1, K1 = (k + 1) >> 1;
  auto column = [&](int A) -> T {
    return half * (half * (val(A, J, K) + val(A, J1, K)) + half * (val(A, J, K1) + val(A, J1, K1)));
  };
  return half * (column(I) + column(I1));
}

// Full weighting of the residual r (pitch ED) at the coarse unknown (I, J, K),
// all counted from 0.
template <int ED, typename T>
__device__ inline T full_weight(const T* r, int I, int J, int K) {
  const T q = (T)0.25, hf = (T)0.5;
  const T* p = r + ((2 * K + 1) * ED + 2 * J + 1) * ED + 2 * I + 1;
  auto rx = [&](int dy, int dz) -> T {
    const T* x = p + (dz * ED + dy) * ED;
    return hf * x[0] + q * (x[-1] + x[1]);
  };
  auto ry = [&](int dz) -> T { return hf * rx(0, dz) + q * (rx(-1, dz) + rx(1, dz)); };
  T acc = q * ry(-1);
  acc += hf * ry(0);
  return acc + q * ry(1);
}

// What thread p N + q does in the coarsest solve (a table of the N parts
// threads that do anything precedes the blocks): it multiplies the columns p,
// p + parts, ... of row q of the blocks (sector by sector).
struct CoarseRow {
  int row;   // natural index of row q | first row of its sector << 16
  int part;  // size of the sector | p << 16 (size 0: nothing to do)
  int col;   // entry (j, q) of the block at col + j size
  int ijk;   // coordinates of the node with natural index q, eight bits each
};
// Threads per row: no more than the largest sector has columns, so that few
// unknowns (1, 8 or 27) don't leave one thread a thousand empty parts to add up.
inline int coarse_parts(int E) { return std::min(kTailThreads / (E * E * E), sector_size(E, 0)); }
// doubles of the table; a single unknown's row needs none
inline size_t row_table(int E) {
  return E == 1 ? 0 : (size_t)E * E * E * coarse_parts(E) * sizeof(CoarseRow) / sizeof(double);
}

// Coarsest solve: f (pitch ED) into e, natural order with pitch ED + 2 and a
// layer of zeros around the unknowns.  v: N + 1024 doubles; blocks: in LDS, or
// in global memory where they do not fit there.
template <typename LC, typename T>
__device__ inline void coarse_blocks(T* e, const T* f, double* v, const double* __restrict__ blocks, CoarseRow R,
                                     int E, int N, int parts) {
  const int tid = threadIdx.x;
  const int pos = R.row & 0xffff, size = R.part & 0xffff;
  const double rt = 0.70710678118654752440;
  const int ti = R.ijk & 255, tj = (R.ijk >> 8) & 255, tk = R.ijk >> 16;  // N <= the block: one node each
  if (tid < N) v[tid] = (double)f[(tk * LC::ED + tj) * LC::ED + ti];
  __syncthreads();
  double* w = v + N;
#pragma unroll 1
  for (int way = 0; way < 2; ++way) {
    // pairs along each axis become (sum, difference) / sqrt 2, the middle
    // stays; the same again undoes it
    int stride = 1;
#pragma unroll 1
    for (int d = 0; d < 3; ++d, stride *= E) {
      const int i = d == 0 ? ti : d == 1 ? tj : tk;
      if (tid < N && i < E / 2) {
        double* x = v + tid;
        const double lo = x[0], hi = x[(E - 1 - 2 * i) * stride];
        x[0] = rt * (lo + hi);
        x[(E - 1 - 2 * i) * stride] = rt * (lo - hi);
      }
      __syncthreads();
    }
    if (way) break;
    if (tid < N) w[tid] = v[pos];
    __syncthreads();
    double acc = 0.0;
    const double* ws = w + (R.row >> 16);
    const double* col = blocks + R.col;
#pragma unroll 8
    for (int j = R.part >> 16; j < size; j += parts) acc += col[j * size] * ws[j];
    __syncthreads();
    w[tid] = acc;
    __syncthreads();
    if (tid < N) {
      double s = 0.0;
      for (int t = 0; t < parts; ++t) s += w[t * N + tid];
      v[pos] = s;
    }
    __syncthreads();
  }
  constexpr int PE = LC::ED + 2;
  if (tid < N) e[((tk + 1) * PE + tj + 1) * PE + ti + 1] = (T)v[tid];
  __syncthreads();
}

// One V(nu1, nu2) cycle on a zero guess from level L (NT intervals at most)
// down.  Colours and the two ways are loops, not unrolled code.
template <typename T, int C, int NT, int L>
struct Cycle {
  typedef Lev<T, C, NT> V;
  // each(c, fn): fn(j, k, row, a, f) for the thread's nodes of colour c
  template <typename Each>
  __device__ static void run(T* lds, const TailArgs& A, const double* blocks, const CoarseRow& R, Each&& each) {
    T* u = lds + Arena<T, C, NT, L>::u;
    T* r = lds + A.r;
    const T h2 = (T)A.d[L].h2, ih2 = (T)A.d[L].ih2;
    typedef Lev<T, C, NT / 2> VC;
    const int Ec = A.d[L + 1].n - 1;
    T* fc = lds + A.f + Arena<T, C, NT / 2, L + 1>::f;
    T* uc = lds + Arena<T, C, NT / 2, L + 1>::u;
#pragma unroll 1
    for (int way = 0; way < 2; ++way) {
      const int passes = (way ? A.nu2 : A.nu1) * C;
#pragma unroll 1
      for (int q = 0; q < passes; ++q) {
        const int c = way ? C - 1 - (q & (C - 1)) : q & (C - 1);
        each(c, [&](int, int, int row, int a, T f) {
          u[c * V::CS + row + (a >> V::lc)] = V::relaxed(u + row, c, a, f, h2);
        });
        __syncthreads();
      }
      if (way) break;
#pragma unroll 1
      for (int c = 0; c < C; ++c) {
        const bool gone = c == C - 1 && A.nu1 > 0;
        each(c, [&](int j, int k, int row, int a, T f) {
          r[(k * V::ED + j) * V::ED + a - V::g] = gone ? (T)0 : V::residual(u + row, c, a, f, ih2);
        });
      }
      __syncthreads();
      for (int t = threadIdx.x; t < VC::ED * VC::ED * VC::ED; t += kTailThreads) {
        const int I = t % VC::ED, J = (t / VC::ED) % VC::ED, K = t / (VC::ED * VC::ED);
        if (I < Ec && J < Ec && K < Ec) fc[t] = full_weight<V::ED>(r, I, J, K);
      }
      __syncthreads();
      const bool last = L + 2 == A.nl;
      if (last) {
        coarse_blocks<VC>(uc, fc, reinterpret_cast<double*>(r), blocks, R, Ec, A.N, A.parts);
      } else if constexpr (NT / 2 >= kTailLow) {
        Cycle<T, C, NT / 2, L + 1>::run(lds, A, blocks, R, [&](int c, auto&& fn) {
          for (int slot = threadIdx.x; slot < VC::SLOTS; slot += kTailThreads) {
            int t, j, k;
            VC::decode(slot, t, j, k);
            const int a = VC::node(c, VC::shift(j, k), t);
            if (j < Ec && k < Ec && a < VC::g + Ec)
              fn(j, k, VC::row(j, k), a, fc[(k * VC::ED + j) * VC::ED + a - VC::g]);
          }
        });
      }
      const int corrected = A.nu2 > 0 ? C - 1 : C;  // the first pass overwrites the last colour
#pragma unroll 1
      for (int c = 0; c < corrected; ++c)
        each(c, [&](int j, int k, int row, int a, T) {
          const int i = a - V::g + 1;
          T& x = u[c * V::CS + row + (a >> V::lc)];
          if (last) {
            constexpr int PE = VC::ED + 2;
            x += interpolate<T>(i, j + 1, k + 1, [&](int I, int J, int K) { return uc[(K * PE + J) * PE + I]; });
          } else if constexpr (NT / 2 >= kTailLow) {
            x += interpolate<T>(i, j + 1, k + 1, [&](int I, int J, int K) { return VC::at(uc, I, J, K); });
          }
        });
      __syncthreads();
    }
  }
};

// The tail: right-hand side F, result X (both in the global layout G of the
// top level).  The top level's right-hand side is read once and stays in
// registers: thread t owns the nodes t, t + 1024, ... of each colour.  As in
// the launched cycle the residuals of the last colour swept vanish and are not
// formed, and the last colour is not corrected when a pass over it follows.
template <typename T, int C, int NT>
__global__ __launch_bounds__(kTailThreads) void k_tail(const T* __restrict__ F, T* __restrict__ X, Geom G,
                                                       TailArgs A, const double* __restrict__ pinv) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  typedef Lev<T, C, NT> V;
  constexpr int NR = V::NR;
  T* lds = reinterpret_cast<T*>(smem);
  const int tid = threadIdx.x, E = G.n - 1, cs = (int)G.cs;
  int at[NR], jk[NR];  // number of the node in its row, row and plane
  T fr[C][NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    int t, j, k;
    V::decode(tid + i * kTailThreads, t, j, k);
    at[i] = j < E && k < E ? t : NT;  // NT: no unknown
    jk[i] = j | k << 8;
    const int row = (int)G.row(j + V::g, k + V::g);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int a = V::node(c, V::shift(j, k), at[i]);
      fr[c][i] = a < V::g + E ? F[c * cs + row + (a >> V::lc)] : (T)0;
    }
  }
  CoarseRow R = {0, tid < A.N ? 1 : 0, 0, 0};  // a single unknown
  if (A.rows) R = tid < A.N * A.parts ? reinterpret_cast<const CoarseRow*>(pinv)[tid] : CoarseRow{0, 0, 0, 0};
  const double* blocks = pinv + A.rows;
  if (A.staged) {
    double* staged = reinterpret_cast<double*>(smem + A.staged);
    for (int i = tid; i < A.blocks; i += kTailThreads) staged[i] = blocks[i];
    blocks = staged;
  }
  for (int i = tid; i < A.clear; i += kTailThreads) lds[i] = (T)0;
  __syncthreads();
  auto each = [&](int c, auto&& fn) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      // hidden from the compiler, which would otherwise keep every address
      // derived from it in registers across the passes and spill
      int q = jk[i];
      asm volatile("" : "+v"(q));
      const int j = q & 255, k = q >> 8;
      const int a = V::node(c, V::shift(j, k), at[i]);
      T f = fr[0][i];
#pragma unroll
      for (int d = 1; d < C; ++d) {
        T x = fr[d][i];
        asm("" : "+v"(x));  // keeps the selection among registers
        f = c == d ? x : f;
      }
      if (a < V::g + E) fn(j, k, V::row(j, k), a, f);
    }
  };
  Cycle<T, C, NT, 0>::run(lds, A, blocks, R, each);
#pragma unroll 1
  for (int c = 0; c < C; ++c)
    each(c, [&](int j, int k, int row, int a, T) {
      X[c * cs + (int)G.row(j + V::g, k + V::g) + (a >> V::lc)] = lds[c * V::CS + row + (a >> V::lc)];
    });
}

// LDS of a tail sized for NT intervals with nl levels: elements of the
// potentials and of the right-hand sides below the top, and bytes in all
template <typename T, int C>
constexpr size_t tail_bytes(int NT, int nl, int& u, int& f) {
  u = f = 0;
  for (int l = 0, n = NT; l < nl; ++l, n /= 2) {
    const int M = n + 1 + (C == 2 ? 0 : 4);
    u += C * M * M * ((M + C - 1) / C);
    if (l > 0) f += (n - 1) * (n - 1) * (n - 1);
  }
  const size_t e = NT - 1, r = e * e * e * sizeof(T), v = 2 * kTailThreads * sizeof(double);
  return ((u + f + 3) & ~3) * sizeof(T) + (r > v ? r : v);
}
template <typename T, int C, int NT>
constexpr bool tail_possible() {
  int u = 0, f = 0;
  return tail_bytes<T, C>(NT, 2, u, f) <= kTailLds;
}

// fn(integral_constant NT) for the smallest tail size that holds n intervals;
// false if none does
template <typename T, int C, typename Fn>
bool tail_size(int n, Fn&& fn) {
  if (n <= 12) return fn(std::integral_constant<int, 12>());
  if (n <= 16) return fn(std::integral_constant<int, 16>());
  if constexpr (tail_possible<T, C, 20>()) {
    if (n <= 20) return fn(std::integral_constant<int, 20>());
  }
  if constexpr (tail_possible<T, C, 24>()) {
    if (n <= 24) return fn(std::integral_constant<int, 24>());
  }
  return false;
}

template <typename T, int C>
void tail_go(const void* f, void* x, const Geom& G, const TailArgs& A, const double* pinv, hipStream_t st) {
  tail_size<T, C>(G.n, [&](auto nt) {
    k_tail<T, C, nt><<<1, kTailThreads, A.lds, st>>>((const T*)f, (T*)x, G, A, pinv);
    return true;
  });
}

template <typename T, int C>
bool tail_fit(const Geom* lev, int nl, TailArgs& A) {
  return tail_size<T, C>(lev[0].n, [&](auto nt) {
    // levels down to the coarsest must lie above the lowest the kernel has
    if ((nt >> (nl - 2)) < kTailLow) return false;
    int u, f;
    A.lds = tail_bytes<T, C>(nt, nl, u, f);
    A.clear = u;
    A.f = u;
    A.r = (u + f + 3) & ~3;
    const size_t at = (A.lds + 15) & ~(size_t)15, with = at + A.blocks * sizeof(double);
    A.staged = with <= kTailLds ? (int)at : 0;
    if (A.staged) A.lds = with;
    return A.lds <= kTailLds;
  });
}

template <typename T, int C>
bool tail_lds(int n) {
  return tail_size<T, C>(n, [&](auto nt) {
    return hipFuncSetAttribute((const void*)k_tail<T, C, nt>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kTailLds) == hipSuccess;
  });
}

}  // namespace

// entries of the four unlike blocks (sectors 0, 1, 3 and 7)
static size_t block_entries(int E) {
  size_t n = 0;
  for (int s : {0, 1, 3, 7}) n += (size_t)sector_size(E, s) * sector_size(E, s);
  return n;
}

bool tail_args(const Geom* lev, int nl, bool f32, int nu1, int nu2, TailArgs& A) {
  if (nl < 2 || nl > kTailLevels) return false;
  const int Ec = lev[nl - 1].n - 1;
  if (Ec * Ec * Ec > kTailCoarseMax) return false;
  A = TailArgs{};
  A.nl = nl;
  A.nu1 = nu1;
  A.nu2 = nu2;
  A.N = Ec * Ec * Ec;
  A.parts = coarse_parts(Ec);
  A.rows = (int)row_table(Ec);
  A.blocks = (int)block_entries(Ec);
  for (int l = 0; l < nl; ++l) {
    A.d[l].n = lev[l].n;
    A.d[l].h2 = lev[l].h * lev[l].h;
    A.d[l].ih2 = 1.0 / (lev[l].h * lev[l].h);
  }
  if (lev[0].C == 2) return f32 ? tail_fit<float, 2>(lev, nl, A) : tail_fit<double, 2>(lev, nl, A);
  return f32 ? tail_fit<float, 4>(lev, nl, A) : tail_fit<double, 4>(lev, nl, A);
}

bool tail_enable(bool f32, int C, int n) {
  if (C == 2) return f32 ? tail_lds<float, 2>(n) : tail_lds<double, 2>(n);
  return f32 ? tail_lds<float, 4>(n) : tail_lds<double, 4>(n);
}

size_t tail_blocks_size(int E) { return row_table(E) + block_entries(E); }

void tail_blocks(int E, const std::vector<double>& inv, std::vector<double>& out) {
  const int N = E * E * E, H = E / 2;
  const double rt = sqrt(0.5);
  std::vector<double> B(inv);
  // B <- T inv T^t, T the pairwise sums and differences along every axis
  auto fold = [&](double* x, size_t stride) {
    auto axis = [&](size_t st, size_t s1, size_t s2) {
      for (int q = 0; q < E; ++q)
        for (int p = 0; p < E; ++p)
          for (int i = 0; i < H; ++i) {
            double* y = x + (q * s2 + p * s1) * stride;
            double &a = y[i * st * stride], &b = y[(E - 1 - i) * st * stride];
            const double u = a, v = b;
            a = rt * (u + v);
            b = rt * (u - v);
          }
    };
    axis(1, E, (size_t)E * E);
    axis(E, 1, (size_t)E * E);
    axis((size_t)E * E, 1, E);
  };
  for (int i = 0; i < N; ++i) fold(&B[(size_t)i * N], 1);
  for (int i = 0; i < N; ++i) fold(&B[i], N);
  std::vector<CoarseRow> rows;
  std::vector<double> entries;
  int first[4];  // of the block for 0, 1, 2 and 3 odd axes
  for (int s = 0; s < 8; ++s) {
    // unknowns of the sector, the odd axes fastest, so that sectors with
    // equally many odd axes have the same block
    int axis[3], dim[3], n = 0;
    for (int odd = 1; odd >= 0; --odd)
      for (int d = 0; d < 3; ++d)
        if (((s >> d) & 1) == odd) {
          dim[n] = odd ? H : E - H;
          axis[n++] = d;
        }
    std::vector<int> id;
    for (int z = 0; z < dim[2]; ++z)
      for (int y = 0; y < dim[1]; ++y)
        for (int x = 0; x < dim[0]; ++x) {
          const int c[3] = {x, y, z};
          int p[3];
          for (int d = 0; d < 3; ++d) p[axis[d]] = (s >> axis[d]) & 1 ? E - 1 - c[d] : c[d];
          id.push_back((p[2] * E + p[1]) * E + p[0]);
        }
    const int base = (int)rows.size(), size = (int)id.size();
    if (s == 0 || s == 1 || s == 3 || s == 7) {
      first[sector_odd(s)] = (int)entries.size();
      // symmetric: entry (j, q) stands at j size + q
      for (int p : id)
        for (int q : id) entries.push_back(0.5 * (B[(size_t)p * N + q] + B[(size_t)q * N + p]));
    }
    for (int q = 0; q < size; ++q)
      rows.push_back(CoarseRow{id[q] | base << 16, size, first[sector_odd(s)] + q, 0});
  }
  for (int q = 0; q < N; ++q) rows[q].ijk = q % E | (q / E % E) << 8 | (q / (E * E)) << 16;
  for (int t = N; t < N * coarse_parts(E); ++t) {
    CoarseRow r = rows[t % N];
    r.part |= t / N << 16;
    rows.push_back(r);
  }
  out.assign(tail_blocks_size(E), 0.0);
  memcpy(out.data(), rows.data(), row_table(E) * sizeof(double));
  std::copy(entries.begin(), entries.end(), out.begin() + row_table(E));
}

void tail_cycle(const void* f, void* x, bool f32, const Geom& G, const TailArgs& A, const double* pinv,
                hipStream_t st) {
  if (G.C == 2) {
    if (f32)
      tail_go<float, 2>(f, x, G, A, pinv, st);
    else
      tail_go<double, 2>(f, x, G, A, pinv, st);
  } else {
    if (f32)
      tail_go<float, 4>(f, x, G, A, pinv, st);
    else
      tail_go<double, 4>(f, x, G, A, pinv, st);
  }
}

}  // namespace psn
