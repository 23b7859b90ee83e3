// Spherical Poisson operator (Eq. 2 multiplied by r^2) and the fused
// BiCGSTAB kernels (Section 2.1.2: BiCGSTAB for the non-symmetric direct
// finite-difference spherical Laplacian) for gfx950, FP64.
//   r^2 lap u = a u_xixi + b u_xi + u_tt + cot(t) u_t + u_pp / sin^2(t)
// on the radial map coordinate xi (a = 1/ds^2, b = 1/ds on the log grid,
// i.e. u_ss + u_s), with 2nd-order central differences: the radial couplings
// cl = a - b/2, cr = a + b/2 come per radial index from tables; radial ghosts hold Dirichlet values,
// the colatitude neighbour past a pole is the node at phi + pi, phi is
// periodic.  Direction vectors keep zero radial ghosts.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "reduce.h"

namespace psn {

namespace {

constexpr int BX = 64, BY = 4;

struct Coef {
  double idt2, idp2;
  const double* rcl;  // radial couplings per radial index
  const double* rcr;
};

inline dim3 sgrid(const SGeom& S) { return dim3((S.nr + BX - 1) / BX, (S.nth + BY - 1) / BY, S.nph); }

// value of the operator at unknown (i, j, k) for a vector given by functor V
template <typename F>
__device__ inline double sph_op(const F& V, const SGeom& S, const Coef& c, const double* __restrict__ cot2,
                                const double* __restrict__ isin2, int i, int j, int k) {
  const int half = S.nph >> 1;
  const double u = V(i, j, k);
  const double ip = V(i + 1, j, k), im = V(i - 1, j, k);
  const double jp = (j + 1 < S.nth) ? V(i, j + 1, k) : V(i, S.nth - 1, (k + half) % S.nph);
  const double jm = (j > 0) ? V(i, j - 1, k) : V(i, 0, (k + half) % S.nph);
  const double kp = V(i, j, (k + 1) % S.nph), km = V(i, j, (k + S.nph - 1) % S.nph);
  return c.rcr[i] * ip + c.rcl[i] * im - (c.rcl[i] + c.rcr[i]) * u + (jp - 2.0 * u + jm) * c.idt2 +
         cot2[j] * (jp - jm) + (kp - 2.0 * u + km) * isin2[j] * c.idp2;
}

// Grid of the kernels that reduce: a block takes up to 8 consecutive planes, so
// that large grids leave a few thousand partial sums to add up (at 256 x 128 x
// 256 32768 of them took 11.7 us each time) and a plane's values serve as the
// next one's neighbour.
inline dim3 rgrid(const SGeom& S) {
  dim3 g = sgrid(S);
  const int kz = std::min(8, std::max(1, (int)((long long)g.x * g.y * g.z / 2048)));
  g.z = (S.nph + kz - 1) / kz;
  return g;
}

// The thread's column and planes.  Without RUNS (a plane per block) the grid is
// taken as it is: on small grids the divisions of the XCD order and of the run
// are 0.8 us of a residual's 8 (64 x 32 x 80).
template <bool RUNS>
__device__ inline void column(const SGeom& S, int& i, int& j, int& k0, int& k1) {
  int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  if constexpr (RUNS) xcd_block(bx, by, bz);
  i = 1 + bx * BX + threadIdx.x;
  j = by * BY + threadIdx.y;
  const int kz = RUNS ? (S.nph + gridDim.z - 1) / gridDim.z : 1;
  k0 = bz * kz;
  k1 = RUNS ? min(k0 + kz, S.nph) : k0 + 1;
}

// Calls out(k, A u) for the planes k0 .. k1-1 of column (i, j): along phi a
// plane's value is the next one's neighbour.
template <class F, class O>
__device__ inline void sph_op_column(const F& V, const SGeom& S, const Coef& c, const double* __restrict__ cot2,
                                     const double* __restrict__ isin2, int i, int j, int k0, int k1, const O& out) {
  const double rr = c.rcr[i], rl = c.rcl[i], ct = cot2[j], is2 = isin2[j];
  const int half = S.nph >> 1;
  double km = V(i, j, k0 ? k0 - 1 : S.nph - 1), u = V(i, j, k0);
  for (int k = k0; k < k1; ++k) {
    const double kp = V(i, j, k + 1 == S.nph ? 0 : k + 1);
    const double ip = V(i + 1, j, k), im = V(i - 1, j, k);
    const int ka = k + half >= S.nph ? k + half - S.nph : k + half;
    const double jp = (j + 1 < S.nth) ? V(i, j + 1, k) : V(i, S.nth - 1, ka);
    const double jm = (j > 0) ? V(i, j - 1, k) : V(i, 0, ka);
    out(k, rr * ip + rl * im - (rl + rr) * u + (jp - 2.0 * u + jm) * c.idt2 + ct * (jp - jm) +
               (kp - 2.0 * u + km) * is2 * c.idp2);
    km = u;
    u = kp;
  }
}

// one thread per pair of radial indices (the kernels that visit one colour)
inline dim3 black_grid(const SGeom& S) {
  return dim3((S.nr + 2 * BX - 1) / (2 * BX), (S.nth + BY - 1) / BY, S.nph);
}

__device__ inline bool active(const SGeom& S, int i, int j, int k) {
  return i >= 1 && i <= S.nr && j < S.nth && k < S.nph;
}

template <bool RUNS, bool ZU>
__global__ __launch_bounds__(256) void k_sph_residual(const double* __restrict__ U, const double* __restrict__ rho,
                                                      double* __restrict__ R, SGeom S, Coef c,
                                                      const double* __restrict__ cot2,
                                                      const double* __restrict__ isin2,
                                                      const double* __restrict__ r2, double fpg,
                                                      double* __restrict__ partial) {
  int i, j, k0, k1;
  column<RUNS>(S, i, j, k0, k1);
  double acc = 0.0;
  if (i <= S.nr && j < S.nth) {
    auto V = [&](int ii, int jj, int kk) -> double {
      if (ZU && ii >= 1 && ii <= S.nr) return 0.0;
      return U[S.at(ii, jj, kk)];
    };
    sph_op_column(V, S, c, cot2, isin2, i, j, k0, k1, [&](int k, double o) {
      const long long idx = S.at(i, j, k);
      const double res = fpg * r2[i] * rho[idx] - o;
      if (R) R[idx] = res;
      acc += res * res;
    });
  }
  if (partial) {
    const double s = block_sum(acc);
    if (threadIdx.x == 0 && threadIdx.y == 0) partial[linear_block()] = s;
  }
}

__global__ __launch_bounds__(256) void k_sph_apply(const double* __restrict__ U, double* __restrict__ out, SGeom S,
                                                   Coef c, const double* __restrict__ cot2,
                                                   const double* __restrict__ isin2) {
  const int i = 1 + blockIdx.x * BX + threadIdx.x;
  const int j = blockIdx.y * BY + threadIdx.y;
  const int k = blockIdx.z;
  if (!active(S, i, j, k)) return;
  auto V = [&](int ii, int jj, int kk) -> double { return U[S.at(ii, jj, kk)]; };
  out[S.at(i, j, k)] = sph_op(V, S, c, cot2, isin2, i, j, k);
}

// One colour of SOR (Section 2.1.1) on the log-spherical grid.  Colour =
// parity of (i + j + k) plus 2 for phi in the second half turn, so no two
// neighbours -- across a pole included -- share a colour; the grid covers the
// colour's half turn only.  u += omega_j (u_GS - u), u_GS solving the node's
// own row: u_GS - u = residual / diagonal.
__global__ __launch_bounds__(256) void k_sph_sor(double* __restrict__ U, const double* __restrict__ rho, SGeom S,
                                                 Coef c, const double* __restrict__ cot2,
                                                 const double* __restrict__ isin2, const double* __restrict__ r2,
                                                 double fpg, const double* __restrict__ omega, int colour,
                                                 const double* __restrict__ rj, double* __restrict__ omega_out) {
  // thread t of the row takes the node of the pass's parity among radial
  // indices 1 + 2t and 2 + 2t, so every lane has work
  const int j = blockIdx.y * BY + threadIdx.y;
  const int k = blockIdx.z + ((colour >> 1) ? (S.nph >> 1) : 0);
  const int i0 = 1 + 2 * (int)(blockIdx.x * BX + threadIdx.x);
  const int i = i0 + ((colour + i0 + j + k) & 1);
  if (!active(S, i, j, k)) return;
  auto V = [&](int ii, int jj, int kk) -> double { return U[S.at(ii, jj, kk)]; };
  const long long idx = S.at(i, j, k);
  const double res = fpg * r2[i] * rho[idx] - sph_op(V, S, c, cot2, isin2, i, j, k);
  const double d = -(c.rcl[i] + c.rcr[i]) - 2.0 * c.idt2 - 2.0 * isin2[j] * c.idp2;
  const long long t = (long long)j * (S.nr + 2) + i;
  const double w = omega[t];
  U[idx] += w * res / d;
  // next term of the sequence (Eq. omega_n), written by the one thread of
  // (i, j) that is active in the first two planes of the half turn
  if (omega_out && (int)blockIdx.z == ((colour + i + j + (S.nph >> 1)) & 1))
    omega_out[t] = 1.0 / (1.0 - rj[t] * rj[t] * w / 4.0);
}

// next term of the relaxation sequence at every node of the table (Eq. omega_n)
__global__ void k_sph_omega(double* __restrict__ omega, const double* __restrict__ rj, int n) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) omega[e] = 1.0 / (1.0 - rj[e] * rj[e] * omega[e] / 4.0);
}

// Right-preconditioned BiCGSTAB (Section 2.1.2: a multi-colour Gauss-Seidel
// preconditioner B, the block lower triangle of A in red-black order, applied
// by block substitution).  Red nodes (i + j + k even) solve with their
// diagonal, black nodes subtract their red neighbours' values first;
// couplings between nodes of one colour (only across a pole, when nphi/2 is
// even) are left out of B.  scal->v: 0 rho, 1 alpha, 2 omega, 3 beta,
// 4 rhat.v, 5 t.s, 6 t.t, 7 r.r.

__device__ inline double sph_diag(const Coef& c, const double* __restrict__ isin2, int i, int j) {
  return -(c.rcl[i] + c.rcr[i]) - 2.0 * c.idt2 - 2.0 * isin2[j] * c.idp2;
}

__device__ inline bool is_red(int i, int j, int k) { return ((i + j + k) & 1) == 0; }

// p = r + beta (p - omega v)   (in place);   phat = p / D on red nodes; L.f: p in
// FP32 as the multigrid preconditioner's right-hand side
__global__ __launch_bounds__(256) void k_pbicg_p(const double* __restrict__ R, double* __restrict__ P,
                                                 const double* __restrict__ Vv, double* __restrict__ Ph, SGeom S,
                                                 Coef c, const double* __restrict__ isin2,
                                                 const Scalars* __restrict__ scal, SLev L) {
  const int i = 1 + blockIdx.x * BX + threadIdx.x;
  const int j = blockIdx.y * BY + threadIdx.y;
  const int k = blockIdx.z;
  if (!active(S, i, j, k)) return;
  const double beta = scal->v[3], omega = scal->v[2];
  const long long idx = S.at(i, j, k);
  const double pv = R[idx] + beta * (P[idx] - omega * Vv[idx]);
  P[idx] = pv;
  if (L.f) L.f[L.at(i, j, k)] = (float)pv;
  if (Ph && is_red(i, j, k)) Ph[idx] = pv / sph_diag(c, isin2, i, j);
}

// s = r - alpha v;   shat = s / D on red nodes
__global__ __launch_bounds__(256) void k_pbicg_s(const double* __restrict__ R, const double* __restrict__ Vv,
                                                 double* __restrict__ Sv, double* __restrict__ Sh, SGeom S, Coef c,
                                                 const double* __restrict__ isin2,
                                                 const Scalars* __restrict__ scal, SLev L) {
  const int i = 1 + blockIdx.x * BX + threadIdx.x;
  const int j = blockIdx.y * BY + threadIdx.y;
  const int k = blockIdx.z;
  if (!active(S, i, j, k)) return;
  const long long idx = S.at(i, j, k);
  const double sv = R[idx] - scal->v[1] * Vv[idx];
  Sv[idx] = sv;
  if (L.f) L.f[L.at(i, j, k)] = (float)sv;
  if (Sh && is_red(i, j, k)) Sh[idx] = sv / sph_diag(c, isin2, i, j);
}

// black nodes of xhat = B^-1 y: (y - sum over red neighbours of a_n xhat_n) / D
__global__ __launch_bounds__(256) void k_gs_black(const double* __restrict__ Y, double* __restrict__ Xh, SGeom S,
                                                  Coef c, const double* __restrict__ cot2,
                                                  const double* __restrict__ isin2) {
  // thread t of the row takes the black node among radial indices 1 + 2t
  // and 2 + 2t
  const int j = blockIdx.y * BY + threadIdx.y;
  const int k = blockIdx.z;
  const int i0 = 1 + 2 * (int)(blockIdx.x * BX + threadIdx.x);
  const int i = i0 + ((1 + i0 + j + k) & 1);
  if (!active(S, i, j, k)) return;
  const int half = S.nph >> 1;
  // value of a neighbour if it is red, else 0 (radial ghosts of xhat are 0)
  auto red = [&](int ii, int jj, int kk) -> double { return is_red(ii, jj, kk) ? Xh[S.at(ii, jj, kk)] : 0.0; };
  double s = c.rcr[i] * red(i + 1, j, k) + c.rcl[i] * red(i - 1, j, k);
  const double cjp = c.idt2 + cot2[j], cjm = c.idt2 - cot2[j];
  s += cjp * ((j + 1 < S.nth) ? red(i, j + 1, k) : red(i, S.nth - 1, (k + half) % S.nph));
  s += cjm * ((j > 0) ? red(i, j - 1, k) : red(i, 0, (k + half) % S.nph));
  const double cp = isin2[j] * c.idp2;
  s += cp * (red(i, j, (k + 1) % S.nph) + red(i, j, (k + S.nph - 1) % S.nph));
  const long long idx = S.at(i, j, k);
  Xh[idx] = (Y[idx] - s) / sph_diag(c, isin2, i, j);
}

// xhat of the multi-colour preconditioner (FP64, the grid's layout) or of the
// multigrid one (its FP32 finest level, read in place)
struct HatD {
  const double* x;
  SGeom S;
  __device__ double operator()(int i, int j, int k) const { return x[S.at(i, j, k)]; }
};
struct HatF {
  SLev L;
  __device__ double operator()(int i, int j, int k) const { return (double)L.u[L.at(i, j, k)]; }
};

// out = A xhat with dots: mode 0: partial0 += a.out (a = rhat);
// mode 1: partial0 += out.a, partial1 += out.out (a = s).  HBM-bound (20 bytes
// per unknown with an FP32 xhat, 24 with an FP64 one).  256 x 128 x 256: 59 and
// 56 us with the FP32 level (modes 0 and 1), 59 and 37 with an FP64 array,
// whose xhat and a the kernels before have just written; 70-73 before the runs
// of planes and the XCD order.
template <bool RUNS, int MODE, class H>
__global__ __launch_bounds__(256) void k_apply_dot(H Xh, double* __restrict__ Out, const double* __restrict__ Aw,
                                                   SGeom S, Coef c, const double* __restrict__ cot2,
                                                   const double* __restrict__ isin2, double* __restrict__ partial) {
  int i, j, k0, k1;
  column<RUNS>(S, i, j, k0, k1);
  double a0 = 0.0, a1 = 0.0;
  if (i <= S.nr && j < S.nth)
    sph_op_column(Xh, S, c, cot2, isin2, i, j, k0, k1, [&](int k, double o) {
      const long long idx = S.at(i, j, k);
      Out[idx] = o;
      a0 += Aw[idx] * o;
      if (MODE == 1) a1 += o * o;
    });
  const double s0 = block_sum(a0);
  if (threadIdx.x == 0 && threadIdx.y == 0) partial[linear_block()] = s0;
  if (MODE == 1) {
    const double s1 = block_sum(a1);
    if (threadIdx.x == 0 && threadIdx.y == 0) partial[kPartialCap + linear_block()] = s1;
  }
}

// x += alpha phat + omega shat;  r = s - omega t;  partial0 += rhat.r, partial1 += r.r
// (HBM-bound: 56 bytes per unknown with FP32 phat, shat; 256 x 128 x 256 88 us,
// 107 with FP64 copies)
template <bool RUNS, class H>
__global__ __launch_bounds__(256) void k_pbicg_xr(double* __restrict__ X, double* __restrict__ R, H Ph, H Sh,
                                                  const double* __restrict__ Sv, const double* __restrict__ T,
                                                  const double* __restrict__ Rhat, SGeom S,
                                                  const Scalars* __restrict__ scal, double* __restrict__ partial) {
  int i, j, k0, k1;
  column<RUNS>(S, i, j, k0, k1);
  const double alpha = scal->v[1], omega = scal->v[2];
  double a0 = 0.0, a1 = 0.0;
  if (i <= S.nr && j < S.nth)
#pragma unroll 2
    for (int k = k0; k < k1; ++k) {
      const long long idx = S.at(i, j, k);
      X[idx] += alpha * Ph(i, j, k) + omega * Sh(i, j, k);
      const double rn = Sv[idx] - omega * T[idx];
      R[idx] = rn;
      a0 += Rhat[idx] * rn;
      a1 += rn * rn;
    }
  const double s0 = block_sum(a0);
  if (threadIdx.x == 0 && threadIdx.y == 0) partial[linear_block()] = s0;
  const double s1 = block_sum(a1);
  if (threadIdx.x == 0 && threadIdx.y == 0) partial[kPartialCap + linear_block()] = s1;
}

// stage 0: alpha = rho / (rhat.v); stage 1: omega = (t.s)/(t.t);
// stage 2: beta = (rho_new/rho)(alpha/omega), rho = rho_new, v[7] = r.r
__global__ __launch_bounds__(kFinishThreads) void k_bicg_scalars(const double* __restrict__ partial, int nb,
                                                                 Scalars* __restrict__ scal, int stage, Post post) {
  const double s0 = sum_partials(partial, nb);
  __syncthreads();
  const double s1 = stage > 0 ? sum_partials(partial + kPartialCap, nb) : 0.0;
  if (threadIdx.x == 0) {
    double* v = scal->v;
    if (stage == 0) {
      v[4] = s0;
      v[1] = (s0 != 0.0) ? v[0] / s0 : 0.0;
    } else if (stage == 1) {
      v[5] = s0;
      v[6] = s1;
      v[2] = (s1 != 0.0) ? s0 / s1 : 0.0;
    } else {
      v[3] = (v[0] != 0.0 && v[2] != 0.0) ? (s0 / v[0]) * (v[1] / v[2]) : 0.0;
      v[0] = s0;
      v[7] = s1;
    }
    post_scalars(scal, post);
  }
}

__global__ __launch_bounds__(256) void k_sph_fill(double* __restrict__ x, SGeom S) {
  const int i = blockIdx.x * BX + threadIdx.x;
  const int j = blockIdx.y * BY + threadIdx.y;
  const int k = blockIdx.z;
  if (i >= S.p0 || j >= S.nth) return;
  x[S.at(i, j, k)] = 0.0;
}

__global__ __launch_bounds__(256) void k_sph_copy(const double* __restrict__ a, double* __restrict__ b, SGeom S) {
  const int i = blockIdx.x * BX + threadIdx.x;
  const int j = blockIdx.y * BY + threadIdx.y;
  const int k = blockIdx.z;
  if (i >= S.nr + 2 || j >= S.nth) return;
  b[S.at(i, j, k)] = a[S.at(i, j, k)];
}

// ---------------------------------------------------------------- FP32 multigrid preconditioner
// One zebra colour of phi-line Gauss-Seidel.  Block (x, j) takes nl lines
// i = 2 (x nl + line) + ((j + colour) & 1) at colatitude j; thread
// (line, segment) eliminates its segment of seg nodes with the tabulated
// factors (y = T^-1 d, T the segment's tridiagonal block), the segment ends
// meet in the interface system X = G E (X: line values at segment ends,
// E: the y values there), and each segment then adds the end loads:
// x = y - a (x_left v + x_right w).  Y lives in LDS as [seg][thread].
__global__ __launch_bounds__(1024) void k_sline(SLev L, int colour, int zero_guess) {
  extern __shared__ float lds[];
  const int nt = blockDim.x;
  const int t = threadIdx.x;
  const int line = t % L.nl, sgi = t / L.nl;
  const int j = blockIdx.y;
  const int i = 2 * (blockIdx.x * L.nl + line) + ((j + colour) & 1);
  const int SL = L.seg, P = L.nseg;
  float* Y = lds;
  float* E = lds + (size_t)SL * nt;
  const int it = min(i, L.ntab - 1);
  const float* tb = L.ltab + ((size_t)it * L.nth + j) * L.tstride;
  const float* m = tb;
  const float* cp = tb + SL;
  const float* v = tb + 2 * SL;
  const float* w = tb + 3 * SL;
  const float* G = tb + 4 * SL;
  const bool act = i < L.nr;
  const float aphi = L.isin2[j] * L.idp2;
  const int k0 = sgi * SL;
  if (act) {
    const int a = i + 1, half = L.nph >> 1;
    const float cr = L.rcr[i], cl = L.rcl[i];
    const float cjp = L.idt2 + L.cot2[j], cjm = L.idt2 - L.cot2[j];
    float d = 0.0f;
#pragma unroll 8
    for (int q = 0; q < SL; ++q) {
      const int k = k0 + q;
      const long long idx = L.at(a, j, k);
      // zero_guess 1: u is zero everywhere; 2: this colour's lines are still
      // zero (the cross-pole term, which reads the line itself, is zero)
      float rhs = L.f[idx];
      if (zero_guess != 1) {
        const float pole = (zero_guess == 2) ? 0.0f : L.u[L.at(a, j, (k + half) % L.nph)];
        const float up = (j + 1 < L.nth) ? L.u[idx + L.p0] : pole;
        const float um = (j > 0) ? L.u[idx - L.p0] : pole;
        rhs -= cr * L.u[L.at(a + 1, j, k)] + cl * L.u[L.at(a - 1, j, k)] + cjp * up + cjm * um;
      }
      d = (rhs - aphi * d) * m[q];
      Y[(size_t)q * nt + t] = d;
    }
    float y = d;
    for (int q = SL - 2; q >= 0; --q) {
      y = Y[(size_t)q * nt + t] - cp[q] * y;
      Y[(size_t)q * nt + t] = y;
    }
    E[(size_t)(2 * sgi) * L.nl + line] = y;
    E[(size_t)(2 * sgi + 1) * L.nl + line] = d;
  }
  __syncthreads();
  if (!act) return;
  const int rl = 2 * ((sgi + P - 1) % P) + 1, rr = 2 * ((sgi + 1) % P);
  float xl = 0.0f, xr = 0.0f;
  for (int q = 0; q < 2 * P; ++q) {
    const float e = E[(size_t)q * L.nl + line];
    xl += G[rl * 2 * P + q] * e;
    xr += G[rr * 2 * P + q] * e;
  }
  xl *= aphi;
  xr *= aphi;
  const int a = i + 1;
  for (int q = 0; q < SL; ++q)
    L.u[L.at(a, j, k0 + q)] = Y[(size_t)q * nt + t] - (xl * v[q] + xr * w[q]);
}

// The same pass with the split fixed at compile time (SL nodes per segment, P
// segments).  It is bound by latency: one round of workgroups fills the chip,
// so a pass takes as long as one thread's chain.  The segment therefore stays
// in registers (with a runtime split Y went through LDS three times), the 5 SL
// loads are all underway before the recurrences begin, and the interface
// system is read from LDS.  The blocks of neighbouring colatitudes share an
// XCD's L2, since each reads the other's lines.  TAB1: one table per
// colatitude (log grid), read through the scalar cache.
// Per pass, against the runtime split: 256 x 128 x 256 16.7 us (31.3; 23.8
// without the XCD order), 128 x 64 x 128 7.1 (15.5), 64 x 32 x 64 5.0 (9.7),
// 32 x 16 x 32 4.5 (7.5), 16 x 8 x 16 4.1 (6.3).
template <int SL, int P, bool TAB1>
__global__ __launch_bounds__(1024) void k_sline_t(SLev L, int nls, int colour, int zero_guess) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  constexpr int N2 = 2 * P;
  const int nl = 1 << nls, t = threadIdx.x;
  const int line = t & (nl - 1), sgi = t >> nls;
  int bx, j, bz;
  xcd_block(bx, j, bz);
  const int par = (j + colour) & 1;
  if (par >= L.nr) return;
  const int i = 2 * (bx * nl + line) + par;
  float* Gs = lds;              // interface inverse (TAB1)
  float* E = lds + (TAB1 ? N2 * N2 : 0);
  const float* tb = L.ltab + ((size_t)(TAB1 ? 0 : min(i, L.ntab - 1)) * L.nth + j) * L.tstride;
  const float* G = tb + 4 * SL;
  if constexpr (TAB1)
    for (int q = t; q < N2 * N2; q += nl * P) Gs[q] = G[q];
  const bool act = i < L.nr;
  const float aphi = L.isin2[j] * L.idp2;
  const int half = L.nph >> 1, k0 = sgi * SL, p1 = (int)L.p1;
  const int a = min(i, L.nr - 1 - ((L.nr - 1 - par) & 1)) + 1;  // idle lanes load an own-colour line
  // a is odd for even i: its radial neighbours lie in the other half of the row
  const int right = par ? L.hp : 1 - L.hp, left = par ? L.hp - 1 : -L.hp;
  const int o = (int)L.at(a, j, k0);
  float y[SL];
#pragma unroll
  for (int q = 0; q < SL; ++q) y[q] = L.f[o + q * p1];
  if (zero_guess != 1) {
    const float cr = L.rcr[a - 1], cl = L.rcl[a - 1];
    const float cjp = L.idt2 + L.cot2[j], cjm = L.idt2 - L.cot2[j];
    float ur[SL], ul[SL], up[SL], um[SL];
#pragma unroll
    for (int q = 0; q < SL; ++q) {
      const float* u = L.u + o + q * p1;
      ur[q] = u[right];
      ul[q] = u[left];
      // across a pole: the line itself half a turn away (still zero in the
      // first sweep of a cycle)
      const bool top = j + 1 == L.nth, bottom = j == 0;
      float pole = 0.0f;
      if ((top || bottom) && zero_guess != 2) {
        const int k = k0 + q + half;
        pole = L.u[o + ((k >= L.nph ? k - L.nph : k) - k0) * p1];
      }
      up[q] = top ? pole : u[L.p0];
      um[q] = bottom ? pole : u[-L.p0];
    }
#pragma unroll
    for (int q = 0; q < SL; ++q) y[q] -= cr * ur[q] + cl * ul[q] + cjp * up[q] + cjm * um[q];
  }
  float d = 0.0f;
#pragma unroll
  for (int q = 0; q < SL; ++q) {
    d = (y[q] - aphi * d) * tb[q];
    y[q] = d;
  }
#pragma unroll
  for (int q = SL - 2; q >= 0; --q) y[q] -= tb[SL + q] * y[q + 1];
  E[(2 * sgi) * nl + line] = y[0];
  E[(2 * sgi + 1) * nl + line] = y[SL - 1];
  __syncthreads();
  if (!act) return;
  const int rl = 2 * (sgi == 0 ? P - 1 : sgi - 1) + 1, rr = 2 * (sgi == P - 1 ? 0 : sgi + 1);
  const float* gl = (TAB1 ? Gs : G) + rl * N2;
  const float* gr = (TAB1 ? Gs : G) + rr * N2;
  float xl = 0.0f, xr = 0.0f;
#pragma unroll
  for (int q = 0; q < N2; ++q) {
    const float e = E[q * nl + line];
    xl += gl[q] * e;
    xr += gr[q] * e;
  }
  xl *= aphi;
  xr *= aphi;
#pragma unroll
  for (int q = 0; q < SL; ++q) L.u[o + q * p1] = y[q] - (xl * tb[2 * SL + q] + xr * tb[3 * SL + q]);
}

template <int SL, int P>
void sline_go(const SLev& L, int colour, int zero_guess, hipStream_t st) {
  const int lines = (L.nr + 1) / 2;
  // lines per block: the most that leave a block for every CU, down to 16 (64-
  // byte rows): 128 x 64 x 128 takes 7.1 us with 16 lines, 7.8 with 64; at 256 x
  // 128 x 256 16.7 with 32, 19.1 with 16
  int nls = 6;
  while (nls > 4 && ((P << nls) > 512 || (long long)(((lines - 1) >> nls) + 1) * L.nth < 256)) --nls;
  const int nl = 1 << nls;
  const dim3 grid((lines + nl - 1) >> nls, L.nth);
  const size_t lds = sizeof(float) * ((size_t)2 * P * nl + (L.ntab == 1 ? 4 * P * P : 0));
  if (L.ntab == 1)
    k_sline_t<SL, P, true><<<grid, nl * P, lds, st>>>(L, nls, colour, zero_guess);
  else
    k_sline_t<SL, P, false><<<grid, nl * P, lds, st>>>(L, nls, colour, zero_guess);
}

// The splits that line_split makes of the sizes 2^m and 3 2^m up to 256: 64 x 32
// x 64 takes 5.0 us here, 9.7 with the runtime split, which takes every other
// size (nph = 80, 112, 144, 160, 208, 224 and those above 256).
bool sline_fixed(const SLev& L, int colour, int zero_guess, hipStream_t st) {
  if (L.count() >= (1ll << 31)) return false;
  if (L.nseg == 8 && L.seg == 2) {
    sline_go<2, 8>(L, colour, zero_guess, st);
    return true;
  }
  if (L.nseg != 16) return false;
  switch (L.seg) {
    case 2: sline_go<2, 16>(L, colour, zero_guess, st); return true;
    case 3: sline_go<3, 16>(L, colour, zero_guess, st); return true;
    case 4: sline_go<4, 16>(L, colour, zero_guess, st); return true;
    case 6: sline_go<6, 16>(L, colour, zero_guess, st); return true;
    case 8: sline_go<8, 16>(L, colour, zero_guess, st); return true;
    case 12: sline_go<12, 16>(L, colour, zero_guess, st); return true;
    case 16: sline_go<16, 16>(L, colour, zero_guess, st); return true;
    default: return false;
  }
}

// coarse f = mean of the 8 fine residuals f - A u it pairs, without storing
// them.  Coarse unknown I pairs the fine radial indices a = 2I+1 and 2I+2:
// entry I of a row's odd half and I+1 of its even half, so a wavefront's loads
// are contiguous and the radial neighbours are the next entries.  Bound by the
// L2 (u comes twice: the planes k-1 and k+2 of a pair, the rows around a
// block); blocks of neighbouring planes share an XCD.  256 x 128 x 256 with
// the residual stored 38.3 + 14.4 us, here 13.2; 64 x 32 x 64 4.7 + 4.9, here 5.1.
__global__ __launch_bounds__(256) void k_sresrestrict(SLev L, SLev Lc) {
  int bx, by, bz;
  xcd_block(bx, by, bz);
  const int I = bx * BX + threadIdx.x, J = by * BY + threadIdx.y, K = bz;
  if (I >= Lc.nr || J >= Lc.nth) return;
  const int half = L.nph >> 1, nph = L.nph;
  const long long p1 = L.p1;
  const int p0 = L.p0, hp = L.hp;
  const float* __restrict__ U = L.u;
  const float* __restrict__ F = L.f;
  const long long o = 2 * K * p1 + (long long)(2 * J) * p0 + I;  // fine (2I, 2J, 2K): even half
  float u[2][2][4];  // [plane][row]: radial array indices 2I .. 2I+3
  float f[2][2][2], kn[2][2][2], jn[2][2][2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const long long ok = c ? (2 * K + 2 == nph ? -(long long)2 * K * p1 : 2 * p1) : (K ? -p1 : (nph - 1) * p1);
    const int k = 2 * K + c;
    const long long pole = (long long)((k + half >= nph ? k + half - nph : k + half) - 2 * K) * p1;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const long long q = o + c * p1 + b * p0;
      u[c][b][0] = U[q];
      u[c][b][1] = U[q + hp];
      u[c][b][2] = U[q + 1];
      u[c][b][3] = U[q + hp + 1];
      f[c][b][0] = F[q + hp];
      f[c][b][1] = F[q + 1];
      // the neighbour outside the pair: planes 2K-1 and 2K+2, rows 2J-1 and
      // 2J+2 (across a pole: the row itself half a turn away)
      const long long qk = o + ok + b * p0;
      kn[c][b][0] = U[qk + hp];
      kn[c][b][1] = U[qk + 1];
      long long qj = b ? q + p0 : q - p0;
      if (b ? 2 * J + 2 == L.nth : J == 0) qj = o + pole + b * p0;
      jn[c][b][0] = U[qj + hp];
      jn[c][b][1] = U[qj + 1];
    }
  }
  float s = 0.0f;
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int i = 2 * I + a, j = 2 * J + b;
        const float jp = b ? jn[c][1][a] : u[c][1][a + 1], jm = b ? u[c][0][a + 1] : jn[c][0][a];
        const float kp = c ? kn[1][b][a] : u[1][b][a + 1], km = c ? u[0][b][a + 1] : kn[0][b][a];
        const float off = L.rcr[i] * u[c][b][a + 2] + L.rcl[i] * u[c][b][a] + (L.idt2 + L.cot2[j]) * jp +
                          (L.idt2 - L.cot2[j]) * jm + L.isin2[j] * L.idp2 * (kp + km);
        const float diag = -(L.rcl[i] + L.rcr[i]) - 2.0f * L.idt2 - 2.0f * L.isin2[j] * L.idp2;
        s += f[c][b][a] - (off + diag * u[c][b][a + 1]);
      }
  Lc.f[Lc.at(I + 1, J, K)] = 0.125f * s;
}

// Injection of the coarse correction on the lines of colour 0.  The pass over
// colour 1 that follows overwrites its lines and reads, of their old values,
// only those next to a pole: there both halves of a row are corrected.
// 256 x 128 x 256: 23.6 us for every node, here 15.5.
__global__ __launch_bounds__(256) void k_sprolong(SLev Lc, SLev Lf) {
  const int x = blockIdx.x * BX + threadIdx.x;
  const int j = blockIdx.y * BY + threadIdx.y;
  const int k = blockIdx.z;
  if (x >= Lf.hp || j >= Lf.nth) return;
  const bool pole = j == 0 || j + 1 == Lf.nth;
  // colour 0: i = a - 1 has j's parity
  for (int par = pole ? 0 : 1 - (j & 1); par < 2; par += pole ? 1 : 2) {
    const int i = 2 * x + par - 1;
    if (i >= 0 && i < Lf.nr) Lf.u[Lf.at(i + 1, j, k)] += Lc.u[Lc.at((i >> 1) + 1, j >> 1, k >> 1)];
  }
}

// coarsest level: u = A^-1 f with the dense FP64 inverse, one wavefront per row
__global__ __launch_bounds__(256) void k_scoarse(const double* __restrict__ inv, SLev L) {
  const int N = L.nr * L.nth * L.nph;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= N) return;
  double acc = 0.0;
  for (int col = lane; col < N; col += 64) {
    const int i = col % L.nr, j = (col / L.nr) % L.nth, k = col / (L.nr * L.nth);
    acc += inv[(long long)row * N + col] * (double)L.f[L.at(i + 1, j, k)];
  }
  acc = wave_sum(acc);
  if (lane == 0) {
    const int i = row % L.nr, j = (row / L.nr) % L.nth, k = row / (L.nr * L.nth);
    L.u[L.at(i + 1, j, k)] = (float)acc;
  }
}

__global__ __launch_bounds__(256) void k_scast_in(const double* __restrict__ x, SGeom S, SLev L) {
  const int i = blockIdx.x * BX + threadIdx.x;
  const int j = blockIdx.y * BY + threadIdx.y;
  const int k = blockIdx.z;
  if (i >= S.nr || j >= S.nth) return;
  L.f[L.at(i + 1, j, k)] = (float)x[S.at(i + 1, j, k)];
}

__global__ __launch_bounds__(256) void k_scast_out(SLev L, double* __restrict__ x, SGeom S) {
  const int i = blockIdx.x * BX + threadIdx.x;
  const int j = blockIdx.y * BY + threadIdx.y;
  const int k = blockIdx.z;
  if (i >= S.nr || j >= S.nth) return;
  x[S.at(i + 1, j, k)] = (double)L.u[L.at(i + 1, j, k)];
}

Coef make_coef(const SGeom& S, const SphCoef& sc) {
  Coef c;
  c.idt2 = 1.0 / (S.dth * S.dth);
  c.idp2 = 1.0 / (S.dph * S.dph);
  c.rcl = sc.rcl;
  c.rcr = sc.rcr;
  return c;
}

}  // namespace

int sph_tiles(const SGeom& S) {
  const dim3 g = sgrid(S);
  return (int)(g.x * g.y * g.z);
}

int sph_blocks(const SGeom& S) {
  const dim3 g = rgrid(S);
  return (int)(g.x * g.y * g.z);
}

// go(whether blocks take runs of planes)
template <class Go>
static void by_runs(const SGeom& S, const Go& go) {
  if ((int)rgrid(S).z < S.nph)
    go(std::true_type());
  else
    go(std::false_type());
}

void sph_residual(const double* u, const double* rho, double* r, const SGeom& S, const SphCoef& c,
                  double four_pi_G, bool zu, double* partial, hipStream_t st) {
  const Coef cf = make_coef(S, c);
  by_runs(S, [&](auto runs) {
    if (zu)
      k_sph_residual<runs, true><<<rgrid(S), dim3(BX, BY), 0, st>>>(u, rho, r, S, cf, c.cot, c.isin2, c.r2,
                                                                    four_pi_G, partial);
    else
      k_sph_residual<runs, false><<<rgrid(S), dim3(BX, BY), 0, st>>>(u, rho, r, S, cf, c.cot, c.isin2, c.r2,
                                                                     four_pi_G, partial);
  });
}

void sph_apply(const double* u, double* out, const SGeom& S, const SphCoef& c, hipStream_t st) {
  k_sph_apply<<<sgrid(S), dim3(BX, BY), 0, st>>>(u, out, S, make_coef(S, c), c.cot, c.isin2);
}

void pbicg_direction(const double* r, double* p, const double* v, double* phat, const SGeom& S, const SphCoef& c,
                     const Scalars* scal, hipStream_t st) {
  const Coef cf = make_coef(S, c);
  k_pbicg_p<<<sgrid(S), dim3(BX, BY), 0, st>>>(r, p, v, phat, S, cf, c.isin2, scal, SLev{});
  k_gs_black<<<black_grid(S), dim3(BX, BY), 0, st>>>(p, phat, S, cf, c.cot, c.isin2);
}

void pbicg_update_p(const double* r, double* p, const double* v, const SGeom& S, const SphCoef& c,
                    const Scalars* scal, const SLev& L0, hipStream_t st) {
  k_pbicg_p<<<sgrid(S), dim3(BX, BY), 0, st>>>(r, p, v, nullptr, S, make_coef(S, c), c.isin2, scal, L0);
}

void pbicg_update_s(const double* r, const double* v, double* s, const SGeom& S, const SphCoef& c,
                    const Scalars* scal, const SLev& L0, hipStream_t st) {
  k_pbicg_s<<<sgrid(S), dim3(BX, BY), 0, st>>>(r, v, s, nullptr, S, make_coef(S, c), c.isin2, scal, L0);
}

void pbicg_s(const double* r, const double* v, double* s, double* shat, const SGeom& S, const SphCoef& c,
             const Scalars* scal, hipStream_t st) {
  const Coef cf = make_coef(S, c);
  k_pbicg_s<<<sgrid(S), dim3(BX, BY), 0, st>>>(r, v, s, shat, S, cf, c.isin2, scal, SLev{});
  k_gs_black<<<black_grid(S), dim3(BX, BY), 0, st>>>(s, shat, S, cf, c.cot, c.isin2);
}

template <class H>
static void apply_dot(const H& xhat, double* out, const double* w, int mode, const SGeom& S, const SphCoef& c,
                      double* partial, hipStream_t st) {
  const Coef cf = make_coef(S, c);
  by_runs(S, [&](auto runs) {
    if (mode == 0)
      k_apply_dot<runs, 0><<<rgrid(S), dim3(BX, BY), 0, st>>>(xhat, out, w, S, cf, c.cot, c.isin2, partial);
    else
      k_apply_dot<runs, 1><<<rgrid(S), dim3(BX, BY), 0, st>>>(xhat, out, w, S, cf, c.cot, c.isin2, partial);
  });
}

void pbicg_apply(const double* xhat, double* out, const double* w, int mode, const SGeom& S, const SphCoef& c,
                 double* partial, hipStream_t st) {
  apply_dot(HatD{xhat, S}, out, w, mode, S, c, partial, st);
}
void pbicg_apply32(const SLev& xhat, double* out, const double* w, int mode, const SGeom& S, const SphCoef& c,
                   double* partial, hipStream_t st) {
  apply_dot(HatF{xhat}, out, w, mode, S, c, partial, st);
}

void pbicg_xr(double* x, double* r, const double* phat, const double* shat, const double* s, const double* t,
              const double* rhat, const SGeom& S, const Scalars* scal, double* partial, hipStream_t st) {
  by_runs(S, [&](auto runs) {
    k_pbicg_xr<runs><<<rgrid(S), dim3(BX, BY), 0, st>>>(x, r, HatD{phat, S}, HatD{shat, S}, s, t, rhat, S, scal,
                                                        partial);
  });
}
void pbicg_xr32(double* x, double* r, const SLev& phat, const SLev& shat, const double* s, const double* t,
                const double* rhat, const SGeom& S, const Scalars* scal, double* partial, hipStream_t st) {
  by_runs(S, [&](auto runs) {
    k_pbicg_xr<runs><<<rgrid(S), dim3(BX, BY), 0, st>>>(x, r, HatF{phat}, HatF{shat}, s, t, rhat, S, scal, partial);
  });
}

void bicg_scalars(const double* partial, int nb, Scalars* scal, int stage, hipStream_t st, Post post) {
  k_bicg_scalars<<<1, kFinishThreads, 0, st>>>(partial, nb, scal, stage, post);
}

void sph_line_pass(const SLev& L, int colour, int zero_guess, hipStream_t st) {
  if (sline_fixed(L, colour, zero_guess, st)) return;
  const int nt = L.nl * L.nseg;
  const size_t lds = sizeof(float) * ((size_t)L.seg * nt + (size_t)2 * L.nseg * L.nl);
  const int lines = (L.nr + 1) / 2;
  k_sline<<<dim3((lines + L.nl - 1) / L.nl, L.nth), nt, lds, st>>>(L, colour, zero_guess);
}
void sph_resrestrict32(const SLev& Lf, const SLev& Lc, hipStream_t st) {
  const dim3 grid((Lc.nr + BX - 1) / BX, (Lc.nth + BY - 1) / BY, Lc.nph);
  k_sresrestrict<<<grid, dim3(BX, BY), 0, st>>>(Lf, Lc);
}
void sph_prolong_add32(const SLev& Lc, const SLev& Lf, hipStream_t st) {
  const dim3 grid((Lf.hp + BX - 1) / BX, (Lf.nth + BY - 1) / BY, Lf.nph);
  k_sprolong<<<grid, dim3(BX, BY), 0, st>>>(Lc, Lf);
}
void sph_coarse32(const double* inv, const SLev& L, hipStream_t st) {
  const int N = L.nr * L.nth * L.nph;
  k_scoarse<<<(N + 3) / 4, 256, 0, st>>>(inv, L);
}
void sph_cast_in(const double* x, const SGeom& S, const SLev& L0, hipStream_t st) {
  k_scast_in<<<sgrid(S), dim3(BX, BY), 0, st>>>(x, S, L0);
}
void sph_cast_out(const SLev& L0, double* x, const SGeom& S, hipStream_t st) {
  k_scast_out<<<sgrid(S), dim3(BX, BY), 0, st>>>(L0, x, S);
}

void sph_sor_pass(double* u, const double* rho, const SGeom& S, const SphCoef& c, double four_pi_G,
                  const double* omega, int colour, hipStream_t st, const double* rj, double* omega_out) {
  const dim3 g((S.nr + 2 * BX - 1) / (2 * BX), (S.nth + BY - 1) / BY, S.nph / 2);
  k_sph_sor<<<g, dim3(BX, BY), 0, st>>>(u, rho, S, make_coef(S, c), c.cot, c.isin2, c.r2, four_pi_G, omega, colour,
                                        rj, omega_out);
}

void sph_omega_next(double* omega, const double* rj, int n, hipStream_t st) {
  k_sph_omega<<<(n + 255) / 256, 256, 0, st>>>(omega, rj, n);
}

void sph_fill_zero(double* x, const SGeom& S, hipStream_t st) {
  k_sph_fill<<<dim3((unsigned)((S.p0 + BX - 1) / BX), (S.nth + BY - 1) / BY, S.nph), dim3(BX, BY), 0, st>>>(x, S);
}

void sph_copy(const double* src, double* dst, const SGeom& S, hipStream_t st) {
  k_sph_copy<<<dim3((S.nr + 2 + BX - 1) / BX, (S.nth + BY - 1) / BY, S.nph), dim3(BX, BY), 0, st>>>(src, dst, S);
}

}  // namespace psn
