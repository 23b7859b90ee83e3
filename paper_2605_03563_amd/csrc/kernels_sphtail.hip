// The small levels of the spherical preconditioner's V-cycle in one workgroup:
// every level from the tail's top one down to the dense coarsest solve is
// smoothed, restricted and corrected inside one launch, with u in LDS.
//
// What bounds these levels is latency: at 32 x 16 x 32 and below a phi-line
// pass is 4.2-5 us plus 2-3 us to the next launch, whatever its size, and a
// V(2,2) cycle needs eight of them per level.  Inside one workgroup a pass is
// bound by LDS reads, so the split keeps them few.  A wavefront takes one
// colatitude: 16 lines of a colour, four segments of SL nodes per line, one
// segment per lane, with the right-hand sides of both colours in registers.
// A line's segments meet inside the wavefront (one barrier per pass), and the
// factors of a colatitude are scalars; padded grids, whose factors vary along
// r, read them from LDS.  Planes are pitched so that a wavefront's four
// segments lie in different banks.  No level of more than 16 wavefronts (32 x
// 16 x 32) or 160 KB of LDS, where one compute unit takes as long as the
// launches.
//
// The coarsest operator does not change when phi turns by one step, so the
// rows of its inverse that belong to k = 0 hold all of it (64 KB instead of
// 512 KB at 8 x 4 x 8); nor does the interface system of a line when its
// segments do, so a segment reads the ends in the order of their distance.
//
// Measured, one V(2,2) cycle from 32 x 16 x 32 down to 8 x 4 x 8: 36.5
// us, launch by launch 143.
#include <algorithm>

#include "internal.h"
#include "reduce.h"

namespace psn {

namespace {

constexpr int kThreads = 1024;
constexpr size_t kLds = 160 * 1024;  // LDS of one compute unit
constexpr int kSeg = 4;              // segments per line
constexpr int kCoarse = 512;         // coarsest unknowns: one compute unit reads their inverse

typedef const float __attribute__((address_space(4))) cfloat;  // read-only: scalar loads

// One lane's share of a level: segment seg of line l of both colours at
// colatitude j (uniform over the wavefront)
struct Share {
  int l, j, seg;
  bool task;
  float aphi, cjp, cjm;
  float cl[2], cr[2];  // radial couplings of its line of colour 0 and 1
};

__device__ inline Share share(const SLev& L) {
  Share s;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = w / L.nth;
  s.j = w - g * L.nth;
  s.l = g * 16 + (lane & 15);
  s.seg = lane >> 4;
  s.task = s.l < (L.nr + 1) / 2;
  s.aphi = L.isin2[s.j] * L.idp2;
  s.cjp = L.idt2 + L.cot2[s.j];
  s.cjm = L.idt2 - L.cot2[s.j];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int i = min(2 * s.l + ((s.j + c) & 1), L.nr - 1);
    s.cl[c] = L.rcl[i];
    s.cr[c] = L.rcr[i];
  }
  return s;
}

// The lane's line of a colour: u at the segment's first node (planes p1
// apart) and the steps to its neighbours
struct Spot {
  int i, o, right, left, up, down;
  bool live;
};
template <int SL>
__device__ inline Spot spot(const SLev& L, int p1, const Share& s, int colour) {
  Spot p;
  const int par = (s.j + colour) & 1;
  p.i = 2 * s.l + par;
  p.live = s.task && p.i < L.nr;
  p.o = s.seg * SL * p1 + s.j * L.p0 + (par ? 0 : L.hp) + ((p.i + 1) >> 1);
  p.right = par ? L.hp : 1 - L.hp;
  p.left = par ? L.hp - 1 : -L.hp;
  // across a pole: the line itself half a turn away, two segments on
  const int pole = (s.seg < kSeg / 2 ? kSeg / 2 : -(kSeg / 2)) * SL * p1;
  p.up = s.j + 1 < L.nth ? L.p0 : pole;
  p.down = s.j > 0 ? -L.p0 : pole;
  return p;
}

// N consecutive entries of a line's table: scalars, or a lane's own from LDS
// (16-byte aligned)
template <int N>
__device__ inline void entries(cfloat* t, float (&x)[N]) {
#pragma unroll
  for (int q = 0; q < N; ++q) x[q] = t[q];
}
template <int N>
__device__ inline void entries(const float* t, float (&x)[N]) {
  if constexpr (N % 4 == 0) {
#pragma unroll
    for (int q = 0; q < N; q += 4) *(float4*)(x + q) = *(const float4*)(t + q);
  } else {
#pragma unroll
    for (int q = 0; q < N; ++q) x[q] = t[q];
  }
}

// One colour of phi-line Gauss-Seidel (see k_sline).  E: the wavefront's
// segment ends, E[16 (2 seg + end) + line].
template <int SL, typename TAB>
__device__ inline void pass_on(const SLev& L, int p1, const Share& s, const Spot& p, float cl, float cr, bool zero,
                               float (&y)[SL], float* u, TAB tb, float* E) {
  if (!zero) {
#pragma unroll
    for (int q = 0; q < SL; ++q) {
      const float* v = u + p.o + q * p1;
      y[q] -= cr * v[p.right] + cl * v[p.left] + s.cjp * v[p.up] + s.cjm * v[p.down];
    }
  }
  float ma[SL], mb[SL], gl[2 * kSeg], gr[2 * kSeg];
  entries(tb, ma);
  entries(tb + SL, mb);
  float d = 0.0f;
#pragma unroll
  for (int q = 0; q < SL; ++q) {
    d = (y[q] - s.aphi * d) * ma[q];
    y[q] = d;
  }
#pragma unroll
  for (int q = SL - 2; q >= 0; --q) y[q] -= mb[q] * y[q + 1];
  const int lane = threadIdx.x & 63;
  E[lane] = y[0];
  E[64 + lane] = y[SL - 1];
  // the ends are read by other lanes of the wavefront: the barrier alone orders
  // no memory
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  entries(tb + 4 * SL + (2 * (kSeg - 1) + 1) * 2 * kSeg, gl);  // rows of segment 0's neighbours
  entries(tb + 4 * SL + 2 * 2 * kSeg, gr);
  float xl = 0.0f, xr = 0.0f;
#pragma unroll
  for (int q = 0; q < kSeg; ++q)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float x = E[64 * e + ((lane + 16 * q) & 63)];
      xl += gl[2 * q + e] * x;
      xr += gr[2 * q + e] * x;
    }
  xl *= s.aphi;
  xr *= s.aphi;
  entries(tb + 2 * SL, ma);
  entries(tb + 3 * SL, mb);
#pragma unroll
  for (int q = 0; q < SL; ++q) u[p.o + q * p1] = y[q] - (xl * ma[q] + xr * mb[q]);
}

template <int SL, bool UNI>
__device__ inline void pass(const SLev& L, int p1, const Share& s, int colour, bool zero, const float (&f)[2][SL],
                            float* u, const float* tab, float* E) {
  const Spot p = spot<SL>(L, p1, s, colour);
  if (p.live) {
    const float cl = colour ? s.cl[1] : s.cl[0], cr = colour ? s.cr[1] : s.cr[0];
    float y[SL];
#pragma unroll
    for (int q = 0; q < SL; ++q) y[q] = colour ? f[1][q] : f[0][q];
    if constexpr (UNI)
      pass_on<SL>(L, p1, s, p, cl, cr, zero, y, u, (cfloat*)(L.ltab + s.j * L.tstride), E);
    else
      pass_on<SL>(L, p1, s, p, cl, cr, zero, y, u, tab + (min(p.i, L.ntab - 1) * L.nth + s.j) * L.tstride, E);
  }
  __syncthreads();
}

template <int SL, bool UNI>
__device__ inline void smooth(const SLev& L, int p1, const Share& s, int n, int first, bool zero,
                              const float (&f)[2][SL], float* u, const float* tab, float* E) {
#pragma unroll 1
  for (int q = 0; q < 2 * n; ++q) pass<SL, UNI>(L, p1, s, (q & 1) ^ first, zero && q == 0, f, u, tab, E);
}

// Dense coarsest solve: u = A^-1 f, f twice in the order i, j, k.  Thread
// (m, part) adds up its share of the columns for unknown m = (i, j) of four
// planes at a time, so that an entry of A^-1 serves four planes and the sum
// over a wavefront's lanes, longer than the products, is not needed; S holds
// the partial sums.
__device__ inline void solve(const SphTail& A, const SLev& L, const float* f, float* u, double* S) {
  const int M = L.nr * L.nth, N = M * L.nph;
  const int parts = kThreads / M, t = threadIdx.x, pitch = 4 * M + 2;
  const int part = t / M, m = t - part * M;
  const int share = (N + parts - 1) / parts, c0 = part * share, c1 = min(c0 + share, N);
  for (int k0 = 0; k0 < L.nph; k0 += 4) {
    const int last = L.nph - 1 - k0;  // a fourth plane beyond the last repeats it
    const float* fk[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) fk[q] = f + (k0 + min(q, last)) * M;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (part < parts) {
#pragma unroll 8
      for (int c = c0; c < c1; ++c) {
        const double a = A.inv[c * M + m];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] += a * (double)fk[q][c];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) S[part * pitch + q * M + m] = acc[q];
    }
    __syncthreads();
    for (int h = t; h < 4 * M * 8; h += kThreads) {  // eight lanes per sum
      const int e = h >> 3, q = e / M, x = e - q * M;
      double sum = 0.0;
      for (int r = h & 7; r < parts; r += 8) sum += S[r * pitch + e];
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) sum += __shfl_xor(sum, o, 64);
      const int j = x / L.nr;
      if (q <= last && (h & 7) == 0) u[L.at(x - j * L.nr + 1, j, k0 + q)] = (float)sum;
    }
    __syncthreads();
  }
}

// One V cycle from level LV on: u = 0 on entry (LDS), f the lane's right-hand
// sides
template <int SL, int LV, bool UNI>
__device__ inline void cycle(const SphTail& A, const float (&f)[2][SL], char* lds) {
  const SLev& L = A.lv[LV];
  const int p1 = A.p1[LV];
  float* u = (float*)(lds + A.u[LV]);
  const float* tab = (const float*)(lds + A.tab[LV]);
  float* R = (float*)lds;                          // residuals; in a pass
  float* E = (float*)lds + (threadIdx.x >> 6) * 128;  // the segment ends
  Share s = share(L);
  smooth<SL, UNI>(L, p1, s, A.nu1, 0, true, f, u, tab, E);
  // residuals, for an even segment already summed over the planes of a pair
  constexpr int PAIR = SL % 2 == 0 ? 2 : 1;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const Spot p = spot<SL>(L, p1, s, c);
    if (!p.live) continue;
    const float diag = -(s.cl[c] + s.cr[c]) - 2.0f * L.idt2 - 2.0f * s.aphi;
    float v[SL + 2];
    v[0] = u[p.o + (s.seg ? -1 : L.nph - 1) * p1];
#pragma unroll
    for (int q = 0; q < SL; ++q) v[q + 1] = u[p.o + q * p1];
    v[SL + 1] = u[p.o + (s.seg < kSeg - 1 ? SL : SL - L.nph) * p1];
    float r[SL];
#pragma unroll
    for (int q = 0; q < SL; ++q) {
      const float* w = u + p.o + q * p1;
      const float off = s.cr[c] * w[p.right] + s.cl[c] * w[p.left] + s.cjp * w[p.up] + s.cjm * w[p.down] +
                        s.aphi * (v[q + 2] + v[q]);
      r[q] = f[c][q] - (off + diag * v[q + 1]);
    }
#pragma unroll
    for (int q = 0; q < SL; q += PAIR)
      R[((s.seg * SL + q) / PAIR * L.nth + s.j) * L.nr + p.i] = PAIR == 2 ? r[q] + r[q + PAIR - 1] : r[q];
  }
  __syncthreads();
  const SLev& C = A.lv[LV + 1];
  const bool last = LV + 1 == A.nl;
  float* Fc = (float*)(lds + A.f[LV + 1]);
  const unsigned M = C.nr * C.nth * C.nph;
  for (unsigned t = threadIdx.x; t < M; t += kThreads) {
    const unsigned row = t / C.nr, I = t - row * C.nr, K = row / C.nth, J = row - K * C.nth;
    float sum = 0.0f;
#pragma unroll
    for (int c = 0; c < 2 / PAIR; ++c)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int a = 0; a < 2; ++a) sum += R[((K * (2 / PAIR) + c) * L.nth + 2 * J + b) * L.nr + 2 * I + a];
    sum *= 0.125f;
    Fc[t] = sum;
    if (last) Fc[t + M] = sum;
  }
  __syncthreads();
  float* uc = (float*)(lds + A.u[LV + 1]);
  if constexpr (LV + 1 < SphTail::kLevels && SL % 2 == 0 && SL >= 4) {
    if (!last) {
      constexpr int SC = SL / 2;
      const Share sc = share(C);
      float fc[2][SC];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const Spot p = spot<SC>(C, A.p1[LV + 1], sc, c);
#pragma unroll
        for (int q = 0; q < SC; ++q) fc[c][q] = p.live ? Fc[((sc.seg * SC + q) * C.nth + sc.j) * C.nr + p.i] : 0.0f;
      }
      cycle<SC, LV + 1, UNI>(A, fc, lds);
    } else {
      solve(A, C, Fc, uc, (double*)lds);
    }
  } else {
    solve(A, C, Fc, uc, (double*)lds);
  }
  __syncthreads();
  s = share(L);  // read again: held through the levels below it would spill
  // injection on the lines of colour 0, at the poles on both (see k_sprolong)
  const int pc = A.p1[LV + 1];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const Spot p = spot<SL>(L, p1, s, c);
    if (!p.live || (c == 1 && s.j > 0 && s.j + 1 < L.nth)) continue;
    const int oc = (s.j >> 1) * C.p0 + (((p.i >> 1) + 1) & 1) * C.hp + (((p.i >> 1) + 1) >> 1);
    float e[SL];
#pragma unroll
    for (int q = 0; q < SL; ++q) e[q] = uc[oc + ((s.seg * SL + q) >> 1) * pc];
#pragma unroll
    for (int q = 0; q < SL; ++q) u[p.o + q * p1] += e[q];
  }
  __syncthreads();
  smooth<SL, UNI>(L, p1, s, A.nu2, 1, false, f, u, tab, E);
}

// LDS: residuals / segment ends / partial sums, then per level u, tables, right-hand side
template <int SL, bool UNI>
__global__ __launch_bounds__(kThreads) void k_stail(SphTail A) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const SLev& L = A.lv[0];
  const Share s = share(L);
  float f[2][SL];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const Spot p = spot<SL>(L, (int)L.p1, s, c);
#pragma unroll
    for (int q = 0; q < SL; ++q) f[c][q] = 0.0f;
    if (p.live)
#pragma unroll
      for (int q = 0; q < SL; ++q) f[c][q] = L.f[p.o + q * (int)L.p1];
  }
  for (int l = 0; l <= A.nl; ++l) {
    const SLev& K = A.lv[l];
    float4* u = (float4*)(lds + A.u[l]);
    const int n = (A.p1[l] * K.nph + 3) / 4;  // zero: radial ghosts, and the guess
    for (int t = threadIdx.x; t < n; t += kThreads) u[t] = float4{0.0f, 0.0f, 0.0f, 0.0f};
    if (UNI || l == A.nl) continue;
    float* tab = (float*)(lds + A.tab[l]);
    const int nt = K.tstride * K.nth * K.ntab;
    for (int t = threadIdx.x; t < nt; t += kThreads) tab[t] = K.ltab[t];
  }
  __syncthreads();
  cycle<SL, 0, UNI>(A, f, lds);
  const float* u = (const float*)(lds + A.u[0]);
  const Share e = share(L);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const Spot p = spot<SL>(L, A.p1[0], e, c), g = spot<SL>(L, (int)L.p1, e, c);
    if (p.live)
#pragma unroll
      for (int q = 0; q < SL; ++q) L.u[g.o + q * (int)L.p1] = u[p.o + q * A.p1[0]];
  }
}

template <bool UNI, typename F>
bool by_segment(int sl, const F& go) {
  switch (sl) {
    case 2: go(k_stail<2, UNI>); return true;
    case 3: go(k_stail<3, UNI>); return true;
    case 4: go(k_stail<4, UNI>); return true;
    case 5: go(k_stail<5, UNI>); return true;
    case 6: go(k_stail<6, UNI>); return true;
    case 7: go(k_stail<7, UNI>); return true;
    case 8: go(k_stail<8, UNI>); return true;
    default: return false;
  }
}

}  // namespace

// whether a wavefront per colatitude and 16 lines of a colour fits
static bool tail_level(const SLev& L) {
  const int sl = L.nph / kSeg;
  return L.nph % kSeg == 0 && sl >= 2 && sl <= 8 && ((L.nr + 1) / 2 + 15) / 16 * L.nth <= kThreads / 64;
}

void sph_tail_split(SLev& L) {
  L.seg = L.nph / kSeg;
  L.nseg = kSeg;
  L.nl = 1;  // used by the launches of one pass only
  L.tstride = 4 * L.seg + 4 * kSeg * kSeg;
}

bool sph_tail_args(const SLev* lv, int nl, int nu1, int nu2, SphTail& A) {
  if (nl < 2 || nl - 1 > SphTail::kLevels) return false;
  const SLev& last = lv[nl - 1];
  if (last.nr * last.nth * last.nph > kCoarse) return false;
  A.nl = nl - 1;
  A.nu1 = nu1;
  A.nu2 = nu2;
  A.inv = nullptr;
  size_t at = 0;
  auto take = [&](size_t bytes) {
    const size_t o = at;
    at += (bytes + 15) / 16 * 16;
    return (int)o;
  };
  size_t scratch = 8 * (4 + 2) * kThreads;  // partial sums of the coarsest solve; segment ends take less
  A.uniform = true;
  for (int l = 0; l < A.nl; ++l) {
    const SLev& L = lv[l];
    if (!tail_level(L) || (l > 0 && lv[l - 1].nph / kSeg % 2)) return false;  // the kernel halves its segment
    const size_t n = (size_t)L.nr * L.nth * L.nph;
    scratch = std::max(scratch, 4 * (L.nph / kSeg % 2 ? n : n / 2));
    A.uniform = A.uniform && L.ntab == 1;
  }
  take(scratch);
  for (int l = 0; l <= A.nl; ++l) {
    const SLev& L = lv[l];
    A.lv[l] = L;
    A.p1[l] = (int)L.p1;
    if (l < A.nl) {
      // plane pitch: the banks of a wavefront's segments overlap least
      const int w = std::min(16, (L.nr + 1) / 2), sl = L.nph / kSeg;
      int best = 1 << 30;
      for (int pad = 0; pad < 64; ++pad) {
        int hits[64] = {}, most = 0;
        for (int g = 0; g < kSeg; ++g)
          for (int q = 0; q < w; ++q) most = std::max(most, ++hits[(g * sl * ((int)L.p1 + pad) + q) % 64]);
        if (most < best) {
          best = most;
          A.p1[l] = (int)L.p1 + pad;
        }
      }
    }
    A.u[l] = take(4 * (size_t)A.p1[l] * L.nph);
    A.tab[l] = l < A.nl && !A.uniform ? take(4 * (size_t)(L.nph + 4 * kSeg * kSeg) * L.nth * L.ntab) : 0;
    A.f[l] = l ? take((l < A.nl ? 4 : 2 * 4) * (size_t)L.nr * L.nth * L.nph) : 0;
    if (at > kLds) return false;
  }
  A.lds = at;
  return true;
}

bool sph_tail_enable(const SphTail& A) {
  bool ok = false;
  auto set = [&](auto k) {
    ok = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds) == hipSuccess;
  };
  return (A.uniform ? by_segment<true>(A.lv[0].seg, set) : by_segment<false>(A.lv[0].seg, set)) && ok;
}

void sph_tail_inverse(const SLev& L, const std::vector<double>& inv, std::vector<double>& out) {
  const size_t M = (size_t)L.nr * L.nth, N = M * L.nph;
  out.resize(M * N);
  for (size_t c = 0; c < N; ++c)
    for (size_t m = 0; m < M; ++m) out[c * M + m] = inv[m * N + c];
}

void sph_tail_cycle(const SphTail& A, hipStream_t st) {
  auto go = [&](auto k) { k<<<1, kThreads, A.lds, st>>>(A); };
  if (A.uniform)
    by_segment<true>(A.lv[0].seg, go);
  else
    by_segment<false>(A.lv[0].seg, go);
}

}  // namespace psn
