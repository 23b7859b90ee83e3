// Residual and operator of the 7-point and the 19-point star stencil on the
// caller's arrays (natural order), for the operator entry points.
//
// Bound by HBM: f and u are read, r is written, 24 bytes per node.  Converting
// both inputs to the colour-split layout and the result back moved 72 more.  A
// wavefront owns 64 - 2 RAD columns and R rows and marches the planes of its
// run with no LDS and no barrier: lane l holds column x0 - RAD + l, a window of
// 2 RAD + 1 planes of its own rows in registers (the next plane's loads underway),
// x-neighbours come by lane shifts, and the RAD rows on either side, needed
// for one plane only, through the cache from the wavefronts beside, four of
// them stacked in a block.
//
// Measured with the norm, star stencil, 201^3: 60 us, 3.3 TB/s of the 24 bytes
// (2 rows per wavefront 65); conversions, residual and conversion back 197.
#include <algorithm>

#include "internal.h"
#include "reduce.h"

namespace psn {

namespace {

constexpr double kC0 = -49.0 / 18.0, kC1 = 1.5, kC2 = -3.0 / 20.0, kC3 = 1.0 / 90.0;  // 19-point star
constexpr int kRows = 4;

// value of the lane to the left (DIR < 0) or right; only lanes whose
// neighbours lie in the wavefront use it
template <int DIR>
__device__ inline double beside(double v) {
  constexpr int ctrl = DIR < 0 ? 0x138 : 0x130;  // wave_shr:1, wave_shl:1
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), ctrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), ctrl, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// nodes per axis M with g = RAD ghost layers; RES: r = scale rho - L u with the
// squares summed into one partial per block, otherwise r = L u
template <int RAD, bool RES>
__global__ __launch_bounds__(256) void k_star(const double* __restrict__ u, const double* __restrict__ rho,
                                              double* __restrict__ r, long long p0, long long p1, int M, double scale,
                                              double ih2, double* __restrict__ partial) {
  constexpr int R = kRows, WX = 64 - 2 * RAD;
  int bx, by, bz;
  xcd_block(bx, by, bz);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int x = bx * WX + lane, y0 = RAD + (by * 4 + wave) * R;  // array indices
  const int last = M - 1 - RAD;                                   // last unknown
  const int kz = (M - 2 * RAD + (int)gridDim.z - 1) / (int)gridDim.z;
  const int kb = RAD + bz * kz, ke = min(kb + kz - 1, last);
  const bool mine = lane >= RAD && lane < 64 - RAD && x <= last;
  double acc = 0.0;
  if (y0 <= last && kb <= ke) {
    const int cx = min(x, M - 1);  // loads stay in the array
    long long row[R + 2 * RAD];
#pragma unroll
    for (int i = 0; i < R + 2 * RAD; ++i) row[i] = (long long)min(y0 - RAD + i, M - 1) * p0 + cx;
    double w[2 * RAD + 1][R], next[R];  // own rows of planes k - RAD .. k + RAD, and the next
#pragma unroll
    for (int d = 0; d < 2 * RAD; ++d)
#pragma unroll
      for (int i = 0; i < R; ++i) w[d + 1][i] = u[(kb - RAD + d) * p1 + row[RAD + i]];
    double side[2 * RAD], fn[R];  // the next plane's rows on either side, and rho
    auto load = [&](int k) {
      const double* uk = u + k * p1;
      const double* up = u + min(k + RAD, M - 1) * p1;
#pragma unroll
      for (int i = 0; i < RAD; ++i) {
        side[i] = uk[row[i]];
        side[RAD + i] = uk[row[RAD + R + i]];
      }
#pragma unroll
      for (int i = 0; i < R; ++i) next[i] = up[row[RAD + i]];
      if (RES) {
#pragma unroll
        for (int i = 0; i < R; ++i) fn[i] = rho[k * p1 + row[RAD + i]];
      }
    };
    load(kb);
    for (int k = kb; k <= ke; ++k) {
      double c[R + 2 * RAD], f[R];
#pragma unroll
      for (int i = 0; i < R; ++i) {
#pragma unroll
        for (int d = 0; d < 2 * RAD; ++d) w[d][i] = w[d + 1][i];
        w[2 * RAD][i] = next[i];
        f[i] = RES ? __dmul_rn(scale, fn[i]) : 0.0;
        c[RAD + i] = w[RAD][i];
      }
#pragma unroll
      for (int i = 0; i < RAD; ++i) {
        c[i] = side[i];
        c[RAD + R + i] = side[RAD + i];
      }
      const long long pk = k * p1;
      load(min(k + 1, ke));
#pragma unroll
      for (int i = 0; i < R; ++i) {
        // summed in the order of the colour-split residual kernels
        const double m = c[RAD + i];
        double sd[RAD], l = m, q = m;
#pragma unroll
        for (int d = 1; d <= RAD; ++d) {
          l = beside<-1>(l);
          q = beside<1>(q);
          sd[d - 1] = q + l + c[RAD + i + d] + c[RAD + i - d] + w[RAD + d][i] + w[RAD - d][i];
        }
        double lap;
        if constexpr (RAD == 1)
          lap = (sd[0] - 6.0 * m) * ih2;
        else
          lap = (3.0 * kC0 * m + kC1 * sd[0] + kC2 * sd[1] + kC3 * sd[2]) * ih2;
        const double v = RES ? f[i] - lap : lap;
        if (mine && y0 + i <= last) {
          r[pk + row[RAD + i]] = v;
          acc += v * v;
        }
      }
    }
  }
  if (RES) {
    const double b = block_sum(acc);
    if (threadIdx.x == 0) partial[linear_block()] = b;
  }
}

// A few blocks for every CU, in runs of 8 planes or more (a run reads 2 RAD
// planes twice): 201^3 takes 60 us in 9 to 19 runs, 63 in 25.
dim3 star_grid(const Geom& G) {
  const int e = G.n - 1, wx = 64 - 2 * G.g;
  const int bx = (e + wx - 1) / wx, by = (e + 4 * kRows - 1) / (4 * kRows);
  const int runs = std::max(1, std::min((e + 7) / 8, 1024 / (bx * by)));
  return dim3(bx, by, runs);
}

template <int RAD>
void star_go(const double* u, const double* rho, double* r, long long p0, long long p1, const Geom& G, double scale,
             double* partial, hipStream_t st) {
  const double ih2 = 1.0 / (G.h * G.h);
  if (rho)
    k_star<RAD, true><<<star_grid(G), 256, 0, st>>>(u, rho, r, p0, p1, G.M, scale, ih2, partial);
  else
    k_star<RAD, false><<<star_grid(G), 256, 0, st>>>(u, rho, r, p0, p1, G.M, scale, ih2, partial);
}

}  // namespace

int star_blocks(const Geom& G) {
  const dim3 g = star_grid(G);
  return (int)(g.x * g.y * g.z);
}

void star_residual(const double* u, const double* rho, double* r, long long p0, long long p1, const Geom& G,
                   double scale, double* partial, hipStream_t st) {
  if (G.g == 1)
    star_go<1>(u, rho, r, p0, p1, G, scale, partial, st);
  else
    star_go<3>(u, rho, r, p0, p1, G, scale, partial, st);
}

}  // namespace psn
