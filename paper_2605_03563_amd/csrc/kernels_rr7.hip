// Residual of the 7-point operator fused with full weighting on large levels,
// after a Gauss-Seidel pass over colour 1: only colour-0 residuals are formed
// (f and u of colour 0, and u of colour 1 around them, 12 bytes per fine
// unknown in FP64).
//
// A wavefront owns one coarse row, i.e. three fine rows across the whole
// level (V compact columns per lane, V 64 >= n/2), and marches fine planes
// with no LDS and no barrier.  In row b and plane k colour 0 sits at fine
// nodes 2m or 2m + 1 according to the parity of b + k, the same for all
// lanes, so each row takes one of two forms: its neighbours in x are column m
// and m - 1 or m + 1 of colour 1 (lane shifts), those in y and z the same
// column of the rows and planes beside.  Rows of colour 1 for the plane after
// the next, and u, f and the two outer rows of the next one are underway
// while a plane is computed; four wavefronts stacked in y share rows through
// the cache.
//
// Measured (us; in parentheses a block across the level with residuals and
// x-sums in LDS, two barriers per plane): FP64 255^3 44.8 (84.7), 4.4 TB/s of
// the bytes above; FP64 127^3 12.0 (12.6); FP32 127^3 6.4 (9.1).
#include <algorithm>

#include "internal.h"
#include "reduce.h"

namespace psn {

namespace {

// value of the lane to the left (DIR < 0) or right; 0 past the wavefront's ends
template <int DIR>
__device__ inline double beside(double v) {
  constexpr int ctrl = DIR < 0 ? 0x138 : 0x130;  // wave_shr:1, wave_shl:1
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), ctrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), ctrl, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
template <int DIR>
__device__ inline float beside(float v) {
  constexpr int ctrl = DIR < 0 ? 0x138 : 0x130;
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true));
}

template <typename T, int V>
struct Cols {
  T v[V];
};
template <typename T, int V>
__device__ inline Cols<T, V> get(const T* p) {  // aligned to V elements
  typedef T Vec __attribute__((ext_vector_type(V)));
  Cols<T, V> c;
  if constexpr (V == 1) {
    c.v[0] = *p;
  } else {
    const Vec x = *reinterpret_cast<const Vec*>(p);
#pragma unroll
    for (int e = 0; e < V; ++e) c.v[e] = x[e];
  }
  return c;
}

template <typename T, int V>
__global__ __launch_bounds__(256) void k_rr7w(const T* __restrict__ X, const T* __restrict__ F, Geom Gf,
                                              T* __restrict__ Fc, Geom Gc, T ih2) {
  typedef Cols<T, V> C;
  int bx, by, bz;
  xcd_block(bx, by, bz);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int n = Gf.n, nc = Gc.n;
  const int B = 1 + by * 4 + wave;
  const int kz = (nc - 1 + (int)gridDim.z - 1) / (int)gridDim.z;
  const int K0 = 1 + bz * kz, K1 = min(K0 + kz - 1, nc - 1);
  if (B > nc - 1 || K0 > K1) return;
  const int m0 = V * lane, mhi = Gf.mhi();
  const long long plane = (long long)Gf.M * Gf.W;
  const int b0 = 2 * B - 1;
  const int mc = min(m0, Gf.W - V);  // loads stay in the row
  const T* x0 = X + (long long)b0 * Gf.W + mc;
  const T* x1 = x0 + Gf.cs;
  const T* f0 = F + (long long)b0 * Gf.W + mc;
  // the last lane's right neighbour, where the level has 64 V columns
  const bool edge = lane == 63 && mhi >= 64 * V - 1;
  auto own = [&](int k, C (&c)[3]) {  // colour 1, own rows
#pragma unroll
    for (int i = 0; i < 3; ++i) c[i] = get<T, V>(x1 + (long long)k * plane + i * Gf.W);
  };
  C lo[3], cu[3], hi[3], nx[3], sd[2], sn[2], c0[3], c0n[3], f[3], fn[3];
  T er[3] = {}, ern[3] = {};
  auto rest = [&](int k) {
    const long long o = (long long)k * plane;
    sn[0] = get<T, V>(x1 + o - Gf.W);
    sn[1] = get<T, V>(x1 + o + 3 * Gf.W);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      c0n[i] = get<T, V>(x0 + o + i * Gf.W);
      fn[i] = get<T, V>(f0 + o + i * Gf.W);
      if (edge) ern[i] = x1[o + i * Gf.W + V];
    }
  };
  const int kf0 = 2 * K0 - 1, kf1 = 2 * K1 + 1;
  own(kf0 - 1, cu);
  own(kf0, hi);
  own(kf0 + 1, nx);
  rest(kf0);
  T acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] = (T)0;
  const T q = (T)0.25, hf = (T)0.5;
  for (int k = kf0; k <= kf1; ++k) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      lo[i] = cu[i];
      cu[i] = hi[i];
      hi[i] = nx[i];
      c0[i] = c0n[i];
      f[i] = fn[i];
      er[i] = ern[i];
    }
    sd[0] = sn[0];
    sd[1] = sn[1];
    own(min(k + 2, n), nx);
    rest(min(k + 1, kf1));
    T rx[3][V];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const C& dn = i == 0 ? sd[0] : cu[i - 1];
      const C& up = i == 2 ? sd[1] : cu[i + 1];
      const int s = (b0 + i + k + Gf.off) & 1;
      T r[V];
      if (s == 0) {  // colour 0 at nodes 2m
        const T left = beside<-1>(cu[i].v[V - 1]);
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const T sx = (e ? cu[i].v[e - 1] : left) + cu[i].v[e];
          const T sy = dn.v[e] + up.v[e] + (lo[i].v[e] + hi[i].v[e]);
          r[e] = Gf.inner(2 * (m0 + e)) ? f[i].v[e] - ((sx + sy) - (T)6 * c0[i].v[e]) * ih2 : (T)0;
          rx[i][e] = hf * r[e];
        }
      } else {  // at nodes 2m + 1
        T right = beside<1>(cu[i].v[0]);
        right = edge ? er[i] : right;
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const T sx = cu[i].v[e] + (e + 1 < V ? cu[i].v[e + 1] : right);
          const T sy = dn.v[e] + up.v[e] + (lo[i].v[e] + hi[i].v[e]);
          r[e] = Gf.inner(2 * (m0 + e) + 1) ? f[i].v[e] - ((sx + sy) - (T)6 * c0[i].v[e]) * ih2 : (T)0;
        }
        const T left = beside<-1>(r[V - 1]);
#pragma unroll
        for (int e = 0; e < V; ++e) rx[i][e] = q * ((e ? r[e - 1] : left) + r[e]);
      }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const T ry = hf * rx[1][e] + q * (rx[0][e] + rx[2][e]);
      if (k & 1) {
        // odd plane 2K+1: closes coarse plane K (unless k = kf0) and opens K+1
        acc[e] += q * ry;
        const int A = m0 + e;
        if (k > kf0 && A >= 1 && A <= nc - 1) Fc[Gc.at(A, B, (k - 1) >> 1)] = acc[e];
        acc[e] = q * ry;
      } else {
        acc[e] += hf * ry;
      }
    }
  }
}

template <typename T, int V>
void go(const T* phi, const T* f, const Geom& Gf, T* fc, const Geom& Gc, hipStream_t st) {
  const int by = (Gc.n - 1 + 3) / 4;
  // four blocks per CU: 255^3 FP64 44.8 us (47.1 with three, 50.2 with six)
  const int runs = std::max(1, std::min(Gc.n - 1, 1024 / by));
  k_rr7w<T, V><<<dim3(1, by, runs), 256, 0, st>>>(phi, f, Gf, fc, Gc, (T)(1.0 / (Gf.h * Gf.h)));
}

template <typename T>
void go_v(const T* phi, const T* f, const Geom& Gf, T* fc, const Geom& Gc, hipStream_t st) {
  if (Gf.mhi() + 1 <= 64)
    go<T, 1>(phi, f, Gf, fc, Gc, st);
  else
    go<T, 2>(phi, f, Gf, fc, Gc, st);
}

}  // namespace

void resrestrict7_rows(const void* phi, const void* f, bool f32, const Geom& Gf, void* fc, const Geom& Gc,
                       hipStream_t st) {
  if (f32)
    go_v((const float*)phi, (const float*)f, Gf, (float*)fc, Gc, st);
  else
    go_v((const double*)phi, (const double*)f, Gf, (double*)fc, Gc, st);
}

}  // namespace psn
