// Four-colour Gauss-Seidel pass of the 19-point star on large levels
// (Section 2.1.2), the kernel that carries the 19-point multigrid.
//
// A pass reads three quarter arrays and the right-hand side's quarter and
// writes one (10 B per unknown in FP64).  It is bound by the loads' latency
// together with what crosses from memory into the L2s: a plane's values are
// wanted once as the leading value of the window along z, and 1-3 planes later
// by the rows above and below, when the L2 (4 MB per XCD, 2.6 MB per plane of
// its blocks) has lost them.  So blocks are tall (1024 lanes are 16 rows at
// 511^3, whose twelve halo rows are three quarters of a quarter array more),
// runs along z long, and each plane's loads are underway while the one before
// is computed, in LDS, since registers for them would halve the wavefronts.
//
// Measured (us, before: 256-lane blocks of short runs that load each plane
// when it is wanted): FP64 511^3 359 -> 297 (4.5 TB/s algorithmic), 383^3
// 163 -> 139, 255^3 51 -> 39, 191^3 23.3 -> 20.0, 127^3 9.6 -> 8.0; FP32 511^3
// 195 -> 177, 383^3 100 -> 78, 255^3 29 -> 24, 127^3 8.1 -> 6.9.  Bitwise the
// same results.  Rotating the window's registers by unrolling five planes
// instead of moving them spilled: 484 us.
#include <algorithm>

#include "internal.h"
#include "reduce.h"

namespace psn {

namespace {

constexpr double kC0 = -49.0 / 18.0, kC1 = 1.5, kC2 = -3.0 / 20.0, kC3 = 1.0 / 90.0;

template <typename T> struct Vec16;
template <> struct Vec16<double> { typedef double type __attribute__((ext_vector_type(2))); };
template <> struct Vec16<float> { typedef float type __attribute__((ext_vector_type(4))); };

// One 16-byte load per lane from base + off (bytes) straight into LDS, at
// lds + 16 lane (lds: the wavefront's byte offset).  Written in assembly, since the compiler makes
// every LDS read that follows its builtin wait for it; the caller waits with
// loads_done() before the data is read.
__device__ inline void load_to_lds(const void* base, unsigned off, unsigned lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds)
               : "memory", "m0");
}
// barrier for LDS data alone: stores and loads from memory stay underway
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ inline void lds_read() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ inline void loads_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// 16-byte groups per row: up to the column of the last unknown's right-most
// neighbour, so that no x-neighbour lies in the next row's first group
template <typename T>
__host__ __device__ inline int groups(const Geom& G) { return ((G.M - 1) >> 2) / (16 / (int)sizeof(T)) + 1; }

// Positions are the (group of 16 bytes, row) pairs of the unknowns' rows,
// numbered along the rows; a block owns BP consecutive ones, one per lane, and
// marches the planes of its run.  Of colour c + 1 + e (slot e) a lane keeps its
// own column's five planes between the offsets the star reads (k-3 .. k+1,
// k-2 .. k+2, k-1 .. k+3) in registers.  The next plane of each, and of the
// right-hand side, travel into LDS while the current plane is computed, and
// the rows above and below the block into registers; the LDS array of slot e
// holds the centre plane of the block's positions with up(e) rows before and
// dn(e) rows after them, so every x- and y-neighbour is one read at a fixed
// distance.  A plane's result is stored one plane later, after the wait for
// the loads: the store has a plane's time before the next wait, which counts
// stores with the loads.
template <typename T, int BP, bool ZM>
__global__ __launch_bounds__(BP, 4) void k_pass19w(T* __restrict__ X, const T* __restrict__ F, Geom G,
                                                                   int c, T h2, int zmask) {
  typedef typename Vec16<T>::type V;
  constexpr int CPL = 16 / sizeof(T);
  extern __shared__ __attribute__((aligned(16))) char smem[];
  V* lds = reinterpret_cast<V*>(smem);
  int bx, by, bz;
  xcd_block(bx, by, bz);
  const int tid = threadIdx.x;
  const int ngr = groups<T>(G);
  const int E = G.n - 1, nfl = ngr * E;
  const int p0 = bx * BP, p = p0 + tid;
  const bool live = p < nfl;
  const int last = G.g + E - 1;
  const int kz = (E + (int)gridDim.z - 1) / (int)gridDim.z;
  const int k0 = G.g + bz * kz, k1 = min(k0 + kz - 1, last);
  const long long plane = (long long)G.M * G.W;
  // element offset of position q (at most three rows outside the unknowns) in a plane
  auto offset = [&](int q) -> int {
    q = min(q, nfl - 1 + 3 * ngr) + 3 * ngr;
    const int row = q / ngr;
    return (G.g - 3 + row) * G.W + (q - row * ngr) * CPL;
  };
  // positions past the unknowns hold ghost rows, which the last rows read
  const unsigned own = offset(p) * (unsigned)sizeof(T);  // bytes
  const int m0 = p % ngr * CPL, b = G.g + p / ngr;
  bool zero[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) zero[e] = ZM && ((zmask >> ((c + e + 1) & 3)) & 1);
  auto array = [&](int e, int k) -> const char* {  // slot e on plane k
    return reinterpret_cast<const char*>(X + (long long)((c + e + 1) & 3) * G.cs + k * plane);
  };
  // LDS in chunks: four staged chunks per lane, then the slots' centre arrays
  const int up[3] = {3 * ngr, 2 * ngr, ngr}, dn[3] = {ngr, 2 * ngr, 3 * ngr};
  const int base0 = 4 * BP + up[0], base1 = base0 + BP + dn[0] + up[1], base2 = base1 + BP + dn[1] + up[2];
  const unsigned wave = __builtin_amdgcn_readfirstlane((unsigned)(tid & ~63) * 16);
  // halo chunks: up(e) then dn(e) positions of each slot, 12 ngr in all
  unsigned hoff;  // bytes
  int hlds;       // chunk in LDS; -1: none
  bool clear = false;
  {
    const int h = tid;
    const int e = h < 4 * ngr ? 0 : h < 8 * ngr ? 1 : 2;
    const int r = h - 4 * ngr * e;
    const int q = r < up[e] ? r - up[e] : BP + r - up[e];
    hlds = h < 12 * ngr ? (e == 0 ? base0 : e == 1 ? base1 : base2) + q : -1;
    hoff = ((unsigned)(((c + e + 1) & 3) * G.cs) + offset(p0 + q)) * (unsigned)sizeof(T);
    if (ZM && hlds >= 0 && (zmask >> ((c + e + 1) & 3) & 1)) clear = true;  // a zero colour is not loaded
  }
  V hv;
  const T* Fc = F + (long long)c * G.cs;
  auto issue = [&](int k) {
    const char* xk = reinterpret_cast<const char*>(X + k * plane);
    if (hlds >= 0) hv = *reinterpret_cast<const V*>(xk + hoff);
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (!(ZM && zero[e])) load_to_lds(array(e, k + 1 + e), own, wave + e * BP * 16);
    load_to_lds(Fc + k * plane, own, wave + 3 * BP * 16);
  };
  if constexpr (ZM) {
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (zero[e]) lds[e * BP + tid] = V{};
    if (clear) {
      lds[hlds] = V{};
      hlds = -1;
    }
  }
  // w[e][d]: slot e, plane k - 3 + e + d
  V w[3][5];
#pragma unroll
  for (int e = 0; e < 3; ++e)
#pragma unroll
    for (int d = 0; d < 4; ++d)
      w[e][d] = ZM && zero[e] ? V{} : *reinterpret_cast<const V*>(array(e, k0 - 3 + e + d) + own);
  issue(k0);
  const T inv = (T)(1.0 / (3.0 * kC0));
  char* Xc = reinterpret_cast<char*>(X + (long long)c * G.cs);
  V out = V{};
  bool ok[CPL];
#pragma unroll
  for (int i = 0; i < CPL; ++i) ok[i] = false;
  auto store = [&](int k) {
    bool all = true;
#pragma unroll
    for (int i = 0; i < CPL; ++i) all = all && ok[i];
    T* dst = reinterpret_cast<T*>(Xc + k * plane * (long long)sizeof(T) + own);
    if (all) {
      __builtin_nontemporal_store(out, reinterpret_cast<V*>(dst));
    } else {
#pragma unroll
      for (int i = 0; i < CPL; ++i)
        if (ok[i]) __builtin_nontemporal_store(out[i], dst + i);
    }
  };
  V* c0 = lds + base0 + tid;
  V* c1 = lds + base1 + tid;
  V* c2 = lds + base2 + tid;
  for (int k = k0; k <= k1; ++k) {
    loads_done();
    w[0][4] = lds[tid];
    w[1][4] = lds[BP + tid];
    w[2][4] = lds[2 * BP + tid];
    const V fv = lds[3 * BP + tid];
    const V hk = hv;
    store(k - 1);  // nothing before the first plane: ok is false
    lds_read();    // the staged chunks are the lane's own: no other reads them
    if (k < k1) issue(k + 1);
    lds_barrier();  // the centre arrays' readers are done
    *c0 = w[0][3];
    *c1 = w[1][2];
    *c2 = w[2][1];
    if (hlds >= 0) lds[hlds] = hk;
    lds_barrier();
    const int q = (c - b - k - G.off) & 3;  // position of the colour-c node in its compact columns
    // the compact columns before and after the lane's own
    const T* x0 = reinterpret_cast<const T*>(c0);
    const T* x1 = reinterpret_cast<const T*>(c1);
    const T* x2 = reinterpret_cast<const T*>(c2);
    const T l0 = x0[-1], l1 = x1[-1], l2 = x2[-1], r0 = x0[CPL], r1 = x1[CPL], r2 = x2[CPL];
    V s1 = V{}, s2 = V{}, s3 = V{};
    // value of slot e at the lane's compact column j = -1 .. CPL
    auto col = [&](T l, const V& m, T r, int j) -> T { return j < 0 ? l : j >= CPL ? r : m[j]; };
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const T xp1 = q == 3 ? col(l0, w[0][3], r0, i + 1) : w[0][3][i];
      const T xm1 = q == 0 ? col(l2, w[2][1], r2, i - 1) : w[2][1][i];
      const T xp2 = q >= 2 ? col(l1, w[1][2], r1, i + 1) : w[1][2][i];
      const T xm2 = q <= 1 ? col(l1, w[1][2], r1, i - 1) : w[1][2][i];
      const T xp3 = q >= 1 ? col(l2, w[2][1], r2, i + 1) : w[2][1][i];
      const T xm3 = q <= 2 ? col(l0, w[0][3], r0, i - 1) : w[0][3][i];
      s1[i] = xp1 + xm1;
      s2[i] = xp2 + xm2;
      s3[i] = xp3 + xm3;
    }
    s1 = s1 + c0[ngr] + c2[-ngr] + w[0][4] + w[2][0];
    s2 = s2 + c1[2 * ngr] + c1[-2 * ngr] + w[1][4] + w[1][0];
    s3 = s3 + c2[3 * ngr] + c0[-3 * ngr] + w[2][4] + w[0][0];
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const T sum = (T)kC1 * s1[i] + (T)kC2 * s2[i] + (T)kC3 * s3[i];
      out[i] = (h2 * fv[i] - sum) * inv;
      ok[i] = live && G.inner(4 * (m0 + i) + q);
    }
#pragma unroll
    for (int e = 0; e < 3; ++e)
#pragma unroll
      for (int d = 0; d < 4; ++d) w[e][d] = w[e][d + 1];
  }
  store(k1);
}


// Lanes per block: the twelve halo rows take one chunk per lane (256 lanes up to
// 163 intervals in FP64 and 331 in FP32, 512 up to 331 and 667), the reason why
// wide levels want large blocks -- a second chunk per lane spills, and a spill
// waits for every load underway (FP64 at 511^3 with 512 lanes: 321-380 us
// against 297 with 1024).  0: too wide for any.
int lanes_for(int ngr) { return 12 * ngr <= 256 ? 256 : 12 * ngr <= 512 ? 512 : 12 * ngr <= 1024 ? 1024 : 0; }

// Runs along z.  Blocks of 512 and 1024 lanes are few and want one round over
// the chip's 256 compute units: FP64 at 255^3 39 us with 255 blocks, 46 with
// 374, 43 with 493; at 511^3 297 us with 231, 346 with 363, 305 with 495.
// Levels of 256-lane blocks are short of blocks, and runs of two planes do
// best: FP32 at 255^3 24 us with 2176 blocks, 26 with 493; FP64 at 127^3 8.0 us
// with 576, 9.3 with 288.
int runs_for(int bp, int nb, int E) {
  if (bp == 256) return (E + 1) / 2;
  const int most = std::max(1, std::min(E, 256 / nb));
  const int kz = (E + most - 1) / most;
  return (E + kz - 1) / kz;
}

template <typename T, int BP>
void pass_go(T* x, const T* f, const Geom& G, int c, int zmask, hipStream_t st) {
  const int ngr = groups<T>(G), E = G.n - 1;
  const int nb = (ngr * E + BP - 1) / BP;
  const dim3 grid(nb, 1, runs_for(BP, nb, E));
  const size_t lds = (size_t)(7 * BP + 12 * ngr) * 16;
  const T h2 = (T)(G.h * G.h);
  if (zmask)
    k_pass19w<T, BP, true><<<grid, BP, lds, st>>>(x, f, G, c, h2, zmask);
  else
    k_pass19w<T, BP, false><<<grid, BP, lds, st>>>(x, f, G, c, h2, 0);
}

template <typename T>
void pass_t(T* x, const T* f, const Geom& G, int c, int zmask, hipStream_t st) {
  switch (lanes_for(groups<T>(G))) {
    case 256: return pass_go<T, 256>(x, f, G, c, zmask, st);
    case 512: return pass_go<T, 512>(x, f, G, c, zmask, st);
    default: return pass_go<T, 1024>(x, f, G, c, zmask, st);
  }
}

template <typename T, int BP>
bool allow_lds() {
  const int most = (7 * BP + BP) * 16;  // 12 ngr <= BP
  return hipFuncSetAttribute((const void*)k_pass19w<T, BP, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             most) == hipSuccess &&
         hipFuncSetAttribute((const void*)k_pass19w<T, BP, true>, hipFuncAttributeMaxDynamicSharedMemorySize, most) ==
             hipSuccess;
}

}  // namespace

// From 96 intervals (below, the blocks' fixed costs show: FP64 at 95^3 4.9
// against 5.5 us, at 63^3 4.7 against 4.4), while the halo fits and a lane's
// byte offset into an array fits 32 bits.
bool pass19_ok(const Geom& G, bool f32) {
  const int ngr = f32 ? groups<float>(G) : groups<double>(G);
  return G.C == 4 && G.g == 3 && G.n >= 96 && lanes_for(ngr) != 0 &&
         (unsigned long long)G.total() * (f32 ? 4 : 8) < (1ull << 32);
}

void pass19(void* x, const void* f, bool f32, const Geom& G, int colour, int zmask, hipStream_t st) {
  if (f32)
    pass_t((float*)x, (const float*)f, G, colour, zmask, st);
  else
    pass_t((double*)x, (const double*)f, G, colour, zmask, st);
}

bool pass19_enable() {
  return allow_lds<float, 512>() && allow_lds<float, 1024>() && allow_lds<double, 512>() && allow_lds<double, 1024>();
}

}  // namespace psn
