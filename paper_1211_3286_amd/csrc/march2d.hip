// H steps per pass on one D2Q9 lattice (temporal blocking, marching in y).
//
// A wave owns a strip of 64 - 2 (H - 1) columns of a y range and takes each row
// through H steps as a pipeline: stage s works on row r - (s - 1) of iteration
// r. Of a stage's inputs a cell of row y takes the populations with e_y = +1
// from row y - 1 of the stage before, those with e_y = 0 from row y and those
// with e_y = -1 from row y + 1; they wait in registers, shifted to their x
// neighbour by DPP, so that no population between the first and the last step
// leaves the wave: no LDS, no barrier, and every wave runs on its own. Halo
// work is 2 (H - 1) columns in 64 and H - 1 rows a side of the range.
//
// It replaces the tiles in LDS (k_d2q9_tiles: 16 % halo cells, index arithmetic
// per cell, VALU-bound in FP32, two windows a CU in FP64) as the default on
// large lattices. Bound now: FP32 H = 4 moves 39 B per cell update at 0.195 ms
// per 4096^2 step, 3.4 TB/s, with 2 waves per SIMD (178 registers); H = 3 and 6
// take 0.245 and 0.195 ms, FP64 H = 3, 4, 6 0.403, 0.299 and 0.293. us a step,
// best tile and now (H = 4): 4096^2 FP32 265 and 195, FP64 503 and 299; 2048^2
// FP64 120 and 72; 1531 x 1203 FP32 31 and 26, FP64 52 and 35.

#include <hip/hip_runtime.h>

#include <algorithm>

#include "cell2d.hpp"
#include "device_util.hpp"
#include "internal.hpp"

namespace rlb {

namespace {

constexpr int kWaves = 4;  // strips (waves) per block, side by side

// The value of the lane below (wave_shr:1) or above (wave_shl:1); the first
// or last lane keeps its own, which is the zero-gradient rule where the
// window begins or ends at a face.
template <int CTRL>
__device__ __forceinline__ int lane_shift(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v) {
  return __int_as_float(lane_shift<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = lane_shift<CTRL>((int)b), hi = lane_shift<CTRL>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// A population with velocity component e_x at its pull source x - e_x.
template <typename T>
__device__ __forceinline__ T shift_in(int ex, T v) {
  return ex > 0 ? lane_shift<0x138>(v) : ex < 0 ? lane_shift<0x130>(v) : v;
}

// What a stage leaves for the next: populations with e_y = +1 of the last two
// rows, e_y = 0 and e_y = -1 of the last one, at their x sources (3 f, 3 g).
template <typename T>
struct Between {
  T up_old[6], up[6], mid[6], down[6];
};

template <typename T, int H, bool EXT>
__global__ __launch_bounds__(64 * kWaves) void k_d2q9_march(const T* __restrict__ src,
                                                            T* __restrict__ dst, LatticeGeom geo,
                                                            int nstrips, int nbx, int nchunks,
                                                            unsigned long long* __restrict__ bad) {
  constexpr int HALO = H - 1, OWN = 64 - 2 * HALO;
  // XCD j takes one contiguous run of items, x fastest: neighbouring strips
  // share the lines at their edges in its L2.
  const unsigned nb = gridDim.x, b = blockIdx.x;
  const unsigned xj = b & 7, xq = nb >> 3, xr = nb & 7;
  const unsigned item = xj * xq + (xj < xr ? xj : xr) + (b >> 3);
  const int strip = (int)(item % nbx) * kWaves +
                    __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int chunk = (int)(item / nbx);
  if (strip >= nstrips) return;
  const int lane = threadIdx.x & 63;
  const int nx = geo.nx, ny = geo.ny;
  // Columns: a periodic strip has HALO columns a side; between faces the first
  // and last windows begin and end at the face (nx >= 64 there).
  const int own0 = strip * OWN, own1 = min(nx, own0 + OWN);
  int wx = own0 - HALO;
  if (geo.bcx) wx = min(max(wx, 0), nx - 64);
  int x = wx + lane;
  const bool mine = x >= own0 && x < own1;
  if (!geo.bcx) {
    x %= nx;
    if (x < 0) x += nx;
  }
  const uint32_t esz = sizeof(T);
  const uint32_t xs[3] = {(uint32_t)nbr(x, -1, nx, geo.bcx) * esz, (uint32_t)x * esz,
                          (uint32_t)nbr(x, 1, nx, geo.bcx) * esz};
  // Rows: stage s computes [y0 - (H - s), y1 + (H - s)), cut at faces.
  const int y0 = (int)((int64_t)ny * chunk / nchunks);
  const int y1 = (int)((int64_t)ny * (chunk + 1) / nchunks);
  const int ylo = geo.bcy ? 0 : -H, yhi = geo.bcy ? ny - 1 : ny - 1 + H;
  const int first = max(y0 - HALO, ylo), last = min(y1 - 1 + HALO, yhi);

  auto load = [&](int r, T (&f)[9], T (&g)[9]) {
    const int Y = r < 0 ? r + ny : r >= ny ? r - ny : r;  // only beyond a periodic end
    const int ys[3] = {nbr(Y, -1, ny, geo.bcy), Y, nbr(Y, 1, ny, geo.bcy)};
#pragma unroll
    for (int d = -1; d <= 1; ++d) {
      GPtr<const T> p = to_global(src + (int64_t)ys[1 - d] * nx);
      int at = 0;
#pragma unroll
      for (int a = 0; a < 18; ++a)
        if (d2q9::ey(a % 9) == d) {
          advance(p, (a - at) * geo.cs);
          at = a;
          const T v = at_off<T>(p, xs[1 - d2q9::ex(a % 9)]);
          (a < 9 ? f[a % 9] : g[a % 9]) = v;
        }
    }
  };

  T nf[9], ng[9];  // the row being loaded
  Between<T> st[H - 1] = {};
  int nbad = 0;
  load(first, nf, ng);
#pragma unroll 1
  for (int r = first; r <= y1 - 1 + HALO; ++r) {
    T f[9], g[9];
#pragma unroll
    for (int a = 0; a < 9; ++a) {
      f[a] = nf[a];
      g[a] = ng[a];
    }
    if (r < last) load(r + 1, nf, ng);
#pragma unroll
    for (int s = 1; s <= H; ++s) {
      const int y = r - (s - 1);  // this stage's row
      const bool on = y >= max(y0 - (H - s), ylo) && y <= min(y1 - 1 + (H - s), yhi);
      if (on) {
        Sums sums;
        const bool ok = d2q9::collide<T, false, EXT>(f, g, geo.rt, geo.ref, sums, nullptr,
                                                     nullptr, &geo.ext);
        if (mine && y >= y0 && y < y1) nbad += ok ? 0 : 1;
      }
      if (s < H) {
        // Hand the row on: with its e_y = -1 the next stage completes row y - 1.
        Between<T>& w = st[s - 1];
        T up[6], mid[6];
        if (on) {
          int ku = 0, km = 0, kd = 0;
#pragma unroll
          for (int a = 0; a < 18; ++a) {
            const T v = shift_in(d2q9::ex(a % 9), a < 9 ? f[a % 9] : g[a % 9]);
            if (d2q9::ey(a % 9) > 0)
              up[ku++] = v;
            else if (d2q9::ey(a % 9) == 0)
              mid[km++] = v;
            else
              w.down[kd++] = v;
          }
        }
        int ku = 0, km = 0, kd = 0;
#pragma unroll
        for (int a = 0; a < 18; ++a)
          (a < 9 ? f[a % 9] : g[a % 9]) = d2q9::ey(a % 9) > 0    ? w.up_old[ku++]
                                          : d2q9::ey(a % 9) == 0 ? w.mid[km++]
                                                                 : w.down[kd++];
        if (on) {
          const bool face = geo.bcy && y == 0;  // row 0 stands for the row below it
#pragma unroll
          for (int k = 0; k < 6; ++k) {
            w.up_old[k] = face ? up[k] : w.up[k];
            w.up[k] = up[k];
            w.mid[k] = mid[k];
          }
        }
      } else if (on) {
        // The next row's loads are waited for ahead of the stores: the memory
        // counter retires in order.
        landed(nf);
        landed(ng);
        if (mine) {
          GPtr<T> p = to_global(dst + (int64_t)y * nx);
#pragma unroll
          for (int a = 0; a < 18; ++a) {
            if (a > 0) advance(p, geo.cs);
            put_off<false>(p, xs[1], a < 9 ? f[a % 9] : g[a % 9]);
          }
        }
      }
    }
  }
  if (nbad) count_bad(bad, nbad);
}

// Blocks of a kernel that a CU holds at a time (a property of the built kernel).
template <typename T, int H, bool EXT>
int blocks_per_cu() {
  static const int n = [] {
    int v = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &v, (const void*)&k_d2q9_march<T, H, EXT>, 64 * kWaves, 0);
    return e == hipSuccess && v > 0 ? v : 1;
  }();
  return n;
}

// Strips, blocks along x and number of y ranges: as many as let the blocks of a
// launch end together (k rounds of all slots), each range costing H + 1 rows
// more than it owns (the halo rows of the early stages and the pipeline's start).
struct Plan {
  int nstrips, nbx, nchunks;
  double use;  // share of the launch's cell slots that are cells of the lattice
};

Plan plan_of(const LatticeGeom& g, int h, int64_t slots) {
  const int own = 64 - 2 * (h - 1);
  Plan p{};
  p.nstrips = (g.nx + own - 1) / own;
  p.nbx = (p.nstrips + kWaves - 1) / kWaves;
  double least = 1e300;
  for (int k = 1; k <= 6; ++k) {
    const int c = (int)std::max<int64_t>(1, std::min<int64_t>(k * slots / p.nbx, g.ny / 4));
    const int64_t rounds = ((int64_t)p.nbx * c + slots - 1) / slots;
    const double cost = rounds * ((g.ny + c - 1) / c + h + 1.0);
    if (cost < least * 0.999) {
      least = cost;
      p.nchunks = c;
    }
  }
  p.use = (double)g.nx * g.ny / (least * slots * kWaves * own);
  return p;
}

template <typename T, int H, bool EXT>
Plan plan(const LatticeGeom& g, int cus) {
  return plan_of(g, H, (int64_t)cus * blocks_per_cu<T, H, EXT>());
}

template <typename T, int H, bool EXT>
hipError_t launch(const void* src, void* dst, const LatticeGeom& g, int cus,
                  unsigned long long* bad, hipStream_t s) {
  const Plan p = plan<T, H, EXT>(g, cus);
  hipLaunchKernelGGL((k_d2q9_march<T, H, EXT>), dim3((unsigned)(p.nbx * p.nchunks)),
                     dim3(64 * kWaves), 0, s, (const T*)src, (T*)dst, g, p.nstrips, p.nbx,
                     p.nchunks, bad);
  return hipGetLastError();
}

template <typename T, int H>
hipError_t launch_ext(bool ext, const void* src, void* dst, const LatticeGeom& g, int cus,
                      unsigned long long* bad, hipStream_t s) {
  return ext ? launch<T, H, true>(src, dst, g, cus, bad, s)
             : launch<T, H, false>(src, dst, g, cus, bad, s);
}

template <typename T>
hipError_t dispatch(int h, bool ext, const void* src, void* dst, const LatticeGeom& g, int cus,
                    unsigned long long* bad, hipStream_t s) {
  switch (h) {
    case 3: return launch_ext<T, 3>(ext, src, dst, g, cus, bad, s);
    case 4: return launch_ext<T, 4>(ext, src, dst, g, cus, bad, s);
  }
  return hipErrorInvalidValue;
}

constexpr int kSteps[] = {4, 3};
constexpr int kNum = sizeof(kSteps) / sizeof(kSteps[0]);

}  // namespace

int d2q9_num_march_variants() { return kNum; }
int d2q9_march_steps(int v) { return kSteps[v]; }

double d2q9_march_use(int precision, bool ext, const LatticeGeom& g, int cus) {
  constexpr int H = kSteps[0];
  if (precision) return (ext ? plan<float, H, true>(g, cus) : plan<float, H, false>(g, cus)).use;
  return (ext ? plan<double, H, true>(g, cus) : plan<double, H, false>(g, cus)).use;
}

bool d2q9_march_fits(const LatticeGeom& g) { return g.ny >= 8 && (!g.bcx || g.nx >= 64); }

const char* d2q9_march_kernel_name(int precision, int v) {
  static const char* n[2][kNum] = {{"k_d2q9_march<double>/h4", "k_d2q9_march<double>/h3"},
                                   {"k_d2q9_march<float>/h4", "k_d2q9_march<float>/h3"}};
  return v < 0 || v >= kNum ? "?" : n[precision ? 1 : 0][v];
}

hipError_t d2q9_launch_march(int precision, int v, bool ext, const void* src, void* dst,
                             const LatticeGeom& g, int cus, unsigned long long* bad,
                             hipStream_t s) {
  if (v < 0 || v >= kNum || !d2q9_march_fits(g)) return hipErrorInvalidValue;
  return precision ? dispatch<float>(kSteps[v], ext, src, dst, g, cus, bad, s)
                   : dispatch<double>(kSteps[v], ext, src, dst, g, cus, bad, s);
}

}  // namespace rlb
