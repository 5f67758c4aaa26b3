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
// per 4096^2 step, 3.4 TB/s, with the VALU issuing in 0.9 of the cycles of 2 waves
// per SIMD (178 registers); H = 3 and 6 take 0.245 and 0.195 ms, FP64 (76 B, a wave
// per SIMD, 0.5) H = 3, 4, 6 0.403, 0.299 and 0.293. us a step, best tile and now (H
// = 4), one card: 4096^2 FP32 265 and 195, FP64 503 and 299 (217 and 348 on the
// slowest); 2048^2 FP64 120 and 72; 1531 x 1203 FP32 31 and 26, FP64 52 and 35.
//
// With the correction of Eqs. (37)-(38) a stage recovers a row as it arrives and
// collides it one row later, between the fields of its neighbours: one recovery
// per cell, two rows of lag per stage, H = 2 (250 registers in FP32, a wave per
// SIMD in FP64). us a step, best one-step kernel and now: 4096^2 FP32 420 and
// 347, FP64 831 and 557; 1531 x 1203 FP64 125 and 68.

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

// With the correction a stage collides a row once the fields of the next are
// known: the row it holds meanwhile, and the fields of that row and the last.
// (Plain scalars, copied one by one: copies of the structs themselves would keep
// the array in memory. What a few operations give again is not held: N, u^2, P
// and three of the own fields come back by the expressions they came from.)
template <typename T>
struct Held {
  T f[9], g[9];
  double fs, gs, Mx, My, ux, uy, sigma, gam;  // this row
  double b_x1, b_gam, b_su2, b_su;            // fields of the row below
  int ok, b_ok;

  __device__ __forceinline__ d2q9::Recovered rec(const Ref& ref) const {
    d2q9::Recovered r;
    r.N = ref.n + fs;
    r.E = 0.0;  // only for the sums, which no marching launch leaves
    r.Mx = Mx;
    r.My = My;
    r.fs = fs;
    r.gs = gs;
    r.mac.ux = ux;
    r.mac.uy = uy;
    r.mac.uz = 0.0;
    r.mac.u2 = r.mac.ux * r.mac.ux + r.mac.uy * r.mac.uy;
    r.mac.sigma = sigma;
    r.mac.P = 0.25 * r.mac.sigma * (1.0 - r.mac.u2);
    r.ok = ok != 0;
    return r;
  }
  __device__ __forceinline__ d2q9::C7Fields fields(const d2q9::Recovered& r) const {
    d2q9::C7Fields F;
    F.x1 = r.mac.sigma * (1.0 / 3.0) - r.mac.P;
    F.gam = gam;
    F.su = r.mac.sigma * r.mac.uy;
    F.su2 = F.su * r.mac.uy;
    F.ok = r.ok;
    return F;
  }
  __device__ __forceinline__ d2q9::C7Fields below() const {
    return d2q9::C7Fields{b_x1, b_gam, b_su2, b_su, b_ok != 0};
  }
  __device__ __forceinline__ void set_below(const d2q9::C7Fields& F) {
    b_x1 = F.x1;
    b_gam = F.gam;
    b_su2 = F.su2;
    b_su = F.su;
    b_ok = F.ok ? 1 : 0;
  }
  __device__ __forceinline__ void set(const T (&nf)[9], const T (&ng)[9],
                                      const d2q9::Recovered& r, double g_am) {
    fs = r.fs;
    gs = r.gs;
    Mx = r.Mx;
    My = r.My;
    ux = r.mac.ux;
    uy = r.mac.uy;
    sigma = r.mac.sigma;
    gam = g_am;
    ok = r.ok ? 1 : 0;
#pragma unroll
    for (int a = 0; a < 9; ++a) {
      f[a] = nf[a];
      g[a] = ng[a];
    }
  }
};

template <typename T, int H, bool CORR, bool EXT>
__global__ __launch_bounds__(64 * kWaves) void k_d2q9_march(const T* __restrict__ src,
                                                            T* __restrict__ dst, LatticeGeom geo,
                                                            int nstrips, int nbx, int nchunks,
                                                            unsigned long long* __restrict__ bad) {
  constexpr int HALO = H - 1, OWN = 64 - 2 * HALO;
  constexpr int LAG = CORR ? 2 : 1;  // rows a stage is behind the one before
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
  // Rows: stage s computes [y0 - LAG (H - s), y1 + LAG (H - s)) (with the
  // correction it recovers one more a side), cut at faces.
  const int y0 = (int)((int64_t)ny * chunk / nchunks);
  const int y1 = (int)((int64_t)ny * (chunk + 1) / nchunks);
  const int ylo = geo.bcy ? 0 : -2 * H, yhi = geo.bcy ? ny - 1 : ny - 1 + 2 * H;
  const int reach = LAG * HALO + (CORR ? 1 : 0);
  const int first = max(y0 - reach, ylo), last = min(y1 - 1 + reach, yhi);

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
  Held<T> held[CORR ? H : 1] = {};
  int nbad = 0;
  load(first, nf, ng);
#pragma unroll 1
  for (int r = first; r <= y1 - 1 + reach; ++r) {
    T f[9], g[9];  // pulled populations of row r - LAG (s - 1)
#pragma unroll
    for (int a = 0; a < 9; ++a) {
      f[a] = nf[a];
      g[a] = ng[a];
    }
    if (r < last) load(r + 1, nf, ng);
#pragma unroll
    for (int s = 1; s <= H; ++s) {
      const int side = LAG * (H - s);
      const int y = r - LAG * s + 1;  // the row this stage collides
      const bool on = y >= max(y0 - side, ylo) && y <= min(y1 - 1 + side, yhi);
      T of[9], og[9];  // its result
      if constexpr (CORR) {
        Held<T>& h = held[s - 1];
        const int q = y + 1;
        const bool fresh = q >= max(y0 - side - 1, ylo) && q <= min(y1 + side, yhi);
        const d2q9::Recovered hrec = h.rec(geo.ref);
        const d2q9::C7Fields own = h.fields(hrec);
        d2q9::Recovered rec;
        d2q9::C7Fields above = own;  // at the upper face the row stands for the next
        if (fresh) {
          rec = d2q9::recovered<T, EXT>(f, g, geo.ref, &geo.ext);
          above = d2q9::c7_fields(rec.mac, rec.ok);
        }
#pragma unroll
        for (int a = 0; a < 9; ++a) {
          of[a] = h.f[a];
          og[a] = h.g[a];
        }
        if (on) {
          Sums sums;
          const d2q9::C7Fields below = h.below();
          const bool ok = d2q9::collide_recovered<T, true, EXT>(
              of, og, hrec, geo.rt, geo.ref, sums, &below, &above, &geo.ext);
          if (mine && y >= y0 && y < y1) nbad += ok ? 0 : 1;
        }
        if (fresh) {
          h.set_below(geo.bcy && q == 0 ? above : own);
          h.set(f, g, rec, above.gam);
        }
      } else {
        if (on) {
          Sums sums;
          const bool ok = d2q9::collide<T, false, EXT>(f, g, geo.rt, geo.ref, sums, nullptr,
                                                       nullptr, &geo.ext);
          if (mine && y >= y0 && y < y1) nbad += ok ? 0 : 1;
        }
#pragma unroll
        for (int a = 0; a < 9; ++a) {
          of[a] = f[a];
          og[a] = g[a];
        }
      }
      if (s < H) {
        // Hand the row on: with its e_y = -1 the next stage completes row y - 1.
        Between<T>& w = st[s - 1];
        T up[6], mid[6];
        if (on) {
          int ku = 0, km = 0, kd = 0;
#pragma unroll
          for (int a = 0; a < 18; ++a) {
            const T v = shift_in(d2q9::ex(a % 9), a < 9 ? of[a % 9] : og[a % 9]);
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
            put_off<false>(p, xs[1], a < 9 ? of[a % 9] : og[a % 9]);
          }
        }
      }
    }
  }
  if (nbad) count_bad(bad, nbad);
}

// Blocks of a kernel that a CU holds at a time (a property of the built kernel).
template <typename T, int H, bool CORR, bool EXT>
int blocks_per_cu() {
  static const int n = [] {
    int v = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &v, (const void*)&k_d2q9_march<T, H, CORR, EXT>, 64 * kWaves, 0);
    return e == hipSuccess && v > 0 ? v : 1;
  }();
  return n;
}

// Strips, blocks along x and number of y ranges: as many as let the blocks of a
// launch end together (k rounds of all slots), each range costing
// more rows than it owns (the halo rows of the early stages and the pipeline's
// start).
struct Plan {
  int nstrips, nbx, nchunks;
  double use;  // share of the launch's cell slots that are cells of the lattice
};

Plan plan_of(const LatticeGeom& g, int h, int more, int64_t slots) {
  const int own = 64 - 2 * (h - 1);
  Plan p{};
  p.nstrips = (g.nx + own - 1) / own;
  p.nbx = (p.nstrips + kWaves - 1) / kWaves;
  double least = 1e300;
  for (int k = 1; k <= 6; ++k) {
    const int c = (int)std::max<int64_t>(1, std::min<int64_t>(k * slots / p.nbx, g.ny / 4));
    const int64_t rounds = ((int64_t)p.nbx * c + slots - 1) / slots;
    const double cost = rounds * ((g.ny + c - 1) / c + more);
    if (cost < least * 0.999) {
      least = cost;
      p.nchunks = c;
    }
  }
  p.use = (double)g.nx * g.ny / (least * slots * kWaves * own);
  return p;
}

template <typename T, int H, bool CORR, bool EXT>
Plan plan(const LatticeGeom& g, int cus) {
  return plan_of(g, H, CORR ? 2 * H : H + 1, (int64_t)cus * blocks_per_cu<T, H, CORR, EXT>());
}

template <typename T, int H, bool CORR, bool EXT>
hipError_t launch(const void* src, void* dst, const LatticeGeom& g, int cus,
                  unsigned long long* bad, hipStream_t s) {
  const Plan p = plan<T, H, CORR, EXT>(g, cus);
  hipLaunchKernelGGL((k_d2q9_march<T, H, CORR, EXT>), dim3((unsigned)(p.nbx * p.nchunks)),
                     dim3(64 * kWaves), 0, s, (const T*)src, (T*)dst, g, p.nstrips, p.nbx,
                     p.nchunks, bad);
  return hipGetLastError();
}

// Steps of the variants. With the correction 3 steps need a wave per SIMD to
// itself and lose to 2 (4096^2 FP32 0.49 against 0.35 ms).
constexpr int num_of(bool corr) { return corr ? 1 : 2; }
constexpr int steps_of(bool corr, int v) { return corr ? 2 : v == 0 ? 4 : 3; }

// fn.run<T, H, CORR, EXT>() of a form.
template <typename T, bool CORR, bool EXT, typename F>
auto with_form(int v, F fn) {
  if (v == 0) return fn.template run<T, steps_of(CORR, 0), CORR, EXT>();
  return fn.template run<T, steps_of(CORR, num_of(CORR) - 1), CORR, EXT>();
}

template <typename T, bool CORR, typename F>
auto with_form(int v, bool ext, F fn) {
  return ext ? with_form<T, CORR, true>(v, fn) : with_form<T, CORR, false>(v, fn);
}

template <typename F>
auto with_form(int precision, int v, bool corr, bool ext, F fn) {
  if (precision)
    return corr ? with_form<float, true>(v, ext, fn) : with_form<float, false>(v, ext, fn);
  return corr ? with_form<double, true>(v, ext, fn) : with_form<double, false>(v, ext, fn);
}

struct Launch {
  const void* src;
  void* dst;
  const LatticeGeom& g;
  int cus;
  unsigned long long* bad;
  hipStream_t s;
  template <typename T, int H, bool CORR, bool EXT>
  hipError_t run() const {
    return launch<T, H, CORR, EXT>(src, dst, g, cus, bad, s);
  }
};

struct Use {
  const LatticeGeom& g;
  int cus;
  template <typename T, int H, bool CORR, bool EXT>
  double run() const {
    return plan<T, H, CORR, EXT>(g, cus).use;
  }
};

}  // namespace

int d2q9_num_march_variants(bool corr) { return num_of(corr); }
int d2q9_march_steps(int v, bool corr) { return steps_of(corr, v); }

double d2q9_march_use(int precision, int v, bool corr, bool ext, const LatticeGeom& g, int cus) {
  return with_form(precision, v, corr, ext, Use{g, cus});
}

bool d2q9_march_fits(const LatticeGeom& g) { return g.ny >= 8 && (!g.bcx || g.nx >= 64); }

const char* d2q9_march_kernel_name(int precision, int v, bool corr) {
  static const char* n[2][3] = {
      {"k_d2q9_march<double>/h2", "k_d2q9_march<double>/h3", "k_d2q9_march<double>/h4"},
      {"k_d2q9_march<float>/h2", "k_d2q9_march<float>/h3", "k_d2q9_march<float>/h4"}};
  return v < 0 || v >= num_of(corr) ? "?" : n[precision ? 1 : 0][steps_of(corr, v) - 2];
}

hipError_t d2q9_launch_march(int precision, int v, bool corr, bool ext, const void* src, void* dst,
                             const LatticeGeom& g, int cus, unsigned long long* bad,
                             hipStream_t s) {
  if (v < 0 || v >= num_of(corr) || !d2q9_march_fits(g)) return hipErrorInvalidValue;
  return with_form(precision, v, corr, ext, Launch{src, dst, g, cus, bad, s});
}

}  // namespace rlb
