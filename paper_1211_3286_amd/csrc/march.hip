// Two steps per pass on one D3Q19 lattice (temporal blocking, marching in z).
//
// One step at a time, a cell update moves 2 x 38 values of HBM traffic and runs
// at the memory's speed with the VALU at 0.37 busy. Here a block owns a column
// of OX x OY cells of a z range and takes each plane through two steps; the
// populations between them never leave the CU. Per plane zz it
//   1. collides the pulled populations of the WX x WY = (OX + 2) x (OY + 2)
//      window cells (first step; they were loaded a plane earlier) and
//      publishes them in LDS (two plane buffers, one barrier a plane),
//   2. pulls the second step's inputs of plane zz - 1, collides them and stores
//      the owned cells, while the loads of plane zz + 1 are in flight.
// Of the second step's inputs a cell of plane z takes the 10 populations with
// e_z = +1 from plane z - 1, the 18 with e_z = 0 from plane z and the 10 with
// e_z = -1 from plane z + 1: each published plane is read from LDS once, as
// soon as it is there, and what is not needed yet waits in registers.
//
// HBM traffic per two steps: the owned cells written once and the window rows
// read once (x halos hit in L2): 1.07 x 304 B in FP32 (256^3, FETCH_SIZE and
// WRITE_SIZE: 2.92 and 2.55 GB). What bounds it is memory as far as 2 waves per SIMD
// keep it busy: 4.5 TB/s (a copy of two streams 5.2 to 6.3) with the VALU issuing in
// 0.53 to 0.60 of the cycles; 8 % fewer instructions left the time as it was.
// Windows: FP32 34 x 15 (OX = 32 cells = one 128-byte line) on 512 threads; two
// 256-thread blocks of 18 x 14 per CU were slower (0.91 ms a step). FP64 18 x 14
// on 256 threads (one wave per SIMD, 512 registers; on 512 threads it spills);
// 34 x 7 was the same (1.31 ms). ms a step, before (best one-step kernel, plane
// layout) and now: 256^3 FP32 0.90 and 0.61, 512^3 FP32 7.41 and 4.65, 256^3
// FP64 1.85 and 1.28, 187 x 150 x 131 FP64 0.56 and 0.42.

#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_util.hpp"
#include "internal.hpp"

namespace rlb {

namespace {

// Coordinate of window position c on an axis of N cells: wrapped (periodic) or
// held at the face (zero gradient; the first step of the cell beyond a face is
// that of the face cell, which is what the second step pulls there).
__device__ __forceinline__ int on_axis(int c, int N, int bc) {
  if (bc) return min(max(c, 0), N - 1);
  c %= N;
  return c < 0 ? c + N : c;
}

// Byte offset of cell (x, y) within a z-plane of a blocked region (a plane is
// whole blocks).
template <typename T>
__device__ __forceinline__ uint32_t in_plane(int nx, int x, int y) {
  const uint32_t t = (uint32_t)y * (uint32_t)nx + (uint32_t)x;
  return (t + (t >> kBlockShift) * (18u * kBlock)) * (uint32_t)sizeof(T);
}

// Workgroup barrier for data exchanged through LDS only: global loads in
// flight (the next plane's) and stores stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// What the g half of a collision leaves for the f half.
struct Half {
  Macro mac;
  Rates rt;    // EXT: the cell's rates
  double fs;   // EXT: the sum of the stored f
  bool ok;
};

// The collision of a cell in two halves, so that one distribution's
// temporaries are in flight at a time. The arithmetic is that of collide(),
// bit for bit.
template <bool EXT, typename T>
__device__ __forceinline__ void g_half(const T (&f)[19], T (&g)[19], const LatticeGeom& geo,
                                       Half& h) {
  double E, Mx, My, Mz, gs;
  if constexpr (EXT) {  // the extended model recovers from N too
    h.fs = 0.0;
#pragma unroll
    for (int a = 0; a < 19; ++a) h.fs += (double)f[a];
    const double N = geo.ref.n + h.fs;
    g_sums(g, geo.ref, E, Mx, My, Mz, gs);
    h.ok = recover_model(N, E, Mx, My, Mz, geo.ext, h.mac);
    if (h.ok) {
      h.rt = local_rates<T>(geo.rt, geo.ext, N, h.mac);
      collide_g(g, Mx, My, Mz, gs, h.mac, h.rt, geo.ref);
    }
  } else {
    g_sums(g, geo.ref, E, Mx, My, Mz, gs);
    h.ok = recover(E, Mx, My, Mz, h.mac);
    if (h.ok) collide_g(g, Mx, My, Mz, gs, h.mac, geo.rt, geo.ref);
  }
}

template <bool EXT, typename T>
__device__ __forceinline__ void f_half(T (&f)[19], const LatticeGeom& geo, const Half& h) {
  if constexpr (EXT) {
    if (h.ok) collide_f(f, geo.ref.n + h.fs, h.fs, h.mac, h.rt, geo.ref);
  } else {
    double fs = 0.0;
#pragma unroll
    for (int a = 0; a < 19; ++a) fs += (double)f[a];
    if (h.ok) collide_f(f, geo.ref.n + fs, fs, h.mac, geo.rt, geo.ref);
  }
}

template <typename T, int WX, int WY, int NT, bool EXT, bool NTS>
__global__ __launch_bounds__(NT) void k_step_march(const T* __restrict__ src,
                                                   T* __restrict__ dst, LatticeGeom geo,
                                                   int ntx, int ntiles, int nchunks,
                                                   unsigned long long* __restrict__ bad) {
  constexpr int OX = WX - 2, OY = WY - 2;
  static_assert(WX * WY <= NT && 2 * 38 * NT * sizeof(T) <= 160 * 1024, "window and LDS");
  __shared__ T lds[2][38][NT];
  // Blocks go to the 8 XCDs in turn: XCD j takes one contiguous run of items,
  // so that the tiles that share lines and halos share its L2.
  const unsigned nb = gridDim.x, b = blockIdx.x;
  const unsigned xj = b & 7, xq = nb >> 3, xr = nb & 7;
  const unsigned item = xj * xq + (xj < xr ? xj : xr) + (b >> 3);
  const int tile = item % ntiles, chunk = item / ntiles;
  const int x0 = (tile % ntx) * OX, y0 = (tile / ntx) * OY;
  const int ow = min(OX, geo.nx - x0), oh = min(OY, geo.ny - y0);
  const int z0 = (int)((int64_t)geo.nz * chunk / nchunks);
  const int z1 = (int)((int64_t)geo.nz * (chunk + 1) / nchunks);
  const int tid = threadIdx.x;
  const int64_t zel = (int64_t)geo.lay.zcells * 19;  // elements of a z-plane (whole blocks)

  // First step: window cell of this thread and its in-plane pull offsets. A
  // thread without one (past the window, or of a tile cut by the lattice's
  // end) computes some cell of the lattice that nobody reads.
  const int wi = tid % WX, wj = tid / WX;
  const bool own1 = wi >= 1 && wi <= ow && wj >= 1 && wj <= oh;
  uint32_t oxy[3][3];  // [y - 1, y, y + 1][x - 1, x, x + 1]
  {
    const int X = on_axis(x0 - 1 + wi, geo.nx, geo.bcx);
    const int Y = on_axis(y0 - 1 + wj, geo.ny, geo.bcy);
    const int xs[3] = {nbr(X, -1, geo.nx, geo.bcx), X, nbr(X, 1, geo.nx, geo.bcx)};
    const int ys[3] = {nbr(Y, -1, geo.ny, geo.bcy), Y, nbr(Y, 1, geo.ny, geo.bcy)};
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int i = 0; i < 3; ++i) oxy[j][i] = in_plane<T>(geo.nx, xs[i], ys[j]);
  }
  // second step: owned cell of this thread, dealt row by row
  const int i2 = tid % OX, j2 = tid / OX;
  const bool act2 = tid < OX * OY && i2 < ow && j2 < oh;
  const int s2 = act2 ? (j2 + 1) * WX + i2 + 1 : WX + 1;
  const uint32_t self = act2 ? in_plane<T>(geo.nx, x0 + i2, y0 + j2) : 0u;

  T f1[19], g1[19];  // first step: pulled populations of the plane in hand
  T f2[19] = {}, g2[19] = {};  // second step: inputs gathered so far
  T uf[5] = {}, ug[5] = {};    // populations with e_z = +1 of the last plane
  int nbad = 0;

  // Pulled populations of one distribution's region of plane zz: three scalar
  // plane pointers, nine lane offsets, the population as an instruction constant.
  auto load = [&](int zz, const T* region, T (&v)[19]) {
    const int Z = nbr(zz, 0, geo.nz, geo.bcz);
    const int zs[3] = {nbr(Z, -1, geo.nz, geo.bcz), Z, nbr(Z, 1, geo.nz, geo.bcz)};
    GPtr<const T> p[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) p[d] = to_global(region + zs[d] * zel);
#pragma unroll
    for (int a = 0; a < 19; ++a)
      v[a] = at_off<T>(p[1 - ez(a)] + a * kBlock, oxy[1 - ey(a)][1 - ex(a)]);
  };
  auto store = [&](int z, T* region, const T (&v)[19]) {
    GPtr<T> p = to_global(region + z * zel);
#pragma unroll
    for (int a = 0; a < 19; ++a) put_off<NTS>(p + a * kBlock, self, v[a]);
  };
  const T* const src_g = src + geo.lay.greg;
  T* const dst_g = dst + geo.lay.greg;

  load(z0 - 1, src_g, g1);
  load(z0 - 1, src, f1);
  int buf = 0;
#pragma unroll 1
  for (int zz = z0 - 1; zz <= z1; ++zz) {
    Half h;
    g_half<EXT>(f1, g1, geo, h);
#pragma unroll
    for (int a = 0; a < 19; ++a) lds[buf][19 + a][tid] = g1[a];
    __builtin_amdgcn_sched_barrier(0);
    f_half<EXT>(f1, geo, h);
#pragma unroll
    for (int a = 0; a < 19; ++a) lds[buf][a][tid] = f1[a];
    if (own1 && zz >= z0 && zz < z1) nbad += h.ok ? 0 : 1;
    // g of the next plane is loaded from here on, f between the halves of the
    // second step: all 38 at once, or later, measured 3-10 % slower
    if (zz < z1) load(zz + 1, src_g, g1);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    const bool out2 = act2 && zz > z0;
    if (out2) {
#pragma unroll
      for (int a = 0; a < 19; ++a)
        if (ez(a) < 0) {
          f2[a] = lds[buf][a][s2 - ey(a) * WX - ex(a)];
          g2[a] = lds[buf][19 + a][s2 - ey(a) * WX - ex(a)];
        }
      g_half<EXT>(f2, g2, geo, h);
      __builtin_amdgcn_sched_barrier(0);
      store(zz - 1, dst_g, g2);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (zz < z1) load(zz + 1, src, f1);
    __builtin_amdgcn_sched_barrier(0);
    if (out2) {
      f_half<EXT>(f2, geo, h);
      nbad += h.ok ? 0 : 1;
    }
    // The loads of plane zz + 1 are waited for here, ahead of the f stores: the
    // memory counter retires in order, and a wait behind those stores would be
    // one for them too.
    landed(g1);
    landed(f1);
    if (out2) store(zz - 1, dst, f2);
    if (act2) {
      int k = 0;
#pragma unroll
      for (int a = 0; a < 19; ++a) {
        if (ez(a) == 0) {
          f2[a] = lds[buf][a][s2 - ey(a) * WX - ex(a)];
          g2[a] = lds[buf][19 + a][s2 - ey(a) * WX - ex(a)];
        }
        if (ez(a) > 0) {
          f2[a] = uf[k];
          g2[a] = ug[k];
          uf[k] = lds[buf][a][s2 - ey(a) * WX - ex(a)];
          ug[k] = lds[buf][19 + a][s2 - ey(a) * WX - ex(a)];
          ++k;
        }
      }
    }
    buf ^= 1;
  }
  if (nbad) count_bad(bad, nbad);
}

// Window (of each precision) and threads of a block.
template <typename T>
struct Window;
template <>
struct Window<float> {
  static constexpr int wx = 34, wy = 15, nt = 512;
};
template <>
struct Window<double> {
  static constexpr int wx = 18, wy = 14, nt = 256;
};

// Tiles of the lattice and number of z ranges. The blocks of a launch run one
// per CU, and each adds two planes of first-step work (about 1.2 planes' time)
// to its range.
template <typename T>
MarchGrid grid_of(const LatticeGeom& g, int cus) {
  constexpr int OX = Window<T>::wx - 2, OY = Window<T>::wy - 2;
  MarchGrid m{};
  m.ntx = (g.nx + OX - 1) / OX;
  m.ntiles = m.ntx * ((g.ny + OY - 1) / OY);
  const int per_xcd = std::max(1, cus / 8);
  double least = 1e300;
  for (int c = 1; c <= std::max(1, g.nz / 4); ++c) {
    const int64_t rounds = (((int64_t)m.ntiles * c + 7) / 8 + per_xcd - 1) / per_xcd;
    const double cost = rounds * ((g.nz + c - 1) / c + 1.2);
    if (cost < least * 0.999) {
      least = cost;
      m.nchunks = c;
    }
  }
  m.use = (double)g.nx * g.ny * g.nz / (least * cus * OX * OY);
  return m;
}

template <typename T, bool EXT>
hipError_t march_launch(const void* src, void* dst, const LatticeGeom& g, const MarchGrid& m,
                        unsigned long long* bad, hipStream_t s) {
  constexpr int WX = Window<T>::wx, WY = Window<T>::wy, NT = Window<T>::nt;
  const dim3 grid((unsigned)((int64_t)m.ntiles * m.nchunks)), block(NT);
  if (g.cached_store)
    hipLaunchKernelGGL((k_step_march<T, WX, WY, NT, EXT, false>), grid, block, 0, s,
                       (const T*)src, (T*)dst, g, m.ntx, m.ntiles, m.nchunks, bad);
  else
    hipLaunchKernelGGL((k_step_march<T, WX, WY, NT, EXT, true>), grid, block, 0, s,
                       (const T*)src, (T*)dst, g, m.ntx, m.ntiles, m.nchunks, bad);
  return hipGetLastError();
}

constexpr int kNumMarch = 1;

}  // namespace

int num_march_variants() { return kNumMarch; }

MarchGrid march_grid(int precision, const LatticeGeom& g, int cus) {
  return precision ? grid_of<float>(g, cus) : grid_of<double>(g, cus);
}

const char* march_kernel_name(int precision, int) {
  return precision ? "k_step_march<float,34,15>/h2" : "k_step_march<double,18,14>/h2";
}

hipError_t launch_step_march(int precision, int variant, bool ext, const void* src, void* dst,
                             const LatticeGeom& g, const MarchGrid& m, unsigned long long* bad,
                             hipStream_t s) {
  if (variant < 0 || variant >= kNumMarch || g.lay.shift != kBlockShift)
    return hipErrorInvalidValue;
  if (precision)
    return ext ? march_launch<float, true>(src, dst, g, m, bad, s)
               : march_launch<float, false>(src, dst, g, m, bad, s);
  return ext ? march_launch<double, true>(src, dst, g, m, bad, s)
             : march_launch<double, false>(src, dst, g, m, bad, s);
}

}  // namespace rlb
