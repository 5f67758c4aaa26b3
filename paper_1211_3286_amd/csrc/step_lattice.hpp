// The fused one-step kernel of a D3Q19 lattice and its launch, for both layouts
// of the populations (StateLayout): planes in kernels.hip, blocks in blocks.hip.
#pragma once

#include <hip/hip_runtime.h>

#include "device_util.hpp"
#include "internal.hpp"

namespace rlb {
namespace {

// Pull sources of a cell, by layout. Cells of a wave share their row (y, z).
template <typename T, bool BLOCKS>
struct Pull;

// Blocks: see StateLayout. A block may straddle rows, hence the phase of a
// row's first cell in its block; the population is an instruction constant.
template <typename T>
struct Pull<T, true> {
  int64_t row[3][3];  // element of the block of [z - 1, z, z + 1][y - 1, y, y + 1]'s first cell
  uint32_t off[19];   // a lane's byte offset from there, by population
  uint32_t self;

  __device__ __forceinline__ Pull(const LatticeGeom& g, int x, int y, int z) {
    const int xs[3] = {nbr(x, -1, g.nx, g.bcx), x, nbr(x, 1, g.nx, g.bcx)};
    const int ys[3] = {nbr(y, -1, g.ny, g.bcy), y, nbr(y, 1, g.ny, g.bcy)};
    const int zs[3] = {nbr(z, -1, g.nz, g.bcz), z, nbr(z, 1, g.nz, g.bcz)};
    uint32_t phase[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const uint32_t t = (uint32_t)zs[k] * g.lay.zcells + (uint32_t)ys[j] * (uint32_t)g.nx;
        phase[k][j] = t & (kBlock - 1);
        row[k][j] = (int64_t)(t >> kBlockShift) * (19 * kBlock);
      }
#pragma unroll
    for (int a = 0; a < 19; ++a) {
      const uint32_t t = phase[1 - ez(a)][1 - ey(a)] + (uint32_t)xs[1 - ex(a)];
      off[a] = (t + (t >> kBlockShift) * (18u * kBlock)) * (uint32_t)sizeof(T);
    }
    self = off[0];
  }
  __device__ __forceinline__ const T* from(const T* region, int a) const {
    return region + row[1 - ez(a)][1 - ey(a)] + a * kBlock;
  }
  __device__ __forceinline__ T* to(T* region, int a) const {
    return region + row[1][1] + a * kBlock;
  }
};

// Planes: a scalar plane base and a 32-bit byte offset within it.
template <typename T>
struct Pull<T, false> {
  uint32_t off[19], self;
  int64_t cs;

  __device__ __forceinline__ Pull(const LatticeGeom& g, int x, int y, int z) : cs(g.lay.pstr) {
    pull_offsets(x, y, z, g.nx, g.ny, g.nz, g.bcx, g.bcy, g.bcz, 0u, (uint32_t)sizeof(T), off,
                 self);
  }
  __device__ __forceinline__ const T* from(const T* region, int a) const { return region + a * cs; }
  __device__ __forceinline__ T* to(T* region, int a) const { return region + a * cs; }
};

// -------------------------------------------------------------------------
// Fused step on one lattice: grid (ceil(nx/BX), ceil(ny/BY), ceil(nz/CZ)),
// block (BX, BY); each thread updates CZ cells along z. EXT: relaxation times
// of each cell from eta/s. Tiles are taken in the row-per-XCD order of
// block_tile. NTS: nontemporal stores; without, plain stores, which the host
// picks when the double-buffered state fits the memory-side cache, so that the
// next step reads it back from there. (The store kind is a template argument:
// two store loops that differ only in the hint behind a run-time branch get
// merged by the compiler, which keeps the plain form.)
// -------------------------------------------------------------------------
template <typename T, int BX, int BY, int CZ, bool DIAG, bool EXT, bool NTS, bool BLOCKS>
__global__ __launch_bounds__(BX* BY) void k_step_lattice(const T* __restrict__ src,
                                                        T* __restrict__ dst, LatticeGeom geo,
                                                        double* __restrict__ partials,
                                                        unsigned long long* __restrict__ bad) {
  static_assert(BX % 64 == 0, "a wave holds cells of one row");
  int bx, by, bz;
  block_tile(bx, by, bz);
  const int x = bx * BX + threadIdx.x;
  int y = by * BY + threadIdx.y;
  if constexpr (BLOCKS) y = __builtin_amdgcn_readfirstlane(y);  // one row per wave
  const int tid = threadIdx.y * BX + threadIdx.x;
  const bool act = (x < geo.nx) && (y < geo.ny);
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  int nbad = 0;
#pragma unroll 1
  for (int k = 0; k < CZ; ++k) {
    const int z = bz * CZ + k;
    if (act && z < geo.nz) {
      const Pull<T, BLOCKS> pull(geo, x, y, z);
      const auto get = [&](const T* region, int a) { return ld(pull.from(region, a), pull.off[a]); };
      const auto put = [&](T* region, int a, T v) {
        if constexpr (NTS)
          st_nt(pull.to(region, a), pull.self, v);
        else
          st(pull.to(region, a), pull.self, v);
      };
      if constexpr (!EXT && (sizeof(T) == 8 || CZ == 1)) {
        // g first (its recovery needs no f), then f with the recovered
        // velocity: one distribution's 19 values in flight at a time. FP64:
        // 142 instead of 154 VGPRs, 1.5 % faster; FP32 with one cell per
        // thread: 0.3-0.5 % faster (with several cells per thread FP32 lost
        // 2-9 %, and loads both at once). The arithmetic is that of collide(),
        // bit for bit. (The relaxation times from eta/s and the general
        // equation of state need N before the recovery, so the EXT kernels
        // load both at once.)
        T g[19];
#pragma unroll
        for (int a = 0; a < 19; ++a) g[a] = get(src + geo.lay.greg, a);
        double E, Mx, My, Mz, gs;
        g_sums(g, geo.ref, E, Mx, My, Mz, gs);
        Macro mac;
        const bool ok = recover(E, Mx, My, Mz, mac);
        if (ok) collide_g(g, Mx, My, Mz, gs, mac, geo.rt, geo.ref);
#pragma unroll
        for (int a = 0; a < 19; ++a) put(dst + geo.lay.greg, a, g[a]);
        T f[19];
#pragma unroll
        for (int a = 0; a < 19; ++a) f[a] = get(src, a);
        double fs = 0.0;
#pragma unroll
        for (int a = 0; a < 19; ++a) fs += (double)f[a];
        const double N = geo.ref.n + fs;
        if (ok) collide_f(f, N, fs, mac, geo.rt, geo.ref);
#pragma unroll
        for (int a = 0; a < 19; ++a) put(dst, a, f[a]);
        nbad += ok ? 0 : 1;
        if (DIAG) {
          acc[0] += N;
          acc[1] += E;
          acc[2] += Mx;
          acc[3] += My;
          acc[4] += Mz;
        }
      } else {
        T f[19], g[19];
#pragma unroll
        for (int a = 0; a < 19; ++a) {
          f[a] = get(src, a);
          g[a] = get(src + geo.lay.greg, a);
        }
        Sums s;
        const bool ok = collide<T, EXT, sizeof(T) == 4 && (CZ > 1)>(f, g, geo.rt, geo.ref, s, &geo.ext);
        nbad += ok ? 0 : 1;
        if (DIAG)
#pragma unroll
          for (int i = 0; i < 5; ++i) acc[i] += s.v[i];
#pragma unroll
        for (int a = 0; a < 19; ++a) {
          put(dst, a, f[a]);
          put(dst + geo.lay.greg, a, g[a]);
        }
      }
    }
  }
  if (nbad) count_bad(bad, nbad);
  if (DIAG) {
    block_sum5<BX * BY>(acc, tid);
    if (tid == 0) {
      const int64_t b = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
#pragma unroll
      for (int i = 0; i < 5; ++i) partials[b * 5 + i] = acc[i];
    }
  }
}

// ------------------------------ variants ---------------------------------
// The /w3 forms reserve 44 KiB of LDS per 256-thread block that the kernel
// never touches: 3 blocks fit in a CU's 160 KiB where 4 would by registers, so
// they run 3 waves per SIMD instead of 4. On 512^3 FP32 lattices the 256 x 1
// block ran 2 % faster so (fewer streams in flight per channel); on 256^3
// the blocks were within 1 %.
constexpr unsigned kOcc3Lds = 44 * 1024;
constexpr LatticeVariant kLat[] = {{64, 1, 1},  {64, 4, 1},  {128, 2, 1}, {256, 1, 1},
                                   {64, 4, 2},  {256, 1, 2}, {128, 2, 4}, {256, 1, 4},
                                   {128, 2, 1}, {256, 1, 1}};
constexpr int kNumLat = sizeof(kLat) / sizeof(kLat[0]);
template <typename T, int BX, int BY, int CZ, bool EXT, bool NTS, bool BLOCKS>
void lat_launch_stores(bool diag, dim3 grid, dim3 block, unsigned lds, const void* src, void* dst,
                       const LatticeGeom& g, double* partials, unsigned long long* bad,
                       hipStream_t s) {
  if (diag)
    hipLaunchKernelGGL((k_step_lattice<T, BX, BY, CZ, true, EXT, NTS, BLOCKS>), grid, block, lds, s,
                       (const T*)src, (T*)dst, g, partials, bad);
  else
    hipLaunchKernelGGL((k_step_lattice<T, BX, BY, CZ, false, EXT, NTS, BLOCKS>), grid, block, lds, s,
                       (const T*)src, (T*)dst, g, partials, bad);
}

template <typename T, int BX, int BY, int CZ, bool EXT, bool BLOCKS>
hipError_t lat_launch(bool diag, const void* src, void* dst, const LatticeGeom& g,
                      double* partials, unsigned long long* bad, hipStream_t s,
                      unsigned lds = 0) {
  dim3 block(BX, BY, 1);
  dim3 grid((g.nx + BX - 1) / BX, (g.ny + BY - 1) / BY, (g.nz + CZ - 1) / CZ);
  if (g.cached_store)
    lat_launch_stores<T, BX, BY, CZ, EXT, false, BLOCKS>(diag, grid, block, lds, src, dst, g,
                                                         partials, bad, s);
  else
    lat_launch_stores<T, BX, BY, CZ, EXT, true, BLOCKS>(diag, grid, block, lds, src, dst, g,
                                                        partials, bad, s);
  return hipGetLastError();
}

template <typename T, bool EXT, bool BLOCKS>
hipError_t lat_dispatch(int v, bool diag, const void* src, void* dst, const LatticeGeom& g,
                        double* partials, unsigned long long* bad, hipStream_t s) {
  switch (v) {
    case 0: return lat_launch<T, 64, 1, 1, EXT, BLOCKS>(diag, src, dst, g, partials, bad, s);
    case 1: return lat_launch<T, 64, 4, 1, EXT, BLOCKS>(diag, src, dst, g, partials, bad, s);
    case 2: return lat_launch<T, 128, 2, 1, EXT, BLOCKS>(diag, src, dst, g, partials, bad, s);
    case 3: return lat_launch<T, 256, 1, 1, EXT, BLOCKS>(diag, src, dst, g, partials, bad, s);
    case 4: return lat_launch<T, 64, 4, 2, EXT, BLOCKS>(diag, src, dst, g, partials, bad, s);
    case 5: return lat_launch<T, 256, 1, 2, EXT, BLOCKS>(diag, src, dst, g, partials, bad, s);
    case 6: return lat_launch<T, 128, 2, 4, EXT, BLOCKS>(diag, src, dst, g, partials, bad, s);
    case 7: return lat_launch<T, 256, 1, 4, EXT, BLOCKS>(diag, src, dst, g, partials, bad, s);
    case 8: return lat_launch<T, 128, 2, 1, EXT, BLOCKS>(diag, src, dst, g, partials, bad, s, kOcc3Lds);
    case 9: return lat_launch<T, 256, 1, 1, EXT, BLOCKS>(diag, src, dst, g, partials, bad, s, kOcc3Lds);
  }
  return hipErrorInvalidValue;
}

template <bool BLOCKS>
hipError_t lat_step(int precision, int v, bool diag, bool ext, const void* src, void* dst,
                    const LatticeGeom& g, double* partials, unsigned long long* bad,
                    hipStream_t s) {
  if (precision)
    return ext ? lat_dispatch<float, true, BLOCKS>(v, diag, src, dst, g, partials, bad, s)
               : lat_dispatch<float, false, BLOCKS>(v, diag, src, dst, g, partials, bad, s);
  return ext ? lat_dispatch<double, true, BLOCKS>(v, diag, src, dst, g, partials, bad, s)
             : lat_dispatch<double, false, BLOCKS>(v, diag, src, dst, g, partials, bad, s);
}

}  // namespace
}  // namespace rlb
