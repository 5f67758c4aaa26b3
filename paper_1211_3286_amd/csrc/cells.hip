// One step of every member per launch, one cell per thread: the persistent
// path's form for members larger than a block. A block works on NT consecutive
// cells of one member; the member kernels (one block per member, all steps in
// one launch) leave 255 CUs idle on a single lattice and take a pass over the
// block per NT cells, the price here is a launch per step.
//
// Bound by latency: a step is the launch, one wave's loads, its arithmetic (some
// 850 instructions at 5-6 clocks each with no other wave to fill in) and its
// stores. D3Q19 blocks of 64 cells therefore run a wave for f and one for g, each
// with its own recovery (500 instructions the longer chain), and a single
// lattice's shape comes as an argument, not through a descriptor in memory.
// NT = 64 spreads small members over the CUs; NT = 256 is for batches that fill
// the chip anyway, one thread per cell. 24^3 FP32 periodic, us a step:
// k_step_members<float,512,1> 117, one thread per cell 4.7, this 4.2; 20 x 16 x 12
// 4.5 and 3.8; 8^3 FP64 4.2 and 3.8. (Two steps per launch on tiles of 4^3 cells
// with their halo, 24^3: 5.4.)

#include <hip/hip_runtime.h>

#include "cell.hpp"
#include "cell2d.hpp"
#include "device_util.hpp"
#include "internal.hpp"

namespace rlb {

namespace {

// What a launch works on. A single lattice's shape comes with the launch: its
// blocks need no read of a descriptor before they know their cells.
struct CellsLaunch {
  MemberLaunch m;
  int32_t n_members;
  int32_t diag;
  int32_t nx, ny, nz, bcx, bcy, bcz;  // n_members = 1
};

struct Shape {
  int nx, ny, nz, bcx, bcy, bcz, ncells;
  uint32_t offset;
};

// The member of block b, its shape and the block's index within it (uniform).
template <int NT>
__device__ __forceinline__ const MemberDesc& member_of_block(const CellsLaunch& a, int& b,
                                                             Shape& h) {
  const MemberDesc* __restrict__ descs = a.m.descs;
  if (a.n_members == 1) {
    h = {a.nx, a.ny, a.nz, a.bcx, a.bcy, a.bcz, a.nx * a.ny * a.nz, 0u};
    return descs[0];
  }
  const auto first = [&](int m) { return NT == 64 ? descs[m].first64 : descs[m].first256; };
  int lo = 0, hi = a.n_members - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first(mid) <= b)
      lo = mid;
    else
      hi = mid - 1;
  }
  b -= first(lo);
  const MemberDesc& d = descs[lo];
  h = {d.nx, d.ny, d.nz, d.bcx, d.bcy, d.bcz, d.ncells, (uint32_t)d.offset};
  return d;
}

template <int NT>
__device__ __forceinline__ void leave_sums(bool diag, double (&acc)[5], double* partials) {
  if (!diag) return;
  block_sum5<NT>(acc, threadIdx.x);
  if (threadIdx.x == 0)
#pragma unroll
    for (int i = 0; i < 5; ++i) partials[(int64_t)blockIdx.x * 5 + i] = acc[i];
}

// One distribution of a cell: pulled, collided, stored at `self` (the other one
// is read for the recovery).
template <typename T, bool EXT, bool F>
__device__ __forceinline__ bool half_cell(const T* __restrict__ src, T* __restrict__ dst,
                                          int64_t cs, const uint32_t (&off)[19], uint32_t self,
                                          const MemberDesc& d, Sums& s) {
  T f[19] = {}, g[19];
#pragma unroll
  for (int q = 0; q < 19; ++q) {
    g[q] = ld(src + (int64_t)(19 + q) * cs, off[q]);
    if (F || EXT) f[q] = ld(src + (int64_t)q * cs, off[q]);
  }
  const bool ok = collide_half<T, EXT, F>(f, g, d.rt, d.ref, s, d.ext);
#pragma unroll
  for (int q = 0; q < 19; ++q) st(dst + (int64_t)(F ? q : 19 + q) * cs, self, F ? f[q] : g[q]);
  return ok;
}

template <typename T, int NT, bool SPLIT, bool EXT>
__global__ __launch_bounds__(SPLIT ? 2 * NT : NT) void k_step_cells(CellsLaunch l) {
  const MemberLaunch& a = l.m;
  int b = blockIdx.x;
  Shape h;
  const MemberDesc& d = member_of_block<NT>(l, b, h);
  const T* __restrict__ src = (const T*)a.bufA;
  T* __restrict__ dst = (T*)a.bufB;
  const bool f_half = SPLIT && __builtin_amdgcn_readfirstlane(threadIdx.x) >= NT;
  const int c = b * NT + (int)threadIdx.x - (f_half ? NT : 0);
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (c < h.ncells) {
    const int yz = c / h.nx;
    const int z = yz / h.ny;
    uint32_t off[19], self;
    pull_offsets(c - yz * h.nx, yz - z * h.ny, z, h.nx, h.ny, h.nz, h.bcx, h.bcy, h.bcz, h.offset,
                 (uint32_t)sizeof(T), off, self);
    Sums s;
    if constexpr (SPLIT) {
      if (f_half) {
        half_cell<T, EXT, true>(src, dst, a.cs, off, self, d, s);
#pragma unroll
        for (int i = 0; i < 5; ++i) acc[i] = s.v[i];
      } else if (!half_cell<T, EXT, false>(src, dst, a.cs, off, self, d, s)) {
        count_bad(a.bad, 1);
      }
    } else {
      T f[19], g[19];
#pragma unroll
      for (int q = 0; q < 19; ++q) {
        g[q] = ld(src + (int64_t)(19 + q) * a.cs, off[q]);
        f[q] = ld(src + (int64_t)q * a.cs, off[q]);
      }
      const bool ok = collide<T, EXT>(f, g, d.rt, d.ref, s, &d.ext);
      if (!ok) count_bad(a.bad, 1);
#pragma unroll
      for (int i = 0; i < 5; ++i) acc[i] = s.v[i];
#pragma unroll
      for (int q = 0; q < 19; ++q) {
        st(dst + (int64_t)q * a.cs, self, f[q]);
        st(dst + (int64_t)(19 + q) * a.cs, self, g[q]);
      }
    }
  }
  leave_sums<SPLIT ? 2 * NT : NT>(l.diag, acc, a.partials);
}

template <typename T, int NT, bool CORR, bool EXT>
__global__ __launch_bounds__(NT) void k_d2q9_cells(CellsLaunch l) {
  const MemberLaunch& a = l.m;
  int b = blockIdx.x;
  Shape h;
  const MemberDesc& d = member_of_block<NT>(l, b, h);
  const T* __restrict__ src = (const T*)a.bufA;
  T* __restrict__ dst = (T*)a.bufB;
  const int c = b * NT + threadIdx.x;
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (c < h.ncells) {
    const int y = c / h.nx;
    const int x = c - y * h.nx;
    d2q9::C7Fields fm, fp;
    if constexpr (CORR)
      d2q9::c7_neighbours(src, a.cs, x, y, h.nx, h.ny, h.bcx, h.bcy, h.offset, d.ref, fm, fp);
    uint32_t off[9], self;
    d2q9::pull_offsets(x, y, h.nx, h.ny, h.bcx, h.bcy, h.offset, (uint32_t)sizeof(T), off, self);
    T f[9], g[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      f[q] = ld(src + (int64_t)q * a.cs, off[q]);
      g[q] = ld(src + (int64_t)(9 + q) * a.cs, off[q]);
    }
    Sums s;
    const bool ok = d2q9::collide<T, CORR, EXT>(f, g, d.rt, d.ref, s, &fm, &fp, &d.ext);
    if (!ok) count_bad(a.bad, 1);
#pragma unroll
    for (int i = 0; i < 5; ++i) acc[i] = s.v[i];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      st(dst + (int64_t)q * a.cs, self, f[q]);
      st(dst + (int64_t)(9 + q) * a.cs, self, g[q]);
    }
  }
  leave_sums<NT>(l.diag, acc, a.partials);
}

template <typename T, int NT>
hipError_t cells_launch(bool d2, bool corr, bool ext, const CellsLaunch& a, int nblocks,
                        hipStream_t s) {
  const void* f;
  if (d2)
    f = corr ? (ext ? (const void*)&k_d2q9_cells<T, NT, true, true>
                    : (const void*)&k_d2q9_cells<T, NT, true, false>)
             : (ext ? (const void*)&k_d2q9_cells<T, NT, false, true>
                    : (const void*)&k_d2q9_cells<T, NT, false, false>);
  else
    f = ext ? (const void*)&k_step_cells<T, NT, NT == 64, true>
            : (const void*)&k_step_cells<T, NT, NT == 64, false>;
  void* args[] = {const_cast<CellsLaunch*>(&a)};
  return hipLaunchKernel(f, dim3(nblocks), dim3(NT == 64 && !d2 ? 2 * NT : NT), args, 0, s);
}

}  // namespace

hipError_t launch_step_cells(int precision, bool d2, int variant, bool corr, bool ext, bool diag,
                             const MemberLaunch& m, const MemberDesc& first, int n_members,
                             int nblocks, hipStream_t s) {
  const CellsLaunch a{m,        n_members, diag ? 1 : 0, first.nx, first.ny,
                      first.nz, first.bcx, first.bcy,    first.bcz};
  if (variant == 0)
    return precision ? cells_launch<float, 64>(d2, corr, ext, a, nblocks, s)
                     : cells_launch<double, 64>(d2, corr, ext, a, nblocks, s);
  return precision ? cells_launch<float, 256>(d2, corr, ext, a, nblocks, s)
                   : cells_launch<double, 256>(d2, corr, ext, a, nblocks, s);
}

const char* cells_kernel_name(int precision, bool d2, int v) {
  static const char* n[2][2][2] = {
      {{"k_step_cells<double,64>", "k_step_cells<double,256>"},
       {"k_step_cells<float,64>", "k_step_cells<float,256>"}},
      {{"k_d2q9_cells<double,64>", "k_d2q9_cells<double,256>"},
       {"k_d2q9_cells<float,64>", "k_d2q9_cells<float,256>"}}};
  return v < 0 || v >= kNumCells ? "?" : n[d2 ? 1 : 0][precision ? 1 : 0][v];
}

}  // namespace rlb
