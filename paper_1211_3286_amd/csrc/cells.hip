// One step of every member per launch, one cell per thread: the persistent
// path's form for members larger than a block. A block works on NT consecutive
// cells of one member; the member kernels (one block per member, all steps in
// one launch) leave 255 CUs idle on a single lattice and take a pass over the
// block per NT cells, the price here is a launch per step.
//
// Bound by latency: a step is one wave's loads, arithmetic and stores plus the
// launch, about 5 us while the cells fit the chip once. NT = 64 spreads small
// members over the CUs; NT = 256 is for batches that fill it anyway.
// 24^3 FP32 periodic, us a step, before (k_step_members<float,512,1>) and now:
// 117 and 5.

#include <hip/hip_runtime.h>

#include "cell.hpp"
#include "cell2d.hpp"
#include "device_util.hpp"
#include "internal.hpp"

namespace rlb {

namespace {

// The member of block b, and the block's index within it (uniform).
template <int NT>
__device__ __forceinline__ int member_of_block(const MemberDesc* __restrict__ descs, int n,
                                               int& b) {
  const auto first = [&](int m) { return NT == 64 ? descs[m].first64 : descs[m].first256; };
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first(mid) <= b)
      lo = mid;
    else
      hi = mid - 1;
  }
  b -= first(lo);
  return lo;
}

template <int NT>
__device__ __forceinline__ void leave_sums(bool diag, double (&acc)[5], double* partials) {
  if (!diag) return;
  block_sum5<NT>(acc, threadIdx.x);
  if (threadIdx.x == 0)
#pragma unroll
    for (int i = 0; i < 5; ++i) partials[(int64_t)blockIdx.x * 5 + i] = acc[i];
}

template <typename T, int NT, bool EXT>
__global__ __launch_bounds__(NT) void k_step_cells(MemberLaunch a, int n_members, bool diag) {
  int b = blockIdx.x;
  const MemberDesc& d = a.descs[member_of_block<NT>(a.descs, n_members, b)];
  const T* __restrict__ src = (const T*)a.bufA;
  T* __restrict__ dst = (T*)a.bufB;
  const int c = b * NT + threadIdx.x;
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (c < d.ncells) {
    const int yz = c / d.nx;
    const int z = yz / d.ny;
    uint32_t off[19], self;
    pull_offsets(c - yz * d.nx, yz - z * d.ny, z, d.nx, d.ny, d.nz, d.bcx, d.bcy, d.bcz,
                 (uint32_t)d.offset, (uint32_t)sizeof(T), off, self);
    T f[19], g[19];
#pragma unroll
    for (int q = 0; q < 19; ++q) {
      g[q] = ld(src + (int64_t)(19 + q) * a.cs, off[q]);
      f[q] = ld(src + (int64_t)q * a.cs, off[q]);
    }
    Sums s;
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
  leave_sums<NT>(diag, acc, a.partials);
}

template <typename T, int NT, bool CORR, bool EXT>
__global__ __launch_bounds__(NT) void k_d2q9_cells(MemberLaunch a, int n_members, bool diag) {
  int b = blockIdx.x;
  const MemberDesc& d = a.descs[member_of_block<NT>(a.descs, n_members, b)];
  const T* __restrict__ src = (const T*)a.bufA;
  T* __restrict__ dst = (T*)a.bufB;
  const int c = b * NT + threadIdx.x;
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (c < d.ncells) {
    const int y = c / d.nx;
    const int x = c - y * d.nx;
    d2q9::C7Fields fm, fp;
    if constexpr (CORR)
      d2q9::c7_neighbours(src, a.cs, x, y, d.nx, d.ny, d.bcx, d.bcy, (uint32_t)d.offset, d.ref,
                          fm, fp);
    uint32_t off[9], self;
    d2q9::pull_offsets(x, y, d.nx, d.ny, d.bcx, d.bcy, (uint32_t)d.offset, (uint32_t)sizeof(T),
                       off, self);
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
  leave_sums<NT>(diag, acc, a.partials);
}

template <typename T, int NT>
hipError_t cells_launch(bool d2, bool corr, bool ext, bool diag, const MemberLaunch& a,
                        int n_members, int nblocks, hipStream_t s) {
  const void* f;
  if (d2)
    f = corr ? (ext ? (const void*)&k_d2q9_cells<T, NT, true, true>
                    : (const void*)&k_d2q9_cells<T, NT, true, false>)
             : (ext ? (const void*)&k_d2q9_cells<T, NT, false, true>
                    : (const void*)&k_d2q9_cells<T, NT, false, false>);
  else
    f = ext ? (const void*)&k_step_cells<T, NT, true> : (const void*)&k_step_cells<T, NT, false>;
  void* args[] = {const_cast<MemberLaunch*>(&a), &n_members, &diag};
  return hipLaunchKernel(f, dim3(nblocks), dim3(NT), args, 0, s);
}

}  // namespace

hipError_t launch_step_cells(int precision, bool d2, int variant, bool corr, bool ext, bool diag,
                             const MemberLaunch& a, int n_members, int nblocks, hipStream_t s) {
  if (variant == 0)
    return precision ? cells_launch<float, 64>(d2, corr, ext, diag, a, n_members, nblocks, s)
                     : cells_launch<double, 64>(d2, corr, ext, diag, a, n_members, nblocks, s);
  return precision ? cells_launch<float, 256>(d2, corr, ext, diag, a, n_members, nblocks, s)
                   : cells_launch<double, 256>(d2, corr, ext, diag, a, n_members, nblocks, s);
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
