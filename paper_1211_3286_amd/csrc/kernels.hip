// Kernels of the relativistic MRT lattice Boltzmann step for gfx950.
//
// Population storage (one buffer): 38 planes of cs elements, planes 0..18 hold
// f_a and planes 19..37 hold g_a (velocity order of rlb.h); a cell's element
// in every plane sits at the same index. Two such buffers alternate (A/B):
// a step pulls from one and writes the other, so it is race-free.
//
// The fused step kernel reads 38 values per cell (streaming with periodic or
// zero-gradient sources), collides in registers (cell.hpp) and writes 38
// values: 2 x 38 x sizeof(T) bytes of HBM traffic per cell update, no reuse.
// Loads use a uniform plane base plus a 32-bit byte offset per lane; stores
// are nontemporal (written once, read by the next step from HBM).

#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_util.hpp"
#include "internal.hpp"
#include "step_lattice.hpp"

namespace rlb {

namespace {

// -------------------------------------------------------------------------
// Persistent step over a batch: one block per member, all nsteps inside the
// launch with a block barrier between steps (members are independent, so no
// grid-wide synchronisation exists). Each thread updates CPT cells per sweep,
// interleaved by NT so every load instruction is coalesced.
// -------------------------------------------------------------------------
template <typename T, int NT, int CPT, bool EXT>
__global__ __launch_bounds__(NT) void k_step_members(MemberLaunch a) {
  const MemberDesc d = a.descs[blockIdx.x];
  const int tid = threadIdx.x;
  const uint32_t esz = sizeof(T);
  const uint32_t base = (uint32_t)d.offset;
  const bool tube = d.nx == 1 && d.ny == 1;
  int nbad = 0;
  for (int t = 0; t < a.nsteps; ++t) {
    const bool odd = a.pingpong && (t & 1);
    const T* __restrict__ src = (const T*)(odd ? a.bufB : a.bufA);
    T* __restrict__ dst = (T*)(odd ? a.bufA : a.bufB);
    const int64_t sidx = a.step0 + t + 1;
    const bool diag = a.diag_every > 0 && ((sidx % a.diag_every) == 0 || t == a.nsteps - 1);
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int c0 = 0; c0 < d.ncells; c0 += NT * CPT) {
#pragma unroll
      for (int k = 0; k < CPT; ++k) {
        const int c = c0 + k * NT + tid;
        if (c < d.ncells) {
          int x = 0, y = 0, z = c;  // quasi-1D member (1 x 1 x L): no division
          if (!tube) {
            x = c % d.nx;
            const int yz = c / d.nx;
            y = yz % d.ny;
            z = yz / d.ny;
          }
          uint32_t off[19], self;
          pull_offsets(x, y, z, d.nx, d.ny, d.nz, d.bcx, d.bcy, d.bcz, base, esz, off, self);
          T f[19], g[19];
#pragma unroll
          for (int q = 0; q < 19; ++q) {
            f[q] = ld(src + (int64_t)q * a.cs, off[q]);
            g[q] = ld(src + (int64_t)(19 + q) * a.cs, off[q]);
          }
          Sums s;
          const bool ok = collide<T, EXT, sizeof(T) == 4>(f, g, d.rt, d.ref, s, &d.ext);
          nbad += ok ? 0 : 1;
#pragma unroll
          for (int i = 0; i < 5; ++i) acc[i] += s.v[i];
#pragma unroll
          for (int q = 0; q < 19; ++q) {
            st(dst + (int64_t)q * a.cs, self, f[q]);
            st(dst + (int64_t)(19 + q) * a.cs, self, g[q]);
          }
        }
      }
    }
    if (diag) {
      block_sum5<NT>(acc, tid);
      if (tid == 0)
#pragma unroll
        for (int i = 0; i < 5; ++i) a.partials[(int64_t)blockIdx.x * 5 + i] = acc[i];
    }
    __syncthreads();
  }
  if (nbad) count_bad(a.bad, nbad);
}

// -------------------------------------------------------------------------
// Segmented persistent step over a batch: one block per segment (a range of
// whole z-planes of one member), all nsteps inside the launch. Before step t
// a segment waits until its two neighbour segments have completed t steps
// (their planes z0-1 and z1 are pulled, and they read this segment's planes
// of the buffer it is about to overwrite). After its step every thread
// makes its stores visible device-wide before thread 0 publishes the flag
// with release semantics. A wait that exceeds spin_limit polls sets *error
// and ends the launch for that block (every block reaches the exit).
// -------------------------------------------------------------------------
__device__ __forceinline__ bool wait_flag(const unsigned long long* f, unsigned long long target,
                                          int spin_limit) {
  for (int i = 0; i < spin_limit; ++i) {
    if (__hip_atomic_load(f, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) >= target) return true;
    __builtin_amdgcn_s_sleep(2);
  }
  return false;
}

template <typename T, int NT, int CPT>
__global__ __launch_bounds__(NT) void k_step_segments(SegLaunch a) {
  const Segment sg = a.segs[blockIdx.x];
  const MemberDesc d = a.descs[sg.member];
  const int tid = threadIdx.x;
  const uint32_t esz = sizeof(T);
  const uint32_t base = (uint32_t)d.offset;
  const int plane = d.nx * d.ny;
  const bool tube = plane == 1;
  const int c_begin = sg.z0 * plane, c_end = sg.z1 * plane;
  __shared__ int s_abort;
  int nbad = 0;
  for (int t = 0; t < a.nsteps; ++t) {
    const unsigned long long target = a.epoch + (unsigned long long)t;
    if (tid == 0) {
      bool ok = true;
      if (sg.left >= 0) ok = wait_flag(a.flags + sg.left, target, a.spin_limit);
      if (ok && sg.right >= 0) ok = wait_flag(a.flags + sg.right, target, a.spin_limit);
      s_abort = ok ? 0 : 1;
      if (!ok) atomicOr(a.error, 1);
    }
    __syncthreads();
    if (s_abort) break;
    const bool odd = a.pingpong && (t & 1);
    const T* __restrict__ src = (const T*)(odd ? a.bufB : a.bufA);
    T* __restrict__ dst = (T*)(odd ? a.bufA : a.bufB);
    const int64_t sidx = a.step0 + t + 1;
    const bool diag = a.diag_every > 0 && ((sidx % a.diag_every) == 0 || t == a.nsteps - 1);
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int c0 = c_begin; c0 < c_end; c0 += NT * CPT) {
#pragma unroll
      for (int k = 0; k < CPT; ++k) {
        const int c = c0 + k * NT + tid;
        if (c < c_end) {
          int x = 0, y = 0, z = c;  // quasi-1D member (1 x 1 x L): no division
          if (!tube) {
            x = c % d.nx;
            const int yz = c / d.nx;
            y = yz % d.ny;
            z = yz / d.ny;
          }
          uint32_t off[19], self;
          pull_offsets(x, y, z, d.nx, d.ny, d.nz, d.bcx, d.bcy, d.bcz, base, esz, off, self);
          T f[19], g[19];
#pragma unroll
          for (int q = 0; q < 19; ++q) {
            f[q] = ld(src + (int64_t)q * a.cs, off[q]);
            g[q] = ld(src + (int64_t)(19 + q) * a.cs, off[q]);
          }
          Sums s;
          const bool ok = collide<T>(f, g, d.rt, d.ref, s);
          nbad += ok ? 0 : 1;
#pragma unroll
          for (int i = 0; i < 5; ++i) acc[i] += s.v[i];
#pragma unroll
          for (int q = 0; q < 19; ++q) {
            st(dst + (int64_t)q * a.cs, self, f[q]);
            st(dst + (int64_t)(19 + q) * a.cs, self, g[q]);
          }
        }
      }
    }
    if (diag) {
      block_sum5<NT>(acc, tid);
      if (tid == 0)
#pragma unroll
        for (int i = 0; i < 5; ++i) a.partials[(int64_t)blockIdx.x * 5 + i] = acc[i];
    }
    __threadfence();
    __syncthreads();
    if (tid == 0)
      __hip_atomic_store(a.flags + blockIdx.x, target + 1ull, __ATOMIC_RELEASE,
                         __HIP_MEMORY_SCOPE_AGENT);
  }
  if (nbad) count_bad(a.bad, nbad);
}

// -------------------------------------------------------------------------
// Tube rounds: one block per TubeSeg. A 1 x 1 x L lattice streams only along z:
// the x and y components of e wrap onto the same cell, so a thread keeps its
// cell's populations with e_z = 0 and exchanges the others through LDS, planes of
// NT consecutive words. SPLIT: two threads per window cell, in different waves,
// one for f and one for g. The f thread also reads the cell's whole g for the
// recovery, and in the extended model the g thread its f. Per step: pull,
// barrier, collide in registers, write, barrier. Inadmissible counts and
// diagnostics cover owned cells only (halo cells are computed twice). EXT:
// relaxation times from eta/s and the general equation of state, per cell.
//
// Bound by the serial chain of a step, 5-6 clocks an instruction where a SIMD has
// one wave (a tube of 800 cells is four blocks), and by the chip's issue rate
// for batches that fill it: the split shortens the first (850 to some 500
// instructions) and leaves the second as it was, as only the sums and the
// recovery are done twice. Windows of 512 cells stay whole: 16 waves leave 128
// registers to each, too few for a split FP64 cell; those of 256 because batches
// take them. 800 cells FP64, us a step: one thread with all 38 values exchanged
// 2.0 (rounds of 16 steps), this split 1.3, with rounds of 32 1.2; 64 tubes of up to
// 3200 cells, FP64 4.8 and, whole, 4.3.
// -------------------------------------------------------------------------
template <bool EXT>
struct TubePlanes {
  // LDS planes: g, then f; without EXT nobody reads another cell's f with e_z = 0
  static constexpr int n = EXT ? 38 : 29;
  static constexpr int f(int q) {
    int k = 19;
    for (int i = 0; i < q; ++i) k += EXT || ez(i) != 0 ? 1 : 0;
    return k;
  }
};

// The work of a thread on the distributions it has (F: f, G: g). The f and the g
// waves of a split block run this function in two instantiations and meet at its
// barriers, which count waves wherever they stand in the code: every wave must pass
// as many. So no barrier, and no way out of the loop, may depend on F, G or the
// lane; block_sum5 counts too, and its shared array is the same one for both.
template <typename T, int NT, bool EXT, bool F, bool G>
__device__ __forceinline__ void tube_cell(const TubeRound& a, T (*__restrict__ lds)[NT], int w) {
  using P = TubePlanes<EXT>;
  constexpr int kThreads = F && G ? NT : 2 * NT;
  const TubeSeg sg = a.segs[blockIdx.x];
  const MemberDesc d = a.descs[sg.member];
  const int L = d.nz;
  const bool live = w < sg.wlen;
  const int own_lo = sg.own0 - sg.win0, own_hi = sg.own1 - sg.win0;
  const bool owned = w >= own_lo && w < own_hi;
  // global cell of window cell w
  int z = sg.win0 + w;
  if (z < 0) z += L;
  if (z >= L) z -= L;
  const int64_t gi = d.offset + z;
  T f[19] = {}, g[19] = {};
  const auto leave = [&]() {
#pragma unroll
    for (int q = 0; q < 19; ++q) {
      if (G && (!F || ez(q) != 0)) lds[q][w] = g[q];
      if (F && ((EXT && !G) || ez(q) != 0)) lds[P::f(q)][w] = f[q];
    }
  };
  if (live) {
#pragma unroll
    for (int q = 0; q < 19; ++q) {
      if (F) f[q] = ((const T*)a.src)[q * a.cs + gi];
      if (G) g[q] = ((const T*)a.src)[(19 + q) * a.cs + gi];
    }
    leave();
  }
  // pull sources inside the window for e_z = +1 (from w-1) and e_z = -1 (from w+1)
  int sp = w - 1, sm = w + 1;
  if (sp < 0) sp = sg.left == kEdgeWrap ? sg.wlen - 1 : 0;
  if (sm >= sg.wlen) sm = sg.right == kEdgeWrap ? 0 : sg.wlen - 1;
  if (!live) sp = sm = 0;
  __syncthreads();
  int nbad = 0;
  for (int t = 0; t < a.nsteps; ++t) {
    if (live) {
#pragma unroll
      for (int q = 0; q < 19; ++q) {
        const int src = ez(q) > 0 ? sp : (ez(q) < 0 ? sm : w);
        if (!G || ez(q) != 0) g[q] = lds[q][src];
        if (F ? ez(q) != 0 : EXT) f[q] = lds[P::f(q)][src];
      }
    }
    __syncthreads();
    const int64_t sidx = a.step0 + t + 1;
    const bool diag =
        a.diag_every > 0 && ((sidx % a.diag_every) == 0 || sidx == a.last_step);
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (live) {
      Sums s;
      bool ok;
      if constexpr (F && G)
        ok = collide<T, EXT>(f, g, d.rt, d.ref, s, &d.ext);
      else
        ok = collide_half<T, EXT, F>(f, g, d.rt, d.ref, s, d.ext);
      if (G && owned) nbad += ok ? 0 : 1;
      if (F && owned && diag)
#pragma unroll
        for (int i = 0; i < 5; ++i) acc[i] = s.v[i];
      leave();
    }
    if (diag) {
      block_sum5<kThreads>(acc, threadIdx.x);
      if (threadIdx.x == 0)
#pragma unroll
        for (int i = 0; i < 5; ++i) a.partials[(int64_t)blockIdx.x * 5 + i] = acc[i];
    }
    __syncthreads();
  }
  if (owned) {
#pragma unroll
    for (int q = 0; q < 19; ++q) {
      if (F) ((T*)a.dst)[q * a.cs + gi] = f[q];
      if (G) ((T*)a.dst)[(19 + q) * a.cs + gi] = g[q];
    }
  }
  if (nbad) count_bad(a.bad, nbad);
}

constexpr bool tube_split(int nt) { return nt <= 128; }

template <typename T, int NT, bool EXT>
__global__ __launch_bounds__(tube_split(NT) ? 2 * NT : NT) void k_step_tubes(TubeRound a) {
  __shared__ T lds[TubePlanes<EXT>::n][NT];
  if constexpr (!tube_split(NT))
    tube_cell<T, NT, EXT, true, true>(a, lds, threadIdx.x);
  else if (__builtin_amdgcn_readfirstlane(threadIdx.x) >= NT)
    tube_cell<T, NT, EXT, true, false>(a, lds, (int)threadIdx.x - NT);
  else
    tube_cell<T, NT, EXT, false, true>(a, lds, threadIdx.x);
}

__device__ __forceinline__ int find_member(const MemberDesc* __restrict__ d, int n, int64_t c) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (d[mid].offset <= c)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

__global__ __launch_bounds__(256) void k_begin(unsigned long long* small, size_t n_small,
                                               unsigned long long* flags, size_t n_flags,
                                               MemberDesc one, MemberDesc* descs) {
  const size_t i = blockIdx.x * (size_t)256 + threadIdx.x, step = gridDim.x * (size_t)256;
  for (size_t k = i; k < n_small; k += step) small[k] = 0ull;
  for (size_t k = i; k < n_flags; k += step) flags[k] = 0ull;
  if (descs && i == 0) *descs = one;
}

// Input pass, grid (blocks, members): a block's share of a member's cells is
// validated and summed (n gamma and eps, for the member's reference state). A
// thread adds its cells c, c + 256 kRefBlocks, ... in that order; with kAhead of
// them loaded at once the 64 blocks stream a large lattice (512^3: 2.7 ms,
// one cell at a time in two kernels 5.6 ms).
__global__ __launch_bounds__(256) void k_prepare(const MemberDesc* descs,
                                                 const double* __restrict__ n0,
                                                 const double* __restrict__ eps0,
                                                 const double* __restrict__ u0, int64_t ncells,
                                                 int planar, double* parts, HostView* view) {
  constexpr int kAhead = 8;
  const MemberDesc& d = descs[blockIdx.y];
  const Ext& x = d.ext;
  double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  int nb = 0;
  for (int64_t c0 = blockIdx.x * 256 + threadIdx.x; c0 < d.ncells;
       c0 += (int64_t)kAhead * kRefBlocks * 256) {
    double n[kAhead], e[kAhead], ux[kAhead], uy[kAhead], uz[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const int64_t c = c0 + (int64_t)k * kRefBlocks * 256;
      const int64_t i = d.offset + (c < d.ncells ? c : c0);
      n[k] = n0[i];
      e[k] = eps0[i];
      ux[k] = u0[i];
      uy[k] = u0[ncells + i];
      uz[k] = u0[2 * ncells + i];
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (c0 + (int64_t)k * kRefBlocks * 256 >= d.ncells) break;
      const double uu = ux[k] * ux[k] + uy[k] * uy[k] + uz[k] * uz[k];
      const bool ok = (e[k] > 0.0) && (n[k] >= 0.0) && (uu < 1.0) && (n[k] < INFINITY) &&
                      (e[k] < INFINITY) && (!planar || uz[k] == 0.0) &&
                      (!x.general_eos || e[k] - x.mass * n[k] > 0.0);
      nb += ok ? 0 : 1;
      v[0] += n[k] / sqrt(1.0 - uu);
      v[1] += e[k];
    }
  }
  if (nb) atomicAdd(&view->refused, (unsigned long long)nb);
  block_sum5<256>(v, threadIdx.x);
  if (threadIdx.x == 0) {
    const int64_t b = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    for (int k = 0; k < 5; ++k) parts[b * 5 + k] = v[k];
  }
}

// The members' references from their partial sums (added block by block), one
// wave per member.
__global__ __launch_bounds__(kRefBlocks) void k_member_ref(MemberDesc* descs, const double* parts,
                                                           int nblocks, HostView* view) {
  __shared__ double sh[kRefBlocks][2];
  MemberDesc& d = descs[blockIdx.x];
  const int b = threadIdx.x;
  const double* p = parts + ((int64_t)blockIdx.x * nblocks + b) * 5;
  sh[b][0] = b < nblocks ? p[0] : 0.0;
  sh[b][1] = b < nblocks ? p[1] : 0.0;
  __syncthreads();
  if (b != 0) return;
  double sn = 0.0, se = 0.0;
#pragma unroll 8
  for (int k = 0; k < kRefBlocks; ++k) {
    sn += sh[k][0];
    se += sh[k][1];
  }
  d.ref.n = sn / d.ncells;
  d.ref.P = se / (3.0 * d.ncells);
  if (blockIdx.x == 0) view->ref0 = d.ref;
}

template <typename T>
__global__ __launch_bounds__(256) void k_init(T* state, StateLayout l, const MemberDesc* descs,
                                              int n_members, const double* n0,
                                              const double* eps0, const double* u0,
                                              int64_t ncells) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < ncells;
       i += (int64_t)gridDim.x * 256) {
    const MemberDesc& d = descs[find_member(descs, n_members, i)];
    double f[19], g[19];
    const double P = pressure_of(eps0[i], n0[i], d.ext);
    equilibrium_dev(n0[i], eps0[i], P, u0[i], u0[ncells + i], u0[2 * ncells + i], d.ref, f, g);
    T* const c = state + cell_element(l, cell_index(l, (uint32_t)i));
#pragma unroll
    for (int a = 0; a < 19; ++a) {
      c[a * l.pstr] = (T)f[a];
      c[l.greg + a * l.pstr] = (T)g[a];
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_export(const T* state, StateLayout l,
                                                const MemberDesc* descs, int n_members,
                                                int64_t ncells, double* n, double* eps,
                                                double* P, double* gamma, double* u,
                                                double* partials,
                                                const unsigned long long* refused) {
  if (refused && *refused) return;
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < ncells;
       i += (int64_t)gridDim.x * 256) {
    const MemberDesc& d = descs[find_member(descs, n_members, i)];
    T f[19], g[19];
    const T* const c = state + cell_element(l, cell_index(l, (uint32_t)i));
#pragma unroll
    for (int a = 0; a < 19; ++a) {
      f[a] = c[a * l.pstr];
      g[a] = c[l.greg + a * l.pstr];
    }
    double N, E, Mx, My, Mz, fs, gs;
    cell_sums(f, g, d.ref, N, E, Mx, My, Mz, fs, gs);
    acc[0] += N;
    acc[1] += E;
    acc[2] += Mx;
    acc[3] += My;
    acc[4] += Mz;
    Macro m;
    const bool gen = d.ext.general_eos != 0;
    const bool ok = recover_model(N, E, Mx, My, Mz, d.ext, m);
    const double nan = __builtin_nan("");
    // eps = (eps + P) - P; for P = eps/3 the closed form 3/4 sigma (1 - u^2)
    const double e =
        !ok ? nan : (gen ? m.sigma * (1.0 - m.u2) - m.P : 0.75 * m.sigma * (1.0 - m.u2));
    const double gm = ok ? 1.0 / sqrt(1.0 - m.u2) : nan;
    if (n) n[i] = ok ? N / gm : nan;
    if (eps) eps[i] = e;
    if (P) P[i] = !ok ? nan : (gen ? m.P : e / 3.0);
    if (gamma) gamma[i] = gm;
    if (u) {
      u[i] = ok ? m.ux : nan;
      u[ncells + i] = ok ? m.uy : nan;
      u[2 * ncells + i] = ok ? m.uz : nan;
    }
  }
  block_sum5<256>(acc, threadIdx.x);
  if (threadIdx.x == 0)
    for (int k = 0; k < 5; ++k) partials[(int64_t)blockIdx.x * 5 + k] = acc[k];
}

// Planes [p0, p0 + np) of the state as FP64 populations (reference added back);
// plane p < 19 is f_p, plane p >= 19 is g_(p-19). out[(p - p0) * ncells + cell].
template <typename T>
__global__ __launch_bounds__(256) void k_population_planes(const T* state, StateLayout l,
                                                           const MemberDesc* descs, int n_members,
                                                           int64_t ncells, int p0, int np,
                                                           double* out) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < ncells;
       i += (int64_t)gridDim.x * 256) {
    const Ref ref = descs[find_member(descs, n_members, i)].ref;
    const T* const c = state + cell_element(l, cell_index(l, (uint32_t)i));
    for (int p = p0; p < p0 + np; ++p) {
      const double r = p < 19 ? weight(p) * ref.n : gref_unit(p - 19) * ref.P;
      const int64_t e = p < 19 ? p * l.pstr : l.greg + (p - 19) * l.pstr;
      out[(int64_t)(p - p0) * ncells + i] = (double)c[e] + r;
    }
  }
}

// What the host reads back (single block): the deterministic sum of nparts
// partial 5-vectors and the total of the inadmissible-cell slots.
__global__ __launch_bounds__(256) void k_finish(const double* partials, int nparts,
                                                const unsigned long long* __restrict__ slots,
                                                HostView* view) {
  static_assert(kBadSlots == 256, "one slot per thread");
  __shared__ unsigned long long bad[4];
  double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  unsigned long long t = slots[(size_t)threadIdx.x * kBadStride];
  for (int j = threadIdx.x; j < nparts; j += 256)
#pragma unroll
    for (int k = 0; k < 5; ++k) v[k] += partials[(int64_t)j * 5 + k];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
  if ((threadIdx.x & 63) == 0) bad[threadIdx.x >> 6] = t;
  block_sum5<256>(v, threadIdx.x);
  if (threadIdx.x == 0) {
    for (int k = 0; k < 5; ++k) view->sums[k] = v[k];
    view->bad = (bad[0] + bad[1]) + (bad[2] + bad[3]);
  }
}

// ------------------------------ variants ---------------------------------
// At most 512 threads: with 1024 (4 waves per SIMD, at most 128 VGPRs) every
// member build spills to scratch, which the build refuses for every kernel.
constexpr MemberVariant kMem[] = {{256, 1}, {512, 1}, {256, 2}, {512, 2}};
constexpr int kNumMem = sizeof(kMem) / sizeof(kMem[0]);

constexpr MemberVariant kSeg[] = {{256, 1}, {256, 2}, {512, 1}, {128, 4}, {256, 4}};
constexpr int kNumSeg = sizeof(kSeg) / sizeof(kSeg[0]);

template <typename T>
const void* seg_func(int v) {
  switch (v) {
    case 0: return (const void*)&k_step_segments<T, 256, 1>;
    case 1: return (const void*)&k_step_segments<T, 256, 2>;
    case 2: return (const void*)&k_step_segments<T, 512, 1>;
    case 3: return (const void*)&k_step_segments<T, 128, 4>;
    case 4: return (const void*)&k_step_segments<T, 256, 4>;
  }
  return nullptr;
}

constexpr TubeVariant kTube[] = {{256, 8}, {256, 16}, {512, 16}, {512, 32},
                                 {128, 8}, {128, 16}, {128, 32}};
constexpr int kNumTube = sizeof(kTube) / sizeof(kTube[0]);

template <typename T, bool EXT>
const void* tube_func(int v) {
  switch (v) {
    case 0: return (const void*)&k_step_tubes<T, 256, EXT>;
    case 1: return (const void*)&k_step_tubes<T, 256, EXT>;
    case 2: return (const void*)&k_step_tubes<T, 512, EXT>;
    case 3: return (const void*)&k_step_tubes<T, 512, EXT>;
    case 4: case 5: case 6: return (const void*)&k_step_tubes<T, 128, EXT>;
  }
  return nullptr;
}

int grid_for(int64_t n) {
  int64_t b = (n + 255) / 256;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return (int)b;
}

template <typename T, bool EXT>
const void* mem_func(int v) {
  switch (v) {
    case 0: return (const void*)&k_step_members<T, 256, 1, EXT>;
    case 1: return (const void*)&k_step_members<T, 512, 1, EXT>;
    case 2: return (const void*)&k_step_members<T, 256, 2, EXT>;
    case 3: return (const void*)&k_step_members<T, 512, 2, EXT>;
  }
  return nullptr;
}

}  // namespace

int num_lattice_variants() { return kNumLat; }
int num_segment_variants() { return kNumSeg; }
int num_tube_variants() { return kNumTube; }
TubeVariant tube_variant(int i) { return kTube[i]; }

hipError_t tube_kernel(int precision, int v, bool ext, const void** func, dim3* block) {
  if (v < 0 || v >= kNumTube) return hipErrorInvalidValue;
  if (ext)
    *func = precision ? tube_func<float, true>(v) : tube_func<double, true>(v);
  else
    *func = precision ? tube_func<float, false>(v) : tube_func<double, false>(v);
  *block = dim3((tube_split(kTube[v].nt) ? 2 : 1) * kTube[v].nt, 1, 1);
  return hipSuccess;
}

const char* tube_kernel_name(int precision, int v) {
  static const char* n32[] = {"k_step_tubes<float,256>/h8", "k_step_tubes<float,256>/h16",
                              "k_step_tubes<float,512>/h16", "k_step_tubes<float,512>/h32",
                              "k_step_tubes<float,128>/h8", "k_step_tubes<float,128>/h16",
                              "k_step_tubes<float,128>/h32"};
  static const char* n64[] = {"k_step_tubes<double,256>/h8", "k_step_tubes<double,256>/h16",
                              "k_step_tubes<double,512>/h16", "k_step_tubes<double,512>/h32",
                              "k_step_tubes<double,128>/h8", "k_step_tubes<double,128>/h16",
                              "k_step_tubes<double,128>/h32"};
  if (v < 0 || v >= kNumTube) return "?";
  return precision ? n32[v] : n64[v];
}
MemberVariant segment_variant(int i) { return kSeg[i]; }

hipError_t segment_kernel(int precision, int v, const void** func, dim3* block) {
  if (v < 0 || v >= kNumSeg) return hipErrorInvalidValue;
  *func = precision ? seg_func<float>(v) : seg_func<double>(v);
  *block = dim3(kSeg[v].nt, 1, 1);
  return hipSuccess;
}

const char* segment_kernel_name(int precision, int v) {
  static const char* n32[] = {"k_step_segments<float,256,1>", "k_step_segments<float,256,2>",
                              "k_step_segments<float,512,1>", "k_step_segments<float,128,4>",
                              "k_step_segments<float,256,4>"};
  static const char* n64[] = {"k_step_segments<double,256,1>", "k_step_segments<double,256,2>",
                              "k_step_segments<double,512,1>", "k_step_segments<double,128,4>",
                              "k_step_segments<double,256,4>"};
  if (v < 0 || v >= kNumSeg) return "?";
  return precision ? n32[v] : n64[v];
}
LatticeVariant lattice_variant(int i) { return kLat[i]; }
int num_member_variants() { return kNumMem; }
MemberVariant member_variant(int i) { return kMem[i]; }

int lattice_partials(int v, const LatticeGeom& g) {
  const LatticeVariant lv = kLat[v];
  return ((g.nx + lv.bx - 1) / lv.bx) * ((g.ny + lv.by - 1) / lv.by) *
         ((g.nz + lv.cz - 1) / lv.cz);
}

const char* lattice_kernel_name(int precision, int v) {
  static const char* n32[] = {"k_step_lattice<float,64,1,1>",  "k_step_lattice<float,64,4,1>",
                              "k_step_lattice<float,128,2,1>", "k_step_lattice<float,256,1,1>",
                              "k_step_lattice<float,64,4,2>",  "k_step_lattice<float,256,1,2>",
                              "k_step_lattice<float,128,2,4>", "k_step_lattice<float,256,1,4>",
                              "k_step_lattice<float,128,2,1>/w3",
                              "k_step_lattice<float,256,1,1>/w3"};
  static const char* n64[] = {
      "k_step_lattice<double,64,1,1>",     "k_step_lattice<double,64,4,1>",
      "k_step_lattice<double,128,2,1>",    "k_step_lattice<double,256,1,1>",
      "k_step_lattice<double,64,4,2>",     "k_step_lattice<double,256,1,2>",
      "k_step_lattice<double,128,2,4>",    "k_step_lattice<double,256,1,4>",
      "k_step_lattice<double,128,2,1>/w3", "k_step_lattice<double,256,1,1>/w3"};
  if (v < 0 || v >= kNumLat) return "?";
  return precision ? n32[v] : n64[v];
}

const char* member_kernel_name(int precision, int v) {
  static const char* n32[] = {"k_step_members<float,256,1>", "k_step_members<float,512,1>",
                              "k_step_members<float,256,2>", "k_step_members<float,512,2>"};
  static const char* n64[] = {"k_step_members<double,256,1>", "k_step_members<double,512,1>",
                              "k_step_members<double,256,2>", "k_step_members<double,512,2>"};
  if (v < 0 || v >= kNumMem) return "?";
  return precision ? n32[v] : n64[v];
}

hipError_t launch_begin(unsigned long long* small, size_t n_small, unsigned long long* flags,
                        size_t n_flags, const MemberDesc* one, MemberDesc* descs, hipStream_t s) {
  const int64_t most = (int64_t)std::max(n_small, n_flags);
  const int blocks = (int)std::min<int64_t>((most + 255) / 256, 1024);
  hipLaunchKernelGGL(k_begin, dim3(blocks), dim3(256), 0, s, small, n_small, flags, n_flags,
                     one ? *one : MemberDesc{}, one ? descs : nullptr);
  return hipGetLastError();
}

hipError_t launch_prepare(MemberDesc* descs, int n_members, int nblocks, const double* n0,
                          const double* eps0, const double* u0, int64_t ncells, int planar,
                          double* parts, HostView* view, hipStream_t s) {
  hipLaunchKernelGGL(k_prepare, dim3(nblocks, n_members), dim3(256), 0, s,
                     (const MemberDesc*)descs, n0, eps0, u0, ncells, planar, parts, view);
  hipLaunchKernelGGL(k_member_ref, dim3(n_members), dim3(kRefBlocks), 0, s, descs,
                     (const double*)parts, nblocks, view);
  return hipGetLastError();
}

hipError_t launch_init(int precision, void* state, const StateLayout& l, const MemberDesc* descs,
                       int n_members, const double* n0, const double* eps0, const double* u0,
                       int64_t ncells, hipStream_t s) {
  dim3 grid(grid_for(ncells));
  if (precision)
    hipLaunchKernelGGL(k_init<float>, grid, dim3(256), 0, s, (float*)state, l, descs,
                       n_members, n0, eps0, u0, ncells);
  else
    hipLaunchKernelGGL(k_init<double>, grid, dim3(256), 0, s, (double*)state, l, descs,
                       n_members, n0, eps0, u0, ncells);
  return hipGetLastError();
}

hipError_t launch_step_lattice(int precision, int v, bool diag, bool ext, const void* src,
                               void* dst, const LatticeGeom& g, double* partials,
                               unsigned long long* bad, hipStream_t s) {
  return g.lay.shift == kBlockShift
             ? launch_step_blocks(precision, v, diag, ext, src, dst, g, partials, bad, s)
             : lat_step<false>(precision, v, diag, ext, src, dst, g, partials, bad, s);
}

hipError_t member_kernel(int precision, int v, bool ext, const void** func, dim3* block) {
  if (v < 0 || v >= kNumMem) return hipErrorInvalidValue;
  if (ext)
    *func = precision ? mem_func<float, true>(v) : mem_func<double, true>(v);
  else
    *func = precision ? mem_func<float, false>(v) : mem_func<double, false>(v);
  *block = dim3(kMem[v].nt, 1, 1);
  return hipSuccess;
}

hipError_t launch_export(int precision, const void* state, const StateLayout& l,
                         const MemberDesc* descs, int n_members, int64_t ncells, double* n, double* eps, double* P,
                         double* gamma, double* u, double* partials, int nparts,
                         const unsigned long long* refused, hipStream_t s) {
  if (precision)
    hipLaunchKernelGGL(k_export<float>, dim3(nparts), dim3(256), 0, s, (const float*)state, l,
                       descs, n_members, ncells, n, eps, P, gamma, u, partials, refused);
  else
    hipLaunchKernelGGL(k_export<double>, dim3(nparts), dim3(256), 0, s, (const double*)state,
                       l, descs, n_members, ncells, n, eps, P, gamma, u, partials, refused);
  return hipGetLastError();
}

hipError_t launch_population_planes(int precision, const void* state, const StateLayout& l,
                                    const MemberDesc* descs, int n_members, int64_t ncells,
                                    int p0, int np, double* out, hipStream_t s) {
  dim3 grid(grid_for(ncells));
  if (precision)
    hipLaunchKernelGGL(k_population_planes<float>, grid, dim3(256), 0, s, (const float*)state,
                       l, descs, n_members, ncells, p0, np, out);
  else
    hipLaunchKernelGGL(k_population_planes<double>, grid, dim3(256), 0, s,
                       (const double*)state, l, descs, n_members, ncells, p0, np, out);
  return hipGetLastError();
}

hipError_t launch_finish(const double* partials, int nparts, const unsigned long long* slots,
                         HostView* view, hipStream_t s) {
  hipLaunchKernelGGL(k_finish, dim3(1), dim3(256), 0, s, partials, nparts, slots, view);
  return hipGetLastError();
}

}  // namespace rlb
