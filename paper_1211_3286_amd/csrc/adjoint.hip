// Tape and adjoint of the g update (rlb_grad).
//
// Forward: rlb_step keeps g every K steps (checkpoints). Reverse: for each
// segment [kK, kK + K), last first, the g states are recomputed from the
// checkpoint with a g-only step that is bit-identical to the forward (g never
// reads f), then one adjoint kernel per step runs backwards. Each adjoint
// kernel reads, per cell, the 19 forward populations it pulled at that step
// (from the recomputed state), gathers the 19 adjoint populations of the cells
// that pulled from it (the transpose of streaming: one source per population
// in the interior, up to four at clamped corners, never an atomic), applies
// the transposed collision Jacobian (adjoint_cell.hpp) and writes 19 values:
// 3 x 19 populations of traffic per cell-step. dL/dtau is accumulated in FP64
// per block across all steps and reduced once at the end. The recomputation of
// a segment runs beside the reverse steps of the one after it (two segment
// buffers): on a second stream, or on small lattices in the same launches.
//
// Bound by memory and, in the reverse step, by FP64 arithmetic as much: 100
// populations' traffic per cell and step, at 512 x 512 FP32 20 MB a g state that
// the last-level cache holds: a pair of steps takes 20 us, 5 TB/s. The launches go
// out one by one: a graph of them, built anew for each handle, kept the GPU idle
// for 0.9 ms per 200 steps. Forward and backward, 512 x 512 FP32 200 steps 8.2 and
// now 7.1 ms; smaller lattices are bound by the launches, of which there are
// half as many: 150 x 170 FP32 60 steps 1.6 and 1.1 ms, 100 x 90 FP64 80 steps 1.9
// and 1.2.

#include <hip/hip_runtime.h>

#include <algorithm>

#include "adjoint.hpp"
#include "adjoint_cell.hpp"
#include "device_util.hpp"

namespace rlb {

namespace {

size_t al(size_t v) { return (v + 255) / 256 * 256; }

int grid_of(int64_t n) {
  int64_t b = (n + 255) / 256;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return (int)b;
}

// What the reverse-sweep kernels read of the lattice (a small argument, held
// in scalar registers): shape, boundaries, relaxation rates and reference.
struct AdjGeom {
  int32_t nx, ny, nz, bcx, bcy, bcz;
  Rates rt;
  Ref ref;
};

AdjGeom adj_geom(const MemberDesc& d) {
  AdjGeom g;
  g.nx = d.nx;
  g.ny = d.ny;
  g.nz = d.nz;
  g.bcx = d.bcx;
  g.bcy = d.bcy;
  g.bcz = d.bcz;
  g.rt = d.rt;
  g.ref = d.ref;
  return g;
}

template <typename G>
__device__ __forceinline__ void decompose(int c, const G& d, int& x, int& y, int& z) {
  x = c % d.nx;
  const int yz = c / d.nx;
  y = yz % d.ny;
  z = yz / d.ny;
}

// The step kernels' geometry: each wave takes 64 consecutive x-cells of one
// row (y, z), a block kRows rows, one cell per thread. The row index is
// uniform in a wave, so (y, z) come from a scalar division and no cell index
// is divided; with no loop over cells the reverse step fits 117 VGPRs (4
// waves per SIMD).
constexpr int kRows = 4;

// The 8 XCDs of the chip take the blocks of a launch in turn (block b on XCD
// b mod 8), each XCD behind its own L2. Taken as launched, the 8 blocks of a
// 512-cell row went to 8 XCDs: each XCD kept a 64-cell column strip, and the
// line at each edge of a strip, which the x-shifted pulls of the waves on
// both sides share, was fetched by two XCDs. The kernels renumber their
// blocks so that each XCD takes one contiguous run of row blocks, a band of
// whole rows: no row is split over XCDs.
constexpr unsigned kXcds = 8;

int64_t row_blocks(const AdjGeom& g) {
  const int64_t rows = (int64_t)g.ny * g.nz;
  return (g.nx + 63) / 64 * ((rows + kRows - 1) / kRows);
}

// This thread's cell in block b of nb: x, and its row r = y + ny z (uniform in
// its wave). Block b, on XCD j = b mod 8, is the (b / 8)-th of that XCD's run
// of logical blocks: XCD j takes q + (j < rem) of the nb = 8q + rem blocks,
// starting at jq + min(j, rem). The renumbering is one to one for any nb.
__device__ __forceinline__ void row_cell(unsigned b, unsigned nb, int nx, int& x, int& r) {
  const unsigned j = b % kXcds, q = nb / kXcds, rem = nb % kXcds;
  const unsigned lb = j * q + (j < rem ? j : rem) + b / kXcds;
  const unsigned gx = (unsigned)(nx + 63) / 64;
  x = (int)((lb % gx) * 64 + threadIdx.x);
  r = __builtin_amdgcn_readfirstlane((int)((lb / gx) * kRows + threadIdx.y));
}

// Cells y with src(y, e) = c along one axis (the pull source is y - e,
// wrapped or clamped): one in the interior, up to two at a clamped end.
__device__ __forceinline__ int preimages(int c, int e, int N, int bc, int (&out)[2]) {
  if (e == 0) {
    out[0] = c;
    return 1;
  }
  int s = c + e;
  if (bc == 0) {
    if (s < 0) s += N;
    if (s >= N) s -= N;
    out[0] = s;
    return 1;
  }
  int n = 0;
  if (s >= 0 && s <= N - 1) out[n++] = s;
  if (e > 0 && c == 0) out[n++] = 0;
  if (e < 0 && c == N - 1) out[n++] = N - 1;
  return n;
}

// Transposed streaming: adjoint of the pre-collision populations of the cells
// that pulled population a from cell (x, y, z), summed. Away from clamped
// faces that cell is x + e_a, the pull source of the opposite population
// (e_opp = -e_a), so the gather is 19 plain loads; cells on a clamped face
// walk the preimage sets per axis.
__device__ __forceinline__ int opposite(int a) { return a == 0 ? 0 : ((a & 1) ? a + 1 : a - 1); }

template <typename T, typename G>
__device__ __forceinline__ void gather_adjoint(const T* __restrict__ adj, int64_t cs, int x, int y,
                                               int z, const G& d, T (&gb)[19]) {
  const bool face = (d.bcx && (x == 0 || x == d.nx - 1)) ||
                    (d.bcy && (y == 0 || y == d.ny - 1)) ||
                    (d.bcz && (z == 0 || z == d.nz - 1));
  if (!face) {
    uint32_t off[19], self;
    pull_offsets(x, y, z, d.nx, d.ny, d.nz, d.bcx, d.bcy, d.bcz, 0u, (uint32_t)sizeof(T), off,
                 self);
#pragma unroll
    for (int a = 0; a < 19; ++a) gb[a] = ld(adj + (int64_t)a * cs, off[opposite(a)]);
    return;
  }
#pragma unroll
  for (int a = 0; a < 19; ++a) {
    int px[2], py[2], pz[2];
    const int nxp = preimages(x, ex(a), d.nx, d.bcx, px);
    const int nyp = preimages(y, ey(a), d.ny, d.bcy, py);
    const int nzp = preimages(z, ez(a), d.nz, d.bcz, pz);
    T s = T(0.0);
    for (int k = 0; k < nzp; ++k)
      for (int j = 0; j < nyp; ++j)
        for (int i = 0; i < nxp; ++i)
          s += adj[(int64_t)a * cs + ((int64_t)pz[k] * d.ny + py[j]) * d.nx + px[i]];
    gb[a] = s;
  }
}

// One DPP exchange of a double between the lanes of a row of 16 (CTRL a
// permutation within the row, so every lane receives a value).
template <int CTRL>
__device__ __forceinline__ double dpp_row(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Sum of a double over the 64 lanes of a wave (all lanes active), uniform in
// the wave: four DPP exchanges make every lane of a row of 16 hold the row's
// sum (quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror,
// row_mirror), then the four row sums are read out. VALU work only: no LDS
// round trips, which matter when every wave of a single-round launch reduces
// at the same time.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_row<0xB1>(v);
  v += dpp_row<0x4E>(v);
  v += dpp_row<0x141>(v);
  v += dpp_row<0x140>(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// g-only forward step between g-plane buffers (recomputation of a segment).
template <typename T>
__device__ __forceinline__ void gstep_block(const T* __restrict__ src, T* __restrict__ dst,
                                            int64_t cs, const AdjGeom& d, unsigned b,
                                            unsigned nb) {
  const uint32_t esz = sizeof(T);
  int x, r;
  row_cell(b, nb, d.nx, x, r);
  if (x < d.nx && r < d.ny * d.nz) {
    const int y = r % d.ny, z = r / d.ny;
    uint32_t off[19], self;
    pull_offsets(x, y, z, d.nx, d.ny, d.nz, d.bcx, d.bcy, d.bcz, 0u, esz, off, self);
    T g[19];
#pragma unroll
    for (int a = 0; a < 19; ++a) g[a] = ld(src + (int64_t)a * cs, off[a]);
    collide_g_only(g, d.rt, d.ref);
#pragma unroll
    for (int a = 0; a < 19; ++a) st(dst + (int64_t)a * cs, self, g[a]);
  }
}

// dL/dg* of the final state from dL/du, dL/deps.
template <typename T>
__global__ __launch_bounds__(256) void k_adj_loss(const T* __restrict__ state, int64_t cs,
                                                  MemberDesc d, const double* __restrict__ dLdu,
                                                  const double* __restrict__ dLdeps,
                                                  T* __restrict__ out) {
  const int64_t nc = d.ncells;
  for (int c = blockIdx.x * 256 + threadIdx.x; c < d.ncells; c += gridDim.x * 256) {
    T g[19], gb[19];
#pragma unroll
    for (int a = 0; a < 19; ++a) g[a] = state[(int64_t)a * cs + c];
    loss_adjoint(g, d.ref, dLdu[c], dLdu[nc + c], dLdu[2 * nc + c], dLdeps[c], gb);
#pragma unroll
    for (int a = 0; a < 19; ++a) out[(int64_t)a * cs + c] = gb[a];
  }
}

// One reverse step. state: g*(t) (the step's input); adj_in: either the
// adjoint of g*(t+1) (GATHER = false, straight from the loss) or the
// pre-collision adjoint of step t+1 (GATHER = true, transposed streaming
// applied here). adj_out: pre-collision adjoint of step t. dL/dtau partials per
// block.
template <typename T, bool GATHER>
__device__ __forceinline__ void adjoint_block(const T* __restrict__ state,
                                              const T* __restrict__ adj_in,
                                              T* __restrict__ adj_out, int64_t cs,
                                              const AdjGeom& d, double* __restrict__ partials,
                                              unsigned b, unsigned nb) {
  const uint32_t esz = sizeof(T);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  int x, r;
  row_cell(b, nb, d.nx, x, r);
  if (x < d.nx && r < d.ny * d.nz) {
    const int y = r % d.ny, z = r / d.ny;
    uint32_t off[19], self;
    pull_offsets(x, y, z, d.nx, d.ny, d.nz, d.bcx, d.bcy, d.bcz, 0u, esz, off, self);
    AdjPrep<T> pr;
    {
      T g[19];
#pragma unroll
      for (int a = 0; a < 19; ++a) g[a] = ld(state + (int64_t)a * cs, off[a]);
      adjoint_prepare(g, d.ref, pr);
    }
    T gb[19];
    if (GATHER) {
      gather_adjoint(adj_in, cs, x, y, z, d, gb);
    } else {
      const int64_t c = (int64_t)r * d.nx + x;
#pragma unroll
      for (int a = 0; a < 19; ++a) gb[a] = adj_in[(int64_t)a * cs + c];
    }
    adjoint_apply(pr, gb, d.rt, acc);
#pragma unroll
    for (int a = 0; a < 19; ++a) st(adj_out + (int64_t)a * cs, self, gb[a]);
  }
  // The block's four dL/dtau sums: one per wave by DPP, then thread 0 adds
  // the kRows waves' sums into the block's own partials slot.
  __shared__ double sh[kRows][4];
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = wave_sum(acc[q]);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) sh[threadIdx.y][q] = acc[q];
  __syncthreads();
  if (threadIdx.x == 0 && threadIdx.y == 0) {
    double* p = partials + (int64_t)b * 5;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < kRows; ++w) s += sh[w][q];
      p[q] += s;
    }
  }
}

// What a launch of the reverse sweep works on: a reverse step (k_adj_step), a
// recomputed step (k_gstep) or both (k_sweep_pair). Each kind has a kernel of its
// own: one kernel for all of them holds the registers of the reverse step and takes
// its branches in every launch (300 x 300 FP32, 49 recomputed steps and 50 reverse
// ones 783 us so, 760 apart; 60 x 60, 50 reverse steps, 336 and 321).
template <typename T>
struct SweepLaunch {
  const T* state;
  const T* adj_in;
  T* adj_out;
  const T* gsrc;
  T* gdst;
  int64_t cs;
  AdjGeom d;
  double* partials;
  uint32_t nb;  // blocks of either kind
};

template <typename T, bool GATHER>
__global__ __launch_bounds__(256) void k_adj_step(SweepLaunch<T> a) {
  adjoint_block<T, GATHER>(a.state, a.adj_in, a.adj_out, a.cs, a.d, a.partials, blockIdx.x,
                           gridDim.x);
}

// W: at most so many waves of it on a SIMD (by register count; 0: as many as fit).
template <typename T, int W>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(W ? W : 1, W ? W : 8))) void k_gstep(SweepLaunch<T> a) {
  gstep_block(a.gsrc, a.gdst, a.cs, a.d, blockIdx.x, gridDim.x);
}

// Both: groups of 8 blocks alternate, so that either kind keeps its XCDs and the
// CUs hold waves of both at a time.
template <typename T, bool GATHER>
__global__ __launch_bounds__(256) void k_sweep_pair(SweepLaunch<T> a) {
  const unsigned b = blockIdx.x / (2 * kXcds) * kXcds + blockIdx.x % kXcds;
  if (b >= a.nb) return;
  if (blockIdx.x & kXcds)
    gstep_block(a.gsrc, a.gdst, a.cs, a.d, b, a.nb);
  else
    adjoint_block<T, GATHER>(a.state, a.adj_in, a.adj_out, a.cs, a.d, a.partials, b, a.nb);
}

// dL/deps0, dL/du0 from the adjoint of the initial state.
template <typename T, bool GATHER>
__global__ __launch_bounds__(256) void k_adj_init(const T* __restrict__ adj_in, int64_t cs,
                                                  MemberDesc d, const double* __restrict__ f0,
                                                  double* __restrict__ deps0,
                                                  double* __restrict__ du0) {
  const int64_t nc = d.ncells;
  for (int c = blockIdx.x * 256 + threadIdx.x; c < d.ncells; c += gridDim.x * 256) {
    T gb[19];
    if (GATHER) {
      int x, y, z;
      decompose(c, d, x, y, z);
      gather_adjoint(adj_in, cs, x, y, z, d, gb);
    } else {
#pragma unroll
      for (int a = 0; a < 19; ++a) gb[a] = adj_in[(int64_t)a * cs + c];
    }
    double de, dx, dy, dz;
    init_adjoint(gb, f0[c], f0[nc + c], f0[2 * nc + c], f0[3 * nc + c], de, dx, dy, dz);
    deps0[c] = de;
    du0[c] = dx;
    du0[nc + c] = dy;
    du0[2 * nc + c] = dz;
  }
}

__global__ __launch_bounds__(256) void k_sum_parts(const double* parts, int n, double* out) {
  double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int j = threadIdx.x; j < n; j += 256)
#pragma unroll
    for (int k = 0; k < 5; ++k) v[k] += parts[(int64_t)j * 5 + k];
  block_sum5<256>(v, threadIdx.x);
  if (threadIdx.x == 0)
    for (int k = 0; k < 5; ++k) out[k] = v[k];
}

// Up to this many blocks of 256 cells a launch of the sweep runs both kinds of
// steps. Above, where they fill the chip, each kind has its stream: kernels of
// their own overlap better than blocks of one (512 x 512 FP32, 1000 steps: 20.0
// and 22.4 ms; 300 x 300, 375 blocks, 400 steps 4.1 and 4.2), while 150 x 170, 129
// blocks, is bound by the launches (60 steps forward and backward 1.1 ms, with a
// graph of single kernels 1.6).
constexpr int64_t kPairBlocks = 256;

// Recomputed steps on the second stream keep to the reverse step's 4 waves a SIMD
// while a launch has at most this many blocks. FP32 ones would fit 6 and then crowd
// the reverse steps, which end the chain; FP64 fits 4 by itself. FP32 gradients in
// us, 6 and 4 waves: 512 x 512 (1024 blocks), 200 steps 4100 and 3950, 1000 steps
// 19 950 and 18 700; 900 x 700 3050 and 2945; 900 x 900 (3375 blocks) 3929 and 3893;
// 1024 x 1024 (4096) 3000 and 3110; 1400 x 1000 4355 and 4400.
constexpr int64_t kBesideBlocks = 3584;

// The second stream and its events, made at the first gradient that wants them
// and kept with the tape.
hipError_t side_stream(Tape& t) {
  if (t.side) return hipSuccess;
  hipError_t e = hipStreamCreateWithFlags(&t.side, hipStreamNonBlocking);
  for (hipEvent_t* v : {&t.recomputed, &t.reversed})
    if (e == hipSuccess) e = hipEventCreateWithFlags(v, hipEventDisableTiming);
  return e;
}

// The reverse sweep over every checkpointed segment, last first. R(k): the
// reverse steps of segment k; G(k): the g-only recomputation of its states from
// checkpoint k. Segments alternate between two state buffers: G(k-1) runs beside
// R(k), after R(k+1), the last reader of its buffer. *cur: the adjoint buffer
// written last.
template <typename T>
hipError_t sweep(Tape& t, const GradContext& c, int* cur) {
  const TapeLayout& L = t.L;
  const int K = L.K;
  auto ckpt = [&](int64_t k) { return (const T*)(t.base + L.off_ckpt + (size_t)k * L.gbytes); };
  auto seg = [&](int64_t k, int64_t j) {
    return (T*)(t.base + L.off_seg + (size_t)((k & 1) * K + j) * L.gbytes);
  };
  T* const adj[2] = {(T*)(t.base + L.off_adj), (T*)(t.base + L.off_adj + L.gbytes)};
  SweepLaunch<T> r{};  // the reverse step of a launch
  r.cs = c.cs;
  r.d = adj_geom(c.desc);
  r.partials = (double*)(t.base + L.off_tparts);
  r.nb = (uint32_t)row_blocks(r.d);
  SweepLaunch<T> g = r;  // its recomputed step
  *cur = 0;
  const int64_t kmax = (c.steps - 1) / K;
  const auto steps_of = [&](int64_t k) { return std::min<int64_t>(K, c.steps - k * K); };
  const bool pair = r.nb <= kPairBlocks;
  const bool side = !pair && kmax > 0 && K > 1;
  hipError_t e = hipSuccess;
  if (side) e = side_stream(t);
  const auto reverse = [&](int64_t k, int64_t j) {
    r.state = j == 0 ? ckpt(k) : (const T*)seg(k, j);
    r.adj_in = adj[*cur];
    r.adj_out = adj[1 - *cur];
  };
  const auto recompute = [&](int64_t k, int64_t j) {  // state j - 1 of segment k to state j
    g.gsrc = j == 1 ? ckpt(k) : (const T*)seg(k, j - 1);
    g.gdst = seg(k, j);
  };
  bool gathered = false;
  const dim3 block(64, kRows);
  const auto launch_gstep = [&](hipStream_t s) {
    if (sizeof(T) == 4 && s != c.stream && g.nb <= kBesideBlocks)
      hipLaunchKernelGGL((k_gstep<T, 4>), dim3(g.nb), block, 0, s, g);
    else
      hipLaunchKernelGGL((k_gstep<T, 0>), dim3(g.nb), block, 0, s, g);
  };
  const auto launch_reverse = [&](bool with_gstep) {  // on the caller's stream
    const dim3 grid(with_gstep ? 2 * ((r.nb + kXcds - 1) / kXcds * kXcds) : r.nb);
    if (with_gstep) {
      r.gsrc = g.gsrc;
      r.gdst = g.gdst;
    }
    if (gathered && with_gstep)
      hipLaunchKernelGGL((k_sweep_pair<T, true>), grid, block, 0, c.stream, r);
    else if (gathered)
      hipLaunchKernelGGL((k_adj_step<T, true>), grid, block, 0, c.stream, r);
    else if (with_gstep)
      hipLaunchKernelGGL((k_sweep_pair<T, false>), grid, block, 0, c.stream, r);
    else
      hipLaunchKernelGGL((k_adj_step<T, false>), grid, block, 0, c.stream, r);
    gathered = true;
    *cur = 1 - *cur;
  };
  for (int64_t j = 1; j < steps_of(kmax); ++j) {
    recompute(kmax, j);
    launch_gstep(c.stream);
  }
  const auto after = [&](hipEvent_t v, hipStream_t done, hipStream_t waits) {
    if (e == hipSuccess) e = hipEventRecord(v, done);
    if (e == hipSuccess) e = hipStreamWaitEvent(waits, v, 0);
  };
  for (int64_t k = kmax; k >= 0 && e == hipSuccess; --k) {
    const int64_t nr = steps_of(k), ng = k > 0 ? K - 1 : 0;
    if (side && ng) after(t.reversed, c.stream, t.side);
    for (int64_t i = 0; i < std::max(nr, ng); ++i) {
      if (i < ng) recompute(k - 1, i + 1);
      if (i < nr) reverse(k, nr - 1 - i);
      const bool both = pair && i < ng && i < nr;
      if (i < ng && !both) launch_gstep(side ? t.side : c.stream);
      if (i < nr) launch_reverse(both);
    }
    if (side && ng) after(t.recomputed, t.side, c.stream);
  }
  if (e == hipSuccess) e = hipGetLastError();
  // an error on the way leaves nothing of the sweep behind on the side stream
  if (e != hipSuccess && t.side) (void)hipStreamSynchronize(t.side);
  return e;
}

template <typename T>
rlb_status run_grad(Tape& t, const GradContext& c, const double* dLdu, const double* dLdeps,
                    double dL_dtau[3], double* deps0, double* du0) {
  const TapeLayout& L = t.L;
  const MemberDesc d = c.desc;
  const int64_t cs = c.cs;
  const int64_t T_steps = c.steps;
  hipStream_t s = c.stream;
  const dim3 grid(grid_of(c.ncells)), block(256);
  const int nparts = (int)row_blocks(adj_geom(d));
  T* adj[2] = {(T*)(t.base + L.off_adj), (T*)(t.base + L.off_adj + L.gbytes)};
  const double* f0 = (const double*)(t.base + L.off_fields);
  double* parts = (double*)(t.base + L.off_tparts);
  if (hipMemsetAsync(parts, 0, sizeof(double) * 5 * (size_t)nparts, s) != hipSuccess)
    return RLB_E_DEVICE;
  const T* final_g = (const T*)((const char*)c.state + 19 * (size_t)cs * sizeof(T));
  hipLaunchKernelGGL(k_adj_loss<T>, grid, block, 0, s, final_g, cs, d, dLdu, dLdeps, adj[0]);
  int cur = 0;
  if (T_steps > 0 && sweep<T>(t, c, &cur) != hipSuccess) return RLB_E_DEVICE;
  if (T_steps > 0)
    hipLaunchKernelGGL((k_adj_init<T, true>), grid, block, 0, s, adj[cur], cs, d, f0, deps0, du0);
  else
    hipLaunchKernelGGL((k_adj_init<T, false>), grid, block, 0, s, adj[cur], cs, d, f0, deps0,
                       du0);
  hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(256), 0, s, parts, nparts, c.sums_out);
  if (hipGetLastError() != hipSuccess) return RLB_E_DEVICE;
  double h[5];
  if (hipMemcpyAsync(h, c.sums_out, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return RLB_E_DEVICE;
  // groups: v, e, eps, q (q folds into v when the ghost rows follow tau_v)
  dL_dtau[0] = h[0] + (c.tau_q_tied ? h[3] : 0.0);
  dL_dtau[1] = h[1];
  dL_dtau[2] = h[2];
  return RLB_OK;
}

}  // namespace

TapeLayout tape_layout(int nx, int ny, int nz, int64_t cs, size_t esz, int K, int tape_steps,
                       int max_parts) {
  TapeLayout L;
  const int64_t ncells = (int64_t)nx * ny * nz;
  AdjGeom g{};
  g.nx = nx;
  g.ny = ny;
  g.nz = nz;
  L.K = K;
  L.gbytes = 19 * (size_t)cs * esz;
  L.n_ckpt = tape_steps / K + 1;
  L.max_parts = (int)std::max<int64_t>(max_parts, row_blocks(g));  // reverse-step partials
  size_t o = 0;
  L.off_ckpt = o;
  o = al(o + L.gbytes * L.n_ckpt);
  L.off_seg = o;  // two segments' states: the one reversed, the next recomputed
  o = al(o + L.gbytes * 2 * (size_t)K);
  L.off_adj = o;
  o = al(o + 2 * L.gbytes);
  L.off_fields = o;
  o = al(o + sizeof(double) * 4 * (size_t)ncells);
  L.off_tparts = o;
  o = al(o + sizeof(double) * 5 * (size_t)L.max_parts);
  L.total = o;
  return L;
}

rlb_status tape_init(Tape& t, const TapeLayout& L, char* base, int precision, int64_t ncells,
                     int64_t cs, int K, int tape_steps, const double* n0, const double* eps0,
                     const double* u0, const void* state, hipStream_t s) {
  (void)n0;
  (void)K;
  (void)tape_steps;
  t.base = base;
  t.L = L;
  t.precision = precision;
  t.ncells = ncells;
  t.cs = cs;
  double* f = (double*)(base + L.off_fields);
  if (hipMemcpyAsync(f, eps0, sizeof(double) * ncells, hipMemcpyDeviceToDevice, s) != hipSuccess)
    return RLB_E_DEVICE;
  if (hipMemcpyAsync(f + ncells, u0, sizeof(double) * 3 * ncells, hipMemcpyDeviceToDevice, s) !=
      hipSuccess)
    return RLB_E_DEVICE;
  return tape_checkpoint(t, 0, state, s);
}

rlb_status tape_checkpoint(Tape& t, int64_t idx, const void* state, hipStream_t s) {
  if (idx < 0 || idx >= t.L.n_ckpt) return RLB_E_STATE;
  const char* g = (const char*)state + t.L.gbytes;  // 19 f planes precede the g planes
  char* dst = t.base + t.L.off_ckpt + (size_t)idx * t.L.gbytes;
  return hipMemcpyAsync(dst, g, t.L.gbytes, hipMemcpyDeviceToDevice, s) == hipSuccess
             ? RLB_OK
             : RLB_E_DEVICE;
}

rlb_status tape_grad(Tape& t, const GradContext& c, const double* dL_du, const double* dL_deps,
                     double dL_dtau[3], double* dL_deps0, double* dL_du0, int io_on_device) {
  if (!t.base) return RLB_E_STATE;
  const int64_t nc = c.ncells;
  const double *du = dL_du, *de = dL_deps;
  double *oe = dL_deps0, *ou = dL_du0;
  if (!io_on_device) {
    double* st = c.stage;
    if (hipMemcpyAsync(st, dL_du, sizeof(double) * 3 * nc, hipMemcpyHostToDevice, c.stream) !=
            hipSuccess ||
        hipMemcpyAsync(st + 3 * nc, dL_deps, sizeof(double) * nc, hipMemcpyHostToDevice,
                       c.stream) != hipSuccess)
      return RLB_E_DEVICE;
    du = st;
    de = st + 3 * nc;
    oe = st + 4 * nc;
    ou = st + 5 * nc;
  }
  rlb_status r = c.precision ? run_grad<float>(t, c, du, de, dL_dtau, oe, ou)
                             : run_grad<double>(t, c, du, de, dL_dtau, oe, ou);
  if (r != RLB_OK) return r;
  if (!io_on_device) {
    if (hipMemcpyAsync(dL_deps0, oe, sizeof(double) * nc, hipMemcpyDeviceToHost, c.stream) !=
            hipSuccess ||
        hipMemcpyAsync(dL_du0, ou, sizeof(double) * 3 * nc, hipMemcpyDeviceToHost, c.stream) !=
            hipSuccess ||
        hipStreamSynchronize(c.stream) != hipSuccess)
      return RLB_E_DEVICE;
  }
  return RLB_OK;
}

void tape_release(Tape& t) {
  for (hipEvent_t v : {t.recomputed, t.reversed})
    if (v) (void)hipEventDestroy(v);
  if (t.side) (void)hipStreamDestroy(t.side);
  t.recomputed = t.reversed = nullptr;
  t.side = nullptr;
  t.base = nullptr;
}

}  // namespace rlb
