// C ABI of the relativistic lattice Boltzmann library (include/rlb.h):
// argument validation, workspace carving, dispatch, autotuning.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/rlb.h"
#include "adjoint.hpp"
#include "internal.hpp"

using rlb::LatticeGeom;
using rlb::MemberDesc;

namespace {

constexpr size_t kAlign = 256;
// A single lattice at least this large takes the lattice path (one fused
// launch per step, or D2Q9 tile rounds); smaller lattices and batches take the
// persistent path (per-member kernels, segments, tube or strip rounds).
constexpr int64_t kLatticeMinCells = 16384;
// Double-buffered states up to this size are stored with plain stores.
constexpr size_t kCachedStateBytes = size_t(1) << 30;
// The last-level cache.
constexpr uint64_t kCacheBytes = uint64_t(256) << 20;
// Smallest z-plane and state of a lattice stored in blocks (blocked_layout).
constexpr int64_t kBlockedMinPlane = 1024;
constexpr uint64_t kBlockedMinState = uint64_t(128) << 20;
// Pad after each population plane (see make_layout).
constexpr int64_t kPlanePadBytes = 1280;
// Pad after each distribution's region of a blocked lattice.
constexpr int64_t kRegionPadBytes = 1280;

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

struct Layout {
  int64_t ncells = 0, cs = 0;
  rlb::StateLayout lay{};  // D3Q19 populations
  size_t esz = 0;
  size_t off_descs = 0, off_small = 0, off_bad = 0, off_partials = 0, off_xparts = 0,
         off_buf0 = 0, off_buf1 = 0;
  size_t off_stage = 0, off_segs = 0, off_flags = 0, off_tape = 0, total = 0;
  int max_parts = 0;
  int export_parts = 0;  // blocks of the field export (its own partials region)
  int blocks[rlb::kNumCells] = {};  // persistent path: blocks of a k_*_cells launch
  int64_t max_member = 0;           // cells of the largest member
  int ref_blocks = 0;               // blocks per member of the input pass
  int64_t max_segs = 0;  // persistent path: one segment per z-plane (D2Q9: per row) at most
  rlb::TapeLayout tape;
};

bool finite_tau(double t) { return std::isfinite(t) && t > 0.5; }

rlb_status check_members(const rlb_params* m, int32_t n, int64_t* ncells) {
  if (!m || n < 1) return RLB_E_ARG;
  int64_t tot = 0;
  for (int i = 0; i < n; ++i) {
    const rlb_params& p = m[i];
    if (p.nx < 1 || p.ny < 1 || p.nz < 1) return RLB_E_ARG;
    for (int k = 0; k < 3; ++k)
      if (p.bc[k] != RLB_PERIODIC && p.bc[k] != RLB_ZERO_GRADIENT) return RLB_E_ARG;
    const int64_t c = (int64_t)p.nx * p.ny * p.nz;
    if (c >= (int64_t(1) << 31)) return RLB_E_UNSUPPORTED;
    tot += c;
  }
  for (int i = 0; i < n; ++i) {
    const rlb_params& p = m[i];
    if (!finite_tau(p.tau_f) || !finite_tau(p.tau_v) || !finite_tau(p.tau_e) ||
        !finite_tau(p.tau_eps))
      return RLB_E_TAU;
    if (p.tau_q > 0.0 && !finite_tau(p.tau_q)) return RLB_E_TAU;
    if (std::isnan(p.tau_q)) return RLB_E_TAU;
    if (!std::isfinite(p.eta_over_s) || p.eta_over_s < 0.0) return RLB_E_ARG;
    if (!(p.eos_gamma == 0.0 || (p.eos_gamma > 1.0 && p.eos_gamma <= 2.0))) return RLB_E_ARG;
    if (!std::isfinite(p.mass) || p.mass < 0.0) return RLB_E_ARG;
    if (p.eta_over_s > 0.0) {
      if (!std::isfinite(p.kappa) || !(p.kappa > 0.0)) return RLB_E_ARG;
      if (!std::isfinite(p.dof) || !(p.dof > 0.0)) return RLB_E_ARG;
      for (double a : {p.a_f, p.a_e, p.a_eps, p.a_q})
        if (!std::isfinite(a) || a < 0.0) return RLB_E_ARG;
    }
  }
  *ncells = tot;
  return RLB_OK;
}

// The paper's equation of state P = eps/3 (Gamma 0 or 4/3, no rest mass)?
bool paper_eos(const rlb_params& p) {
  return (p.eos_gamma == 0.0 || p.eos_gamma == 4.0 / 3.0) && p.mass == 0.0;
}

bool lattice_path(int32_t n_members, int64_t ncells) {
  return n_members == 1 && ncells >= kLatticeMinCells;
}

// Velocities per distribution of a lattice kind.
int nvel(int32_t lattice) { return lattice == RLB_D2Q9 ? 9 : 19; }

// Is a D3Q19 lattice stored in blocks of 32 cells (StateLayout)? Its z-planes
// must be large enough that rounding them up to whole blocks costs at most 3 %
// of the memory, and small enough for 32-bit byte offsets within a plane. The
// adjoint reads its tape in planes. Blocks pay once a step is bound by memory
// (one-step kernels, planes against blocks: 96^3 FP32 47.6 and 43.1 us, 128^3
// FP64 237 and 218 us, 256^3 FP32 908 and 877 us); below about 128 MiB of
// double-buffered state the steps are bound by latency and the block
// arithmetic shows (40^3 FP64 9.4 and 9.9 us).
bool blocked_layout(const rlb_params& p, int32_t n, const rlb_options& o, int64_t ncells,
                    size_t esz) {
  const int64_t nxy = (int64_t)p.nx * p.ny;
  return o.lattice == RLB_D3Q19 && o.ckpt_every == 0 && lattice_path(n, ncells) &&
         nxy >= kBlockedMinPlane && 2 * 38 * (uint64_t)ncells * esz >= kBlockedMinState &&
         (uint64_t)(nxy + rlb::kBlock) * 19 * esz < (uint64_t(1) << 32);
}

// Tile geometry of a D2Q9 tile variant on an nx x ny lattice: halo cells a
// side (y doubled with the correction term), owned cells per tile and the
// grid. false when a tiled axis leaves no owned cell.
bool tile_geometry(const rlb::TileVariant& v, int nx, int ny, bool corr, rlb::TileRound& a,
                   dim3& grid) {
  a.hx = v.h;
  a.hy = corr ? 2 * v.h : v.h;
  a.ox = v.tx - 2 * a.hx;
  a.oy = v.ty - 2 * a.hy;
  if ((nx > v.tx && a.ox < 1) || (ny > v.ty && a.oy < 1)) return false;
  grid = dim3(nx <= v.tx ? 1 : (nx + a.ox - 1) / a.ox, ny <= v.ty ? 1 : (ny + a.oy - 1) / a.oy, 1);
  return true;
}

rlb_status make_layout(const rlb_params* m, int32_t n, const rlb_options* opt, Layout& L) {
  if (!opt) return RLB_E_ARG;
  if (opt->precision != RLB_FP32 && opt->precision != RLB_FP64) return RLB_E_ARG;
  if (opt->ckpt_every < 0 || opt->tape_steps < 0 || opt->diag_every < 0) return RLB_E_ARG;
  if (opt->lattice != RLB_D3Q19 && opt->lattice != RLB_D2Q9) return RLB_E_ARG;
  if (opt->correction != 0 && opt->correction != 1) return RLB_E_ARG;
  if (opt->correction && opt->lattice != RLB_D2Q9) return RLB_E_UNSUPPORTED;
  rlb_status st = check_members(m, n, &L.ncells);
  if (st != RLB_OK) return st;
  const bool d2 = opt->lattice == RLB_D2Q9;
  if (d2) {
    for (int i = 0; i < n; ++i)
      if (m[i].nz != 1) return RLB_E_ARG;
    if (opt->ckpt_every > 0) return RLB_E_UNSUPPORTED;  // the adjoint covers D3Q19
  }
  if (opt->ckpt_every > 0 && n != 1) return RLB_E_UNSUPPORTED;
  if (opt->ckpt_every > 0 && (m[0].eta_over_s > 0.0 || !paper_eos(m[0])))
    return RLB_E_UNSUPPORTED;  // the adjoint covers fixed taus and P = eps/3
  if (opt->correction)
    for (int i = 0; i < n; ++i)
      if (!paper_eos(m[i])) return RLB_E_UNSUPPORTED;  // C_7 is derived for P = eps/3
  L.esz = opt->precision == RLB_FP32 ? 4 : 8;
  // Plane stride: a multiple of 64 elements plus 1280 bytes, so that planes of
  // a power-of-two lattice do not all start alike on the HBM channels
  // (measured: 3-5 % faster at 256^3 than unpadded planes in both precisions,
  // and at 512^3 FP32 2 % faster than a 256-byte pad).
  L.cs = (L.ncells + 63) / 64 * 64 + kPlanePadBytes / (int64_t)L.esz;
  // every population byte offset of a plane is a 32-bit quantity in the kernels
  if ((uint64_t)L.cs * L.esz >= (uint64_t(1) << 32)) return RLB_E_UNSUPPORTED;
  int parts = std::max<int64_t>(n, (L.ncells + 255) / 256 > 65536 ? 65536 : (L.ncells + 255) / 256);
  if (lattice_path(n, L.ncells)) {
    LatticeGeom g{};
    g.nx = m[0].nx;
    g.ny = m[0].ny;
    g.nz = m[0].nz;
    if (d2) {
      for (int v = 0; v < rlb::d2q9_num_lattice_variants(); ++v)
        parts = std::max(parts, rlb::d2q9_lattice_partials(v, g));
      for (int v = 0; v < rlb::d2q9_num_tile_variants(); ++v) {
        rlb::TileRound a{};
        dim3 grid;
        if (tile_geometry(rlb::d2q9_tile_variant(v), g.nx, g.ny, opt->correction != 0, a, grid))
          parts = std::max<int64_t>(parts, (int64_t)grid.x * grid.y);
      }
    }
    else
      for (int v = 0; v < rlb::num_lattice_variants(); ++v)
        parts = std::max(parts, rlb::lattice_partials(v, g));
  }
  for (int i = 0; i < n; ++i)
    L.max_member = std::max(L.max_member, (int64_t)m[i].nx * m[i].ny * m[i].nz);
  L.ref_blocks = rlb::ref_blocks(L.max_member);
  parts = std::max<int64_t>(parts, (int64_t)n * L.ref_blocks);
  if (!lattice_path(n, L.ncells)) {  // segment tables of the persistent path
    // D3Q19: segments of whole z-planes (at most nz per member); D2Q9 strip
    // rounds: segments of whole rows (at most ny per member)
    for (int i = 0; i < n; ++i) L.max_segs += d2 ? m[i].ny : m[i].nz;
    parts = std::max<int64_t>(parts, L.max_segs);
    for (int i = 0; i < n; ++i) {
      const int64_t c = (int64_t)m[i].nx * m[i].ny * m[i].nz;
      L.blocks[0] += (int)((c + 63) / 64);
      L.blocks[1] += (int)((c + 255) / 256);
    }
    parts = std::max<int64_t>(parts, L.blocks[0]);
  }
  L.max_parts = std::max(parts, 1);
  size_t o = 0;
  L.off_descs = o;
  o = align_up(o + sizeof(MemberDesc) * n);
  L.off_small = o;
  o = align_up(o + 1024);
  L.off_bad = o;  // the inadmissible-cell slots and their copy kept across tuning trials
  o = align_up(o + 2 * rlb::kBadBytes);
  L.off_partials = o;
  o = align_up(o + sizeof(double) * 5 * (size_t)L.max_parts);
  // The field export keeps its partial sums apart, so that rlb_moments never
  // overwrites the diagnostics partials of the latest step.
  L.export_parts = rlb::export_blocks(L.ncells);
  L.off_xparts = o;
  o = align_up(o + sizeof(double) * 5 * (size_t)L.export_parts);
  size_t buf = 2 * (size_t)nvel(opt->lattice) * (size_t)L.cs * L.esz;
  const int64_t nxy = (int64_t)m[0].nx * m[0].ny;
  L.lay = rlb::plane_layout(L.cs, n == 1 ? (uint32_t)nxy : 1u);
  if (blocked_layout(m[0], n, *opt, L.ncells, L.esz)) {
    L.lay.shift = rlb::kBlockShift;
    L.lay.nxy = (uint32_t)nxy;
    L.lay.zcells = (uint32_t)((nxy + rlb::kBlock - 1) / rlb::kBlock * rlb::kBlock);
    L.lay.pstr = rlb::kBlock;
    L.lay.bextra = 18 * rlb::kBlock;
    L.lay.greg = (int64_t)L.lay.zcells * m[0].nz * 19 + kRegionPadBytes / (int64_t)L.esz;
    buf = 2 * (size_t)L.lay.greg * L.esz;
  }
  L.off_buf0 = o;
  o = align_up(o + buf);
  L.off_buf1 = o;
  o = align_up(o + buf);
  L.off_stage = o;
  o = align_up(o + sizeof(double) * 8 * (size_t)L.ncells);
  L.off_segs = o;
  o = align_up(o + std::max(sizeof(rlb::Segment), sizeof(rlb::TubeSeg)) * (size_t)L.max_segs);
  L.off_flags = o;
  o = align_up(o + sizeof(unsigned long long) * (size_t)L.max_segs);
  L.off_tape = o;
  if (opt->ckpt_every > 0) {
    L.tape = rlb::tape_layout(m[0].nx, m[0].ny, m[0].nz, L.cs, L.esz, opt->ckpt_every,
                              opt->tape_steps, L.max_parts);
    o = align_up(o + L.tape.total);
  }
  L.total = o;
  return RLB_OK;
}

struct DeviceGuard {
  int prev = -1;
  bool ok = true;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) {
      ok = false;
      return;
    }
    if (prev != dev && hipSetDevice(dev) != hipSuccess) ok = false;
  }
  ~DeviceGuard() {
    int cur;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

}  // namespace

struct rlb_sim {
  int device = 0;
  hipStream_t stream = nullptr;
  int precision = RLB_FP32;
  rlb_options opt{};
  int n_members = 0;
  std::vector<rlb_params> params;
  std::vector<MemberDesc> descs;  // host copy, refs filled at init
  Layout L;
  char* ws = nullptr;
  MemberDesc* d_descs = nullptr;
  double* d_small = nullptr;  // the host's view, then the gradient's sums
  unsigned long long* d_bad = nullptr;
  rlb::HostView* d_view = nullptr;  // what the host reads back, in one copy
  unsigned long long* d_bad_save = nullptr;
  double* d_partials = nullptr;
  double* d_xparts = nullptr;  // export partials (rlb_moments)
  void* buf[2] = {nullptr, nullptr};
  double* d_stage = nullptr;
  int cur = 0;
  bool d2 = false;  // D2Q9 model (9 velocities, 18 planes per buffer)
  bool corr = false;  // D2Q9 with the correction term of Eqs. (37)-(38)
  bool eos = false;    // some member has a general equation of state
  bool ext = false;    // some member takes its relaxation times from eta/s per cell or
                       // has the general equation of state (the EXT kernels)
  int q = 19;
  bool lattice = false;
  LatticeGeom geom{};
  rlb::MarchGrid march{};  // blocked D3Q19 lattices
  int variant = 0;
  int64_t steps = 0;
  int64_t diag_step = -1;
  int diag_parts = 0;
  // persistent kernels
  rlb::MemberLaunch margs{};
  rlb::SegLaunch sargs{};
  rlb::Segment* d_segs = nullptr;
  unsigned long long* d_flags = nullptr;
  unsigned long long epoch = 0;  // steps every segment flag holds
  int seg_built = -1;             // variant the device segment table describes (segments:
                                  // sv; tube rounds: 1000 + tv; strip rounds: 2000 + sv)
  bool seg_whole = false;         // tube or strip segments: every member is one, whole
  int seg_halo = 0;               // else the steps of a round
  bool all_tubes = false;
  int nseg = 0;
  int num_cu = 0;
  // tape
  rlb::Tape tape{};
  bool tape_ok = false;
};

namespace {

rlb_status dev_err(hipError_t e) { return e == hipSuccess ? RLB_OK : RLB_E_DEVICE; }

#define RLB_HIP(call)                              \
  do {                                             \
    hipError_t _e = (call);                        \
    if (_e != hipSuccess) return RLB_E_DEVICE;     \
  } while (0)

void* state_buf(rlb_sim* h) { return h->buf[h->cur]; }
void* spare_buf(rlb_sim* h) { return h->buf[1 - h->cur]; }

// The host's view, once the stream has reached it.
rlb_status read_view(rlb_sim* h, rlb::HostView* v) {
  RLB_HIP(hipMemcpyAsync(v, h->d_view, sizeof(*v), hipMemcpyDeviceToHost, h->stream));
  RLB_HIP(hipStreamSynchronize(h->stream));
  return RLB_OK;
}

rlb_status launch_lattice_step(rlb_sim* h, int variant, bool diag, const void* src, void* dst) {
  if (h->d2)
    return dev_err(rlb::d2q9_launch_step_lattice(h->precision, variant, diag, h->corr, h->ext,
                                                 src, dst, h->geom, h->d_partials, h->d_bad,
                                                 h->stream));
  return dev_err(rlb::launch_step_lattice(h->precision, variant, diag, h->ext, src, dst, h->geom,
                                          h->d_partials, h->d_bad, h->stream));
}

// One-step blocks of a corrected D2Q9 lattice: 64 x 4, which share the neighbours'
// fields, or 128 x 2 where rows begin off the memory's granules and the state is far
// out of the caches. us a step, 64 x 4, 128 x 2 and 256 x 1 blocks: 1531 x 1203 FP64
// 130, 137, 140, FP32 56, 71, 73, 2048^2 FP32 130, 140, 152, 1500 x 4000 211, 240, 235;
// 1082 x 2685 FP64 222, 206, 210, FP32 125, 124, 123, 1906 x 1500 FP64 224, 202, 205,
// FP32 125, 121, 118, 2925 x 2045 FP32 259, 240, 240.
int corrected_blocks(const rlb_sim* h) {
  const rlb_params& p = h->params[0];
  return p.nx % 4 != 0 && (int64_t)p.nx * p.ny > 2500000 ? 4 : 3;
}

// Marching variants (D3Q19: two steps per launch, D2Q9: H); steps that do not
// fill a launch (the last of a call, diagnostics steps) run a one-step kernel, in
// blocks as the rows are long. us a step, 128 x 2, 64 x 4 and 256 x 1 blocks: D3Q19
// 96^3 FP32 44, 47, 44, 160^3 245, 213, 208, 187 x 150 x 131 339, 319, 343, 256^3 880,
// 874, 885; D2Q9, the last two: 300^2 FP64 6.4 and 8.2, 700 x 500 FP32 11.9 and 10.8,
// 1000 x 800 22.8 and 20.9, 1531 x 1203 FP64 122 and 117, 219 x 4482 65 and 57, 2048^2
// 223 and 226, 200^2 4.5 and 5.0; with the correction corrected_blocks.
int march_step(const rlb_sim* h) {
  const rlb_params& p = h->params[0];
  if (!h->d2) return p.nx > 64 && p.nx <= 128 ? 2 : 1;
  const auto lanes = [&](int bx) { return (p.nx + bx - 1) / bx * bx; };  // of a row
  const bool idle = 5 * lanes(256) > 6 * lanes(64) || (int64_t)p.nx * p.ny < 65536;
  return h->corr ? corrected_blocks(h) : idle ? 3 : 2;
}

int march_base(const rlb_sim* h) {
  return h->d2 ? rlb::d2q9_num_lattice_variants() + rlb::d2q9_num_tile_variants()
               : rlb::num_lattice_variants();
}

bool is_march_variant(const rlb_sim* h, int v) { return h->lattice && v >= march_base(h); }

// Where a marching variant cannot launch (D3Q19 lattices stored in planes;
// D2Q9: fewer columns between faces than a wave has, or few rows) it runs its
// steps one by one.
bool can_march(const rlb_sim* h) {
  if (h->d2) return rlb::d2q9_march_fits(h->geom);
  return h->L.lay.shift == rlb::kBlockShift;
}

int march_steps(const rlb_sim* h, int v) {
  if (!can_march(h)) return 1;
  return h->d2 ? rlb::d2q9_march_steps(v - march_base(h), h->corr) : 2;
}

// The launch that comes next of m steps in a row: a marching variant, or -1 for a
// single step. D2Q9 lattices without the correction have launches of 4 and of 3
// steps and mix them where that leaves no single step over (any m but 1, 2, 5):
// one costs about as much as two steps of a launch (4096^2 FP32: 4 steps 0.79 ms, 3
// steps 0.73, one 0.43; 30 steps as 7 x 4 + 2 6.4 ms, as 6 x 4 + 2 x 3 6.2).
int next_march(const rlb_sim* h, int64_t m) {
  const int per = march_steps(h, h->variant);
  if (per < 2) return -1;
  if (!h->d2 || h->corr) return m >= per ? h->variant : -1;
  const auto whole = [](int64_t r) { return r >= 0 && r != 1 && r != 2 && r != 5; };
  const int other = 2 * march_base(h) + 1 - h->variant;
  if (whole(m - per)) return h->variant;
  if (whole(m - march_steps(h, other))) return other;
  return m >= 4 ? march_base(h) : m == 3 ? march_base(h) + 1 : -1;
}

// The marching variant that is the default from a share `use` of used cells of
// its grid on (MarchGrid::use). us a step, marching and best one-step kernel:
// D3Q19: 40 x 40 x 400 FP32 (use 0.42) 40.5 and 32.7, 80^3 FP32 (0.59) 25.2 and
// 27.4, 64^3 FP64 (0.65) 22.1 and 25.2; eta/s: 60^3 FP64 (0.71) 23.1 and 22.2,
// 96^3 FP32 (0.74) 43.9 and 44.0, 160^3 FP32 (0.79) 205 and 207, 128^3 FP32 (0.85)
// 100 and 114, 80^3 FP64 (0.79) 52 and 60.
// D2Q9: 700 x 500 FP32 (0.33) 10.1 and 10.3, 300^2 FP32 (0.08) 7.3 and 5.9, 1000 x
// 800 FP32 (0.52) 15 and 20. eta/s, where 3 steps a launch do as well as 4 at
// 2000 x 1800 and better below: FP32 1000 x 800 (0.54) 23.3 and 21.0, 1100 x 900
// (0.62) 25.6 and 26.4; FP64 500 x 400 (0.36) 11.2 and 11.3, 700 x 500 (0.57) 13.0
// and 17.3. With the correction: 1000 x 800 FP32 (0.53) 26 and 25, 1531 x 1203 FP32
// (0.69) 45 and 50, 300^2 FP64 (0.18) 14 and 9, 700 x 500 FP64 (0.55) 18 and 21; and
// eta/s: FP64 1000 x 800 (0.63) 39.9 and 39.9, 1400 x 1000 (0.79) 59 and 92; FP32 2000 x
// 1800 (0.82) 140 and 111 (one wave per SIMD: never the default). A general
// equation of state repeats its root search in the halos: a higher share.
struct MarchDefault {
  int variant;
  double least_use;
};

MarchDefault march_default(const rlb_sim* h) {
  const bool fp32 = h->precision == RLB_FP32;
  if (!h->d2) return {0, !h->ext ? 0.6 : h->eos ? 0.8 : 0.72};
  if (h->corr) return {0, !h->ext ? (fp32 ? 0.6 : 0.5) : fp32 ? 2.0 : 0.7};
  if (!h->ext) return {0, 0.35};
  return {1, h->eos ? 0.7 : fp32 ? 0.56 : 0.45};
}

rlb_status launch_march(rlb_sim* h, int variant, const void* src, void* dst) {
  const int v = variant - march_base(h);
  if (h->d2)
    return dev_err(rlb::d2q9_launch_march(h->precision, v, h->corr, h->ext, src, dst, h->geom, h->num_cu,
                                          h->d_bad, h->stream));
  return dev_err(rlb::launch_step_march(h->precision, v, h->ext, src, dst, h->geom, h->march,
                                        h->d_bad, h->stream));
}

bool is_tile_variant(const rlb_sim* h, int v) {
  return h->lattice && h->d2 && v >= rlb::d2q9_num_lattice_variants() && !is_march_variant(h, v);
}

int tile_index(int v) { return v - rlb::d2q9_num_lattice_variants(); }

int lattice_parts(const rlb_sim* h, int variant) {
  if (is_tile_variant(h, variant)) {
    rlb::TileRound a{};
    dim3 grid;
    tile_geometry(rlb::d2q9_tile_variant(tile_index(variant)), h->geom.nx, h->geom.ny, h->corr,
                  a, grid);
    return (int)(grid.x * grid.y);
  }
  if (is_march_variant(h, variant)) variant = march_step(h);
  return h->d2 ? rlb::d2q9_lattice_partials(variant, h->geom)
               : rlb::lattice_partials(variant, h->geom);
}

// The steps left over by rounds on `tiles` windows, 1 or 2 of 3, that run one by one
// instead, and their kernel. us a step, as a round and singly: one step of 128^2
// FP32 6.7 and 5.1, of 300^2 9.9 and 6.5, FP64 11.2 and 8.3; two steps of 300^2 FP32
// (346 windows, 256 CUs) 6.1 and 6.4, 450^2 (779) 9.1 and 8.9, 550^2 (1163) 11.1 and
// 10.2; FP64 300^2 6.8 and 8.1, 550^2 14.5 and 15.8.
int tile_singles(const rlb_sim* h, int64_t tiles, int left) {
  if (left == 2 && h->precision == RLB_FP32 && tiles > 4 * h->num_cu) return 2;
  return left == 1 ? 1 : 0;
}

int tile_single(const rlb_sim* h) { return h->corr ? corrected_blocks(h) : 2; }

// D2Q9 tile rounds: ceil(n / H) launches, each advancing up to H steps of the
// whole lattice; rounds alternate the buffers (pingpong) or always read a and
// write b (trials). *flip tells whether the state changed buffers.
rlb_status launch_tile_rounds(rlb_sim* h, int variant, int nsteps, int pingpong, void* a, void* b,
                              int diag_every, int64_t step0, bool* flip) {
  const rlb::TileVariant v = rlb::d2q9_tile_variant(tile_index(variant));
  rlb::TileRound arg{};
  dim3 grid;
  if (!rlb::d2q9_tile_fits(h->precision, tile_index(variant), h->corr) ||
      !tile_geometry(v, h->geom.nx, h->geom.ny, h->corr, arg, grid))
    return RLB_E_UNSUPPORTED;
  arg.cs = h->L.cs;
  arg.nx = h->geom.nx;
  arg.ny = h->geom.ny;
  arg.bcx = h->geom.bcx;
  arg.bcy = h->geom.bcy;
  arg.diag_every = diag_every;
  arg.last_step = step0 + nsteps;
  arg.rt = h->geom.rt;
  arg.ref = h->geom.ref;
  arg.ext = h->geom.ext;
  arg.partials = h->d_partials;
  arg.bad = h->d_bad;
  const int singles = pingpong ? tile_singles(h, (int64_t)grid.x * grid.y, nsteps % v.h) : 0;
  const int rounds = (nsteps - singles + v.h - 1) / v.h;
  for (int r = 0; r < rounds + singles; ++r) {
    const bool odd = pingpong && (r & 1);
    arg.src = odd ? b : a;
    arg.dst = odd ? a : b;
    if (r >= rounds) {
      const bool diag = diag_every > 0 && r + 1 == rounds + singles;  // the step of the call kept
      rlb_status st = launch_lattice_step(h, tile_single(h), diag, arg.src, arg.dst);
      if (st != RLB_OK) return st;
      continue;
    }
    arg.nsteps = std::min(v.h, nsteps - r * v.h);
    arg.step0 = step0 + (int64_t)r * v.h;
    RLB_HIP(rlb::d2q9_launch_tiles(h->precision, tile_index(variant), h->corr, h->ext, arg, grid,
                                   h->stream));
  }
  *flip = pingpong && ((rounds + singles) & 1);
  if (pingpong && diag_every > 0) {
    h->diag_step = step0 + nsteps;
    h->diag_parts = lattice_parts(h, singles ? tile_single(h) : variant);
  }
  return RLB_OK;
}

// Default of the lattice path where nothing marches. us a step by the choice and
// by 256 x 1 blocks:
//   D3Q19: 64 x 4 blocks, 26^3 FP32 5.3 and 6.1, 60^3 12.4 and 15.6, 31 x 31 x 300
//     19.6 and 27.4, 512 x 512 the same; rows of 65 to 128 cells 128 x 2 blocks, 66^3
//     18.6 and 21.5 (64 x 4 21.6), 80^3 with eta/s 28.0 and 32.7;
//   D2Q9: rounds of 3 steps on 32 x 16 windows, 110 x 160 FP32 2.8 and 3.7, 300^2 4.6
//     and 6.0, 550^2 8.7 and 10.1, FP64 3.2 and 4.2, 5.1 and 8.0, 10.9 and 15.7. With
//     eta/s or the correction, whose halos cost more, only while every window finds
//     a CU: eta/s 250^2 FP32 4.1 and 5.3, 270 x 260 7.3 and 6.5; correction 150^2
//     FP64 4.3 and 5.8, 250^2 10.0 and 9.4; else corrected_blocks with the
//     correction, and 256 x 1. No tiles either where a window is less than half full of rows
//     (100000 x 4 FP32 17.0 and 11.7, x 7 11.5 and 10.5; one row with the correction
//     100000 x 1 7.4 in 64 x 4 blocks and 6.5), nor in FP32 with more than 5
//     windows a CU (700 x 500, 1350, 10.1 and 10.4) or, with diagnostics at every
//     step or two, which end a round's arithmetic in sums, with more than 2 (at every
//     step 550^2, 1163 windows, 13.9 and 11.2, 300^2, 346, 6.8 and 7.5; FP64 550^2
//     16.4 and 16.8).
int default_lattice(const rlb_sim* h) {
  const rlb_params& p = h->params[0];
  if (!h->d2) return p.nx > 64 && p.nx <= 128 ? 2 : 1;
  const int tv = 6;
  const rlb::TileVariant v = rlb::d2q9_tile_variant(tv);
  const bool often = h->opt.diag_every == 1 || h->opt.diag_every == 2;
  const int64_t per_cu = h->ext || h->corr          ? 1
                         : h->precision == RLB_FP64 ? INT32_MAX
                         : often                    ? 2
                                                    : 5;
  rlb::TileRound a{};
  dim3 grid;
  if (2 * p.ny >= v.ty && rlb::d2q9_tile_fits(h->precision, tv, h->corr) &&
      tile_geometry(v, p.nx, p.ny, h->corr, a, grid) &&
      (int64_t)grid.x * grid.y <= per_cu * h->num_cu)
    return rlb::d2q9_num_lattice_variants() + tv;
  return h->corr && p.ny > 1 ? corrected_blocks(h) : 2;
}

constexpr int kSpinLimit = 1 << 24;  // about a second of polling per wait

bool is_segment_variant(const rlb_sim* h, int v) {
  return !h->lattice && !h->d2 && v >= rlb::num_member_variants() &&
         v < rlb::num_member_variants() + rlb::num_segment_variants();
}

// Default of the persistent path. us a step, the choice against the one-block
// member kernel (512 threads), which keeps members of up to 1024 cells, one or two
// passes of its block (9^3 FP32 6.4 against 4.1, but 300 of 10^3 16 and 19):
//   1 x 1 x L tubes: rounds. Windows of 128 cells with a thread per distribution,
//     up to 32 steps a round, while their segments are few, and for tubes that one
//     window holds; else windows of 256 cells, up to 16 steps. The first and the
//     second: 800 cells FP64 1.2 and 1.7 (member kernel 9.3), 24 of 800 FP32 1.3 and
//     1.9, 30 of up to 1500 the same, 100 of up to 1300 3.1 and 2.8, 64 of up to 3200
//     4.3 and 3.8; eta/s FP64 40 of 400 1.9 and 2.2, FP32 64 of up to 1500 4.1 and
//     3.5; 1500 tubes of 100 cells FP64 4.2 and 5.8;
//   narrow D2Q9 members: strip rounds (default_strip), if windows of 256 cells
//     leave an owned row; 4 x 800 FP32 1.6 and 9.4, with the correction 2.0 and 20;
//   batches of members of a few passes: the member kernel (members_fill_the_chip);
//   the rest: one launch per step; 16^3 FP32 3.8 and 29, 24^3 4.2 and 115, 120^2
//     D2Q9 3.3 and 41. Blocks of 64 cells until they fill the chip: D3Q19, where
//     they run a thread per distribution, 864 blocks FP64 9.6 us and 10.2 of
//     256-cell blocks, 1728 blocks FP64 15.1 and 12.9, FP32 10.0 and 10.2; D2Q9
//     up to 4096 blocks.
constexpr int64_t kMemberCells = 1024, kStripCells = 256;

int cells_base(const rlb_sim* h);

// Tube segments with windows of nt cells and `halo` of them a side.
int64_t tube_segments(const rlb_sim* h, int nt, int halo) {
  int64_t n = 0;
  for (const rlb_params& p : h->params)
    n += p.nz <= nt ? 1 : (p.nz + nt - 2 * halo - 1) / (nt - 2 * halo);
  return n;
}

// Steps of a tube variant's rounds: H, or less (down to half) where that saves
// the fullest CU a segment: a round waits for it, while a launch costs as much as
// two steps. 64 tubes of up to 3200 cells, FP32, 256 CUs: 521 segments at H = 16,
// 509 at 14: 3.45 and 3.15 us a step, start and fields included.
int tube_halo(const rlb_sim* h, const rlb::TubeVariant& v) {
  const auto fullest = [&](int halo) {
    return (tube_segments(h, v.nt, halo) + h->num_cu - 1) / h->num_cu;
  };
  int halo = v.halo;
  while (halo > v.halo / 2 && fullest(halo) > fullest(v.halo / 2)) --halo;
  return halo;
}

// The split windows up to two segments per CU (one in the extended model, where
// both threads of a cell work out its rates), as tube_halo would cut them; else 1.
int default_tube(const rlb_sim* h) {
  const int64_t most = (int64_t)h->num_cu * (h->ext ? 1 : 2);
  for (const int v : {6, 5}) {
    const rlb::TubeVariant t = rlb::tube_variant(v);
    if (h->L.max_member <= t.nt || tube_segments(h, t.nt, t.halo / 2) <= most) return v;
  }
  return 1;
}

// Strip segments with windows of nt cells and rounds of `halo` steps; 0 where a
// window owns no row.
int64_t strip_segments(const rlb_sim* h, int nt, int halo) {
  int64_t n = 0;
  for (const rlb_params& p : h->params) {
    const int R = nt / p.nx, S = R - 2 * halo * (h->corr ? 2 : 1);
    if (p.ny > R && S < 1) return 0;
    n += p.ny > R ? (p.ny + S - 1) / S : 1;
  }
  return n;
}

// Steps of a strip variant's rounds: H, or up to twice as many while windows with
// that halo own a row and the fullest CU gets no segment more: a launch costs as
// much as two steps (eta/s, FP64, by 8 and 16 steps of 256 threads: 4 members of 4
// x 800 cells, 100 segments, 1.9 and 1.6 us a step; 12 of them, 300 segments, 2.0
// and 2.4: they take 12 steps, 1.9).
int strip_halo(const rlb_sim* h, const rlb::TubeVariant& v) {
  const auto fullest = [&](int halo) {  // 0: some window owns no row
    return (strip_segments(h, v.nt, halo) + h->num_cu - 1) / h->num_cu;
  };
  int halo = 2 * v.halo;
  while (halo > v.halo && (fullest(halo) == 0 || fullest(halo) > fullest(v.halo))) --halo;
  return halo;
}

// Strip variant of a batch of narrow members, -1 where windows of 256 cells leave
// no owned row. Those windows while each segment has a CU; beyond, windows of 512
// cells where they compute fewer cells, which wide members need: a window of nx
// cells a row owns 256 / nx - 16 rows (15 x 500, one: 17 times the work). us a
// step by 256 and 512 cells, and the member kernel: 16 of 15 x 500 FP64 20.9, 4.0 and
// 35; 256 of 15 x 100 FP32 50, 7.8 and 8.8; 64 of 12 x 500 FP32 13.9, 7.0 and 20;
// 256 of 4 x 100, whole in 512 cells, FP32 2.6, 1.7 and 2.2. By how much fewer: the
// larger blocks lose more registers with eta/s or the correction, 64 of 7 x 500 (0.72
// of the cells) eta/s FP64 8.2 and 8.6, but 64 of 10 x 500 (0.53) 13.8 and 10.5.
// FP32 with eta/s takes rounds of 4 steps instead, whose halos are half as wide: 128
// of 15 x 500 208 by 8 steps, 29.9 by 4, 36.9 by the windows of 512 cells; 256 of 10
// x 500 48, 30 and 40.
int default_strip(const rlb_sim* h) {
  const int small = 3, large = h->precision == RLB_FP32 && h->ext && h->L.max_member > 512 ? 2 : 4;
  const rlb::TubeVariant s = rlb::d2q9_strip_variant(small), l = rlb::d2q9_strip_variant(large);
  const int rows = 2 * s.halo * (h->corr ? 2 : 1) + 1;
  for (const rlb_params& p : h->params)
    if ((int64_t)p.nx * rows > s.nt) return -1;
  const int64_t ns = strip_segments(h, s.nt, s.halo), nl = strip_segments(h, l.nt, l.halo);
  const double fewer = h->ext || h->corr ? 0.7 : 0.9;
  return ns > h->num_cu && nl * l.nt < fewer * ns * s.nt ? large : small;
}

// Is the one-block member kernel better than one launch per step? It takes
// max_member cells in passes of 512, all members at once where they are as many as
// the CUs, and keeps a member's populations near its CU; a launch per step
// spreads the cells over the chip and streams them all. us a step by member kernel
// and launches (256 CUs; 11^3 is 3 passes, 13^3 5, 16^3 and 64^2 8, 40^2 4):
//   D3Q19 FP32: 128 of 11^3 16 and 13, 192 17 and 18, 1024 71 and 119; 256 of 13^3 29
//     and 34, of 16^3 81 and 66; eta/s, from where a step no longer streams from the
//     last-level cache: 512 of 11^3 (198 MiB of state) 47 and 40, 768 (296) 72 and
//     81, 512 of 13^3 (326) 72 and 84;
//   FP64: 64 of 11^3 15 and 13, 96 16 and 17, 1024 135 and 193; 128 of 13^3 27 and 32;
//     256 of 16^3 124 and 136, 384 206 and 191, 512 253 and 265; eta/s the same;
//   D2Q9: 64 of 40^2 FP32 5.4 and 7.3, FP64 7.9 and 8.7; 256 of 64^2 FP32 21 and 26,
//     FP64 47 and 55; one of 33 x 32 FP32 4.0 and 4.8; eta/s FP32 128 of 40^2 11.4
//     and 10.4, 256 12 and 14, 512 26 and 24, of 33 x 32 15 and 18; correction: 128
//     of 40^2 FP32 11.8 and 13.7, FP64 14 and 18, eta/s FP32 256 18 and 19.
bool members_fill_the_chip(const rlb_sim* h) {
  const auto passes_of = [](int64_t cells) { return (cells + 511) / 512; };
  const int64_t passes = passes_of(h->L.max_member);
  int64_t total = 0;
  for (const MemberDesc& d : h->descs) total += passes_of(d.ncells);
  // members, were they all as large as the largest, per CU
  const double load = (double)total / passes / h->num_cu;
  const bool fp32 = h->precision == RLB_FP32;
  if (fp32 && h->ext) {
    if (!h->d2)
      return passes <= 5 && 2 * 38 * sizeof(float) * (uint64_t)h->L.ncells > kCacheBytes;
    return passes <= (h->corr ? 4 : 5) && load >= 0.75 &&
           load <= (!h->corr && passes <= 3 ? 2.0 : 1.0);
  }
  if (h->d2 && !h->corr) {
    if (fp32) return passes <= 3 || (passes <= 16 && load >= (passes <= 5 ? 0.25 : 0.5));
    return passes <= 8 && load >= (passes <= 4 ? 0.25 : passes <= 5 ? 0.375 : 0.5);
  }
  if (passes <= 5) return load >= (fp32 && (!h->d2 || passes == 5) ? 0.75 : 0.375);
  return !fp32 && passes <= 8 && std::ceil(load) - load <= 0.25;  // no CU waits for another
}

int default_persistent(const rlb_sim* h) {
  if (h->all_tubes)
    return rlb::num_member_variants() + rlb::num_segment_variants() + default_tube(h);
  if (h->d2 && h->L.max_member > kStripCells) {
    const int v = default_strip(h);
    if (v >= 0) return rlb::d2q9_num_member_variants() + v;
  }
  if (h->L.max_member <= kMemberCells || members_fill_the_chip(h)) return 1;
  return cells_base(h) + (h->L.blocks[0] <= rlb::small_blocks(h->d2) ? 0 : 1);
}

// First of the one-launch-per-step variants, which follow the others.
int cells_base(const rlb_sim* h) {
  return h->d2 ? rlb::d2q9_num_member_variants() + rlb::d2q9_num_strip_variants()
               : rlb::num_member_variants() + rlb::num_segment_variants() +
                     rlb::num_tube_variants();
}

bool is_cells_variant(const rlb_sim* h, int v) { return !h->lattice && v >= cells_base(h); }

bool is_tube_variant(const rlb_sim* h, int v) {
  return !h->lattice && !h->d2 && !is_cells_variant(h, v) &&
         v >= rlb::num_member_variants() + rlb::num_segment_variants();
}

int tube_index(int v) { return v - rlb::num_member_variants() - rlb::num_segment_variants(); }

bool is_strip_variant(const rlb_sim* h, int v) {
  return !h->lattice && h->d2 && !is_cells_variant(h, v) &&
         v >= rlb::d2q9_num_member_variants();
}

int strip_index(int v) { return v - rlb::d2q9_num_member_variants(); }

// Tube segments for a tube variant: owned ranges of at most NT - 2H cells,
// windows extended by H halo cells (cut at zero-gradient ends); a tube that
// fits the block whole is one segment with exact ends.
rlb_status build_tube_segments(rlb_sim* h, int tv, std::vector<rlb::TubeSeg>& segs) {
  rlb::TubeVariant v = rlb::tube_variant(tv);
  v.halo = tube_halo(h, v);
  const int S = v.nt - 2 * v.halo;
  for (int m = 0; m < h->n_members; ++m) {
    const MemberDesc& d = h->descs[m];
    const int L = d.nz;
    const bool periodic = d.bcz == RLB_PERIODIC;
    if (L <= v.nt) {
      const int kind = periodic ? rlb::kEdgeWrap : rlb::kEdgeClamp;
      segs.push_back(rlb::TubeSeg{m, 0, L, 0, L, kind, kind});
      continue;
    }
    const int n = (L + S - 1) / S;
    for (int j = 0; j < n; ++j) {
      rlb::TubeSeg g{};
      g.member = m;
      g.own0 = (int)((int64_t)L * j / n);
      g.own1 = (int)((int64_t)L * (j + 1) / n);
      if (periodic) {
        g.win0 = g.own0 - v.halo;
        g.wlen = g.own1 - g.own0 + 2 * v.halo;
        g.left = g.right = rlb::kEdgeHalo;
      } else {
        g.win0 = std::max(0, g.own0 - v.halo);
        const int win1 = std::min(L, g.own1 + v.halo);
        g.wlen = win1 - g.win0;
        g.left = g.win0 == 0 ? rlb::kEdgeClamp : rlb::kEdgeHalo;
        g.right = win1 == L ? rlb::kEdgeClamp : rlb::kEdgeHalo;
      }
      segs.push_back(g);
    }
  }
  if ((int64_t)segs.size() > h->L.max_segs) return RLB_E_ARG;
  RLB_HIP(hipMemcpyAsync(h->d_segs, segs.data(), sizeof(rlb::TubeSeg) * segs.size(),
                         hipMemcpyHostToDevice, h->stream));
  h->nseg = (int)segs.size();
  h->seg_whole = h->nseg == h->n_members;  // a cut member has two or more
  h->seg_halo = v.halo;
  h->seg_built = 1000 + tv;
  return RLB_OK;
}

// D2Q9 strip segments for a strip variant: windows of R = nt / nx rows, H
// halo rows a side (2H with the correction term), owned ranges of at most
// R - 2H rows; a member of at most R rows is one segment with exact ends.
// RLB_E_UNSUPPORTED when a member is wider than the block or leaves no
// owned row.
rlb_status build_strip_segments(rlb_sim* h, int sv, std::vector<rlb::TubeSeg>& segs) {
  rlb::TubeVariant v = rlb::d2q9_strip_variant(sv);
  v.halo = strip_halo(h, v);
  const int hr = h->corr ? 2 * v.halo : v.halo;
  for (int m = 0; m < h->n_members; ++m) {
    const MemberDesc& d = h->descs[m];
    if (d.nx > v.nt) return RLB_E_UNSUPPORTED;
    const int R = v.nt / d.nx;
    const int L = d.ny;
    const bool periodic = d.bcy == RLB_PERIODIC;
    if (L <= R) {
      const int kind = periodic ? rlb::kEdgeWrap : rlb::kEdgeClamp;
      segs.push_back(rlb::TubeSeg{m, 0, L, 0, L, kind, kind});
      continue;
    }
    const int S = R - 2 * hr;
    if (S < 1) return RLB_E_UNSUPPORTED;
    const int n = (L + S - 1) / S;
    for (int j = 0; j < n; ++j) {
      rlb::TubeSeg g{};
      g.member = m;
      g.own0 = (int)((int64_t)L * j / n);
      g.own1 = (int)((int64_t)L * (j + 1) / n);
      if (periodic) {
        g.win0 = g.own0 - hr;
        g.wlen = g.own1 - g.own0 + 2 * hr;
        g.left = g.right = rlb::kEdgeHalo;
      } else {
        g.win0 = std::max(0, g.own0 - hr);
        const int win1 = std::min(L, g.own1 + hr);
        g.wlen = win1 - g.win0;
        g.left = g.win0 == 0 ? rlb::kEdgeClamp : rlb::kEdgeHalo;
        g.right = win1 == L ? rlb::kEdgeClamp : rlb::kEdgeHalo;
      }
      segs.push_back(g);
    }
  }
  if ((int64_t)segs.size() > h->L.max_segs) return RLB_E_ARG;
  RLB_HIP(hipMemcpyAsync(h->d_segs, segs.data(), sizeof(rlb::TubeSeg) * segs.size(),
                         hipMemcpyHostToDevice, h->stream));
  h->nseg = (int)segs.size();
  h->seg_whole = h->nseg == h->n_members;  // a cut member has two or more
  h->seg_halo = v.halo;
  h->seg_built = 2000 + sv;
  return RLB_OK;
}

// The device table of a round variant's segments, unless it is there already. The
// copy is enqueued: segs, empty if there was nothing to do, must outlive it.
rlb_status build_round_segments(rlb_sim* h, int variant, std::vector<rlb::TubeSeg>& segs) {
  if (h->d2) {
    const int sv = strip_index(variant);
    return h->seg_built == 2000 + sv ? RLB_OK : build_strip_segments(h, sv, segs);
  }
  const int tv = tube_index(variant);
  return h->seg_built == 1000 + tv ? RLB_OK : build_tube_segments(h, tv, segs);
}

// Tube rounds: ceil(n / H) launches (one when every member fits its block
// whole), each reading one buffer and writing the other (pingpong) or always
// A -> B (trials). *flip tells whether the state changed buffers. The rounds
// are launched one by one: a round runs for 10 us and more, which covers the
// launch of the next, while a graph of them is built and instantiated anew for
// every step count (1 x 1 x 800 FP64, 400 steps: 762 us,
// and 924 as a graph).
// (The D2Q9 strip rounds take the same path with their own segments and
// kernel.)
rlb_status launch_tubes(rlb_sim* h, int variant, int nsteps, int pingpong, void* a, void* b,
                        int diag_every, int64_t step0, bool* flip) {
  const void* func;
  dim3 block;
  if (!h->d2 && !h->all_tubes) return RLB_E_UNSUPPORTED;
  std::vector<rlb::TubeSeg> segs;
  rlb_status st = build_round_segments(h, variant, segs);
  if (st != RLB_OK) return st;
  if (!segs.empty()) RLB_HIP(hipStreamSynchronize(h->stream));
  if (h->d2)
    RLB_HIP(rlb::d2q9_strip_kernel(h->precision, strip_index(variant), h->corr, h->ext, &func,
                                   &block));
  else
    RLB_HIP(rlb::tube_kernel(h->precision, tube_index(variant), h->ext, &func, &block));
  const int per = h->seg_whole ? nsteps : h->seg_halo;
  const int rounds = (nsteps + per - 1) / per;
  rlb::TubeRound arg{};
  arg.descs = h->d_descs;
  arg.segs = (const rlb::TubeSeg*)h->d_segs;
  arg.cs = h->L.cs;
  arg.diag_every = diag_every;
  arg.last_step = step0 + nsteps;
  arg.partials = h->d_partials;
  arg.bad = h->d_bad;
  for (int r = 0; r < rounds; ++r) {
    const bool odd = pingpong && (r & 1);
    arg.src = odd ? b : a;
    arg.dst = odd ? a : b;
    arg.nsteps = std::min(per, nsteps - r * per);
    arg.step0 = step0 + (int64_t)r * per;
    void* args[] = {&arg};
    RLB_HIP(hipLaunchKernel(func, dim3(h->nseg, 1, 1), block, args, 0, h->stream));
  }
  *flip = pingpong && (rounds & 1);
  return RLB_OK;
}

// Cut every member into segments of whole z-planes of about nt * cpt cells
// (one pass of the block per step) and upload the table.
rlb_status build_segments(rlb_sim* h, int sv) {
  const rlb::MemberVariant mv = rlb::segment_variant(sv);
  const int64_t target = (int64_t)mv.nt * mv.cpt;
  std::vector<rlb::Segment> segs;
  for (int m = 0; m < h->n_members; ++m) {
    const MemberDesc& d = h->descs[m];
    const int64_t plane = (int64_t)d.nx * d.ny;
    const int64_t want = std::max<int64_t>(1, (d.ncells + target - 1) / target);
    const int nsm = (int)std::min<int64_t>(want, d.nz);
    const int first = (int)segs.size();
    for (int j = 0; j < nsm; ++j) {
      rlb::Segment g{};
      g.member = m;
      g.z0 = (int)((int64_t)d.nz * j / nsm);
      g.z1 = (int)((int64_t)d.nz * (j + 1) / nsm);
      const bool wrap = d.bcz == RLB_PERIODIC && nsm > 1;
      g.left = j > 0 ? first + j - 1 : (wrap ? first + nsm - 1 : -1);
      g.right = j < nsm - 1 ? first + j + 1 : (wrap ? first : -1);
      segs.push_back(g);
      (void)plane;
    }
  }
  if ((int64_t)segs.size() > h->L.max_segs) return RLB_E_ARG;
  RLB_HIP(hipMemcpyAsync(h->d_segs, segs.data(), sizeof(rlb::Segment) * segs.size(),
                         hipMemcpyHostToDevice, h->stream));
  // Every flag counts from here: a table of fewer segments has left those beyond it
  // behind the epoch, where their neighbours would wait for them in vain.
  RLB_HIP(rlb::launch_begin(nullptr, 0, h->d_flags, (size_t)h->L.max_segs, nullptr, nullptr,
                            h->stream));
  h->epoch = 0;
  RLB_HIP(hipStreamSynchronize(h->stream));
  h->nseg = (int)segs.size();
  h->seg_built = sv;
  return RLB_OK;
}

// Every block of a segment launch must be resident at once (they wait on
// each other); variants whose segments do not fit are refused.
rlb_status segments_fit(rlb_sim* h, int sv, const void* func, int nt) {
  if (h->seg_built != sv) {
    rlb_status st = build_segments(h, sv);
    if (st != RLB_OK) return st;
  }
  int per_cu = 0;
  RLB_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, func, nt, 0));
  if ((int64_t)per_cu * h->num_cu < h->nseg) return RLB_E_UNSUPPORTED;
  return RLB_OK;
}

// The persistent path: nsteps steps by the variant's kernels.
rlb_status launch_persistent(rlb_sim* h, int variant, int nsteps, int pingpong, void* a, void* b,
                             int diag_every, int64_t step0, bool* flip) {
  if (is_tube_variant(h, variant) || is_strip_variant(h, variant))
    return launch_tubes(h, variant, nsteps, pingpong, a, b, diag_every, step0, flip);
  *flip = pingpong && (nsteps & 1);
  if (is_cells_variant(h, variant)) {
    const int cv = variant - cells_base(h);
    rlb::MemberLaunch m{};
    m.descs = h->d_descs;
    m.cs = h->L.cs;
    m.partials = h->d_partials;
    m.bad = h->d_bad;
    for (int t = 0; t < nsteps; ++t) {
      const bool odd = pingpong && (t & 1);
      m.bufA = odd ? b : a;
      m.bufB = odd ? a : b;
      const bool diag =
          diag_every > 0 && ((step0 + t + 1) % diag_every == 0 || t == nsteps - 1);
      RLB_HIP(rlb::launch_step_cells(h->precision, h->d2, cv, h->corr, h->ext, diag, m,
                                     h->descs[0], h->n_members, h->L.blocks[cv], h->stream));
    }
    return RLB_OK;
  }
  const void* func;
  dim3 block, grid;
  void* args[1];
  if (is_segment_variant(h, variant)) {
    if (h->ext) return RLB_E_UNSUPPORTED;  // fixed relaxation times only
    const int sv = variant - rlb::num_member_variants();
    RLB_HIP(rlb::segment_kernel(h->precision, sv, &func, &block));
    rlb_status st = segments_fit(h, sv, func, block.x);
    if (st != RLB_OK) return st;
    rlb::SegLaunch& g = h->sargs;
    g.descs = h->d_descs;
    g.segs = h->d_segs;
    g.bufA = a;
    g.bufB = b;
    g.cs = h->L.cs;
    g.nsteps = nsteps;
    g.pingpong = pingpong;
    g.diag_every = diag_every;
    g.spin_limit = kSpinLimit;
    g.step0 = step0;
    g.epoch = h->epoch;
    g.flags = h->d_flags;
    g.error = (int*)&h->d_view->error;
    g.partials = h->d_partials;
    g.bad = h->d_bad;
    args[0] = &h->sargs;
    grid = dim3(h->nseg, 1, 1);
  } else {
    rlb::MemberLaunch& m = h->margs;
    m.descs = h->d_descs;
    m.bufA = a;
    m.bufB = b;
    m.cs = h->L.cs;
    m.nsteps = nsteps;
    m.pingpong = pingpong;
    m.diag_every = diag_every;
    m.step0 = step0;
    m.partials = h->d_partials;
    m.bad = h->d_bad;
    if (h->d2)
      RLB_HIP(rlb::d2q9_member_kernel(h->precision, variant, h->corr, h->ext, &func, &block));
    else
      RLB_HIP(rlb::member_kernel(h->precision, variant, h->ext, &func, &block));
    args[0] = &h->margs;
    grid = dim3(h->n_members, 1, 1);
  }
  RLB_HIP(hipLaunchKernel(func, grid, block, args, 0, h->stream));
  if (is_segment_variant(h, variant)) h->epoch += (unsigned long long)nsteps;
  return RLB_OK;
}

// Advance n steps without taping.
rlb_status advance(rlb_sim* h, int32_t n) {
  if (n <= 0) return RLB_OK;
  const int D = h->opt.diag_every;
  if (h->lattice && is_tile_variant(h, h->variant)) {
    bool flip = false;
    rlb_status st =
        launch_tile_rounds(h, h->variant, n, 1, state_buf(h), spare_buf(h), D, h->steps, &flip);
    if (st != RLB_OK) return st;
    h->steps += n;
    if (flip) h->cur = 1 - h->cur;
    return RLB_OK;
  }
  if (h->lattice) {
    const bool march = is_march_variant(h, h->variant);
    const int one = march ? march_step(h) : h->variant;
    for (int32_t i = 0; i < n; ++i) {
      const int64_t s = h->steps + 1;
      const auto is_diag = [&](int64_t step, int32_t at) {
        return D > 0 && (step % D == 0 || at == n - 1);
      };
      const bool diag = is_diag(s, i);
      int k = 0;  // steps from here on that may share launches (12: enough to choose)
      while (march && k < 12 && i + k < n && !is_diag(s + k, i + k)) ++k;
      const int v = march ? next_march(h, k) : -1;
      if (v >= 0) {
        rlb_status st = launch_march(h, v, state_buf(h), spare_buf(h));
        if (st != RLB_OK) return st;
        h->cur = 1 - h->cur;
        h->steps += march_steps(h, v);
        i += march_steps(h, v) - 1;
        continue;
      }
      rlb_status st = launch_lattice_step(h, one, diag, state_buf(h), spare_buf(h));
      if (st != RLB_OK) return st;
      if (diag) {
        h->diag_step = s;
        h->diag_parts = lattice_parts(h, one);
      }
      h->cur = 1 - h->cur;
      h->steps = s;
    }
    return RLB_OK;
  }
  bool flip = false;
  rlb_status st =
      launch_persistent(h, h->variant, n, 1, state_buf(h), spare_buf(h), D, h->steps, &flip);
  if (st != RLB_OK) return st;
  if (D > 0) {
    h->diag_step = h->steps + n;
    const bool by_seg = is_segment_variant(h, h->variant) || is_tube_variant(h, h->variant) ||
                        is_strip_variant(h, h->variant);
    h->diag_parts = is_cells_variant(h, h->variant) ? h->L.blocks[h->variant - cells_base(h)]
                    : by_seg                        ? h->nseg
                                                    : h->n_members;
  }
  h->steps += n;
  if (flip) h->cur = 1 - h->cur;
  return RLB_OK;
}

rlb_status copy_fields_in(rlb_sim* h, const double* n0, const double* eps0, const double* u0,
                          int on_device, const double** dn, const double** de,
                          const double** du) {
  const int64_t nc = h->L.ncells;
  if (on_device) {
    *dn = n0;
    *de = eps0;
    *du = u0;
    return RLB_OK;
  }
  double* s = h->d_stage;
  RLB_HIP(hipMemcpyAsync(s, n0, sizeof(double) * nc, hipMemcpyHostToDevice, h->stream));
  RLB_HIP(hipMemcpyAsync(s + nc, eps0, sizeof(double) * nc, hipMemcpyHostToDevice, h->stream));
  RLB_HIP(
      hipMemcpyAsync(s + 2 * nc, u0, sizeof(double) * 3 * nc, hipMemcpyHostToDevice, h->stream));
  *dn = s;
  *de = s + nc;
  *du = s + 2 * nc;
  return RLB_OK;
}

bool host_fields_ok(const double* n0, const double* eps0, const double* u0, int64_t nc,
                    bool planar, const rlb_params* members, int32_t n_members) {
  int64_t i = 0;
  for (int m = 0; m < n_members; ++m) {
    const rlb_params& p = members[m];
    const int64_t end = i + (int64_t)p.nx * p.ny * p.nz;
    const bool gen = !paper_eos(p);
    for (; i < end; ++i) {
      const double uu =
          u0[i] * u0[i] + u0[nc + i] * u0[nc + i] + u0[2 * nc + i] * u0[2 * nc + i];
      if (!(eps0[i] > 0.0) || !(n0[i] >= 0.0) || !(uu < 1.0) || !std::isfinite(n0[i]) ||
          !std::isfinite(eps0[i]) || (planar && u0[2 * nc + i] != 0.0) ||
          (gen && !(eps0[i] - p.mass * n0[i] > 0.0)))
        return false;
    }
  }
  return true;
}

}  // namespace

namespace {

const char* kernel_name_of(const rlb_sim* h, int v) {
  if (is_march_variant(h, v))
    return h->d2 ? rlb::d2q9_march_kernel_name(h->precision, v - march_base(h), h->corr)
                 : rlb::march_kernel_name(h->precision, v - march_base(h));
  if (is_cells_variant(h, v)) return rlb::cells_kernel_name(h->precision, h->d2, v - cells_base(h));
  if (h->d2) {
    if (is_tile_variant(h, v)) return rlb::d2q9_tile_kernel_name(h->precision, tile_index(v));
    if (h->lattice) return rlb::d2q9_lattice_kernel_name(h->precision, v);
    if (is_strip_variant(h, v)) return rlb::d2q9_strip_kernel_name(h->precision, strip_index(v));
    return rlb::d2q9_member_kernel_name(h->precision, v);
  }
  if (h->lattice) return rlb::lattice_kernel_name(h->precision, v);
  if (v < rlb::num_member_variants()) return rlb::member_kernel_name(h->precision, v);
  if (is_segment_variant(h, v))
    return rlb::segment_kernel_name(h->precision, v - rlb::num_member_variants());
  return rlb::tube_kernel_name(h->precision, tube_index(v));
}

// A marching variant that cannot launch on this lattice runs single steps: it has
// the name of their kernel.
bool is_idle_march(const rlb_sim* h, int v) {
  return is_march_variant(h, v) && march_steps(h, v) < 2;
}

void put_name(const rlb_sim* h, int v, char* buf, size_t buflen) {
  const bool idle = is_idle_march(h, v);
  std::snprintf(buf, buflen, "%s%s%s", kernel_name_of(h, idle ? march_step(h) : v),
                h->corr ? "+c7" : "", idle ? " (no march)" : "");
}

// Steps of a variant's launch where it makes a number of its own, else 1.
int launch_steps(const rlb_sim* h, int v) {
  if (is_march_variant(h, v)) return march_steps(h, v);
  if (is_tile_variant(h, v)) return rlb::d2q9_tile_variant(tile_index(v)).h;
  if (is_tube_variant(h, v))
    return h->all_tubes ? tube_halo(h, rlb::tube_variant(tube_index(v))) : 1;
  if (is_strip_variant(h, v)) return strip_halo(h, rlb::d2q9_strip_variant(strip_index(v)));
  return 1;
}

// A persistent segment launch whose neighbour wait timed out leaves a sticky
// error word; it is reported at the next synchronising call.
rlb_status persistent_error(rlb_sim* h) {
  rlb::HostView v;
  rlb_status st = read_view(h, &v);
  return st != RLB_OK ? st : v.error ? RLB_E_DEVICE : RLB_OK;
}

}  // namespace

// ============================================================================
extern "C" {

static_assert(sizeof(rlb_status) == sizeof(int32_t), "rlb_status travels as a 32-bit int");

const char* rlb_status_string(rlb_status s) {
  // A C caller may pass any int: read it as one (loading an enum object that
  // holds a value outside the enumeration's range is undefined in C++).
  int32_t code;
  std::memcpy(&code, &s, sizeof(code));
  switch (code) {
    case RLB_OK: return "ok";
    case RLB_E_ARG: return "invalid argument";
    case RLB_E_TAU: return "relaxation time must be finite and > 1/2";
    case RLB_E_UNPHYSICAL: return "inadmissible cell (eps <= 0, n < 0, |u| >= 1 or E <= 0, |M| >= E)";
    case RLB_E_WORKSPACE: return "workspace missing, misaligned or too small";
    case RLB_E_DEVICE: return "HIP runtime error";
    case RLB_E_STATE: return "call not valid in the current state";
    case RLB_E_UNSUPPORTED: return "unsupported configuration";
    case RLB_E_SCRATCH: return "lattice too large for the fixed scratch array of rlb_run_noalloc";
  }
  return "unknown status";
}

rlb_status rlb_workspace_size(const rlb_params* members, int32_t n_members,
                              const rlb_options* opt, size_t* bytes) {
  if (!bytes) return RLB_E_ARG;
  Layout L;
  rlb_status st = make_layout(members, n_members, opt, L);
  if (st != RLB_OK) return st;
  *bytes = L.total;
  return RLB_OK;
}

rlb_status rlb_init(rlb_handle* out, const rlb_params* members, int32_t n_members,
                    const rlb_options* opt, const double* n0, const double* eps0,
                    const double* u0, int32_t fields_on_device, void* workspace,
                    size_t workspace_bytes, void* hip_stream) {
  if (!out) return RLB_E_ARG;
  *out = nullptr;
  Layout L;
  rlb_status st = make_layout(members, n_members, opt, L);
  if (st != RLB_OK) return st;
  if (!n0 || !eps0 || !u0) return RLB_E_ARG;
  if (fields_on_device != 0 && fields_on_device != 1) return RLB_E_ARG;
  if (!workspace || ((uintptr_t)workspace % kAlign) != 0 || workspace_bytes < L.total)
    return RLB_E_WORKSPACE;
  const bool planar = opt->lattice == RLB_D2Q9;
  if (!fields_on_device && !host_fields_ok(n0, eps0, u0, L.ncells, planar, members, n_members))
    return RLB_E_UNPHYSICAL;

  rlb_sim* h = new (std::nothrow) rlb_sim();
  if (!h) return RLB_E_ARG;
  if (hipGetDevice(&h->device) != hipSuccess) {
    delete h;
    return RLB_E_DEVICE;
  }
  h->stream = (hipStream_t)hip_stream;
  h->precision = opt->precision;
  h->opt = *opt;
  h->n_members = n_members;
  h->params.assign(members, members + n_members);
  h->L = L;
  h->ws = (char*)workspace;
  h->d_descs = (MemberDesc*)(h->ws + L.off_descs);
  h->d_small = (double*)(h->ws + L.off_small);
  h->d_view = (rlb::HostView*)h->d_small;
  h->d_bad = (unsigned long long*)(h->ws + L.off_bad);
  h->d_bad_save = h->d_bad + rlb::kBadBytes / sizeof(unsigned long long);
  h->d_partials = (double*)(h->ws + L.off_partials);
  h->d_xparts = (double*)(h->ws + L.off_xparts);
  h->buf[0] = h->ws + L.off_buf0;
  h->buf[1] = h->ws + L.off_buf1;
  h->d_stage = (double*)(h->ws + L.off_stage);
  h->d_segs = (rlb::Segment*)(h->ws + L.off_segs);
  h->d_flags = (unsigned long long*)(h->ws + L.off_flags);
  h->d2 = planar;
  h->corr = opt->correction != 0;
  h->q = nvel(opt->lattice);
  h->lattice = lattice_path(n_members, L.ncells);
  h->all_tubes = !h->d2;
  for (int i = 0; i < n_members; ++i)
    if (members[i].nx != 1 || members[i].ny != 1) h->all_tubes = false;
  auto fail = [&](rlb_status s) {
    delete h;
    return s;
  };
  if (hipDeviceGetAttribute(&h->num_cu, hipDeviceAttributeMultiprocessorCount, h->device) !=
      hipSuccess)
    return fail(RLB_E_DEVICE);
  // member descriptors (refs are filled on the device)
  h->descs.resize(n_members);
  int64_t off = 0;
  int first64 = 0, first256 = 0;
  for (int i = 0; i < n_members; ++i) {
    const rlb_params& p = members[i];
    MemberDesc& d = h->descs[i];
    std::memset(&d, 0, sizeof(d));
    d.offset = off;
    d.first64 = first64;
    d.first256 = first256;
    d.nx = p.nx;
    d.ny = p.ny;
    d.nz = p.nz;
    d.ncells = p.nx * p.ny * p.nz;
    first64 += (int)(((int64_t)d.ncells + 63) / 64);
    first256 += (int)(((int64_t)d.ncells + 255) / 256);
    d.bcx = p.bc[0];
    d.bcy = p.bc[1];
    d.bcz = p.bc[2];
    const double tq = p.tau_q > 0.0 ? p.tau_q : p.tau_v;
    d.rt.w_f = 1.0 / p.tau_f;
    d.rt.s_e = 1.0 / p.tau_e;
    d.rt.s_eps = 1.0 / p.tau_eps;
    d.rt.s_q = 1.0 / tq;
    d.rt.s_v = 1.0 / p.tau_v;
    d.ext.eta_s = p.eta_over_s;
    d.ext.kappa = p.kappa;
    d.ext.dof = p.dof;
    d.ext.visc = 3.0 * p.kappa * p.eta_over_s;
    d.ext.inv_eq = rlb::kPiSquared / p.dof;
    d.ext.a_f = p.a_f;
    d.ext.a_e = p.a_e;
    d.ext.a_eps = p.a_eps;
    d.ext.a_q = p.a_q;
    d.ext.q_tied = p.tau_q > 0.0 ? 0 : 1;
    d.ext.eos_gamma = p.eos_gamma > 0.0 ? p.eos_gamma : 4.0 / 3.0;
    d.ext.mass = p.mass;
    d.ext.general_eos = paper_eos(p) ? 0 : 1;
    if (p.eta_over_s > 0.0 || d.ext.general_eos) h->ext = true;
    if (d.ext.general_eos) h->eos = true;
    off += d.ncells;
  }
  h->variant = h->lattice ? default_lattice(h) : default_persistent(h);
  // The whole start is enqueued and its one answer read back at the end: the
  // refused cells and the reference the lattice kernels take as an argument. That
  // wait also ends the last read of the caller's fields.
  const double *dn, *de, *du;
  static_assert(sizeof(rlb::HostView) <= 256, "the small area holds the view and more");
  if (rlb::launch_begin((unsigned long long*)h->d_small,
                        (L.off_bad + rlb::kBadBytes - L.off_small) / sizeof(unsigned long long),
                        h->d_flags, (size_t)L.max_segs, n_members == 1 ? &h->descs[0] : nullptr,
                        h->d_descs, h->stream) != hipSuccess)
    return fail(RLB_E_DEVICE);
  if (n_members > 1 &&
      hipMemcpyAsync(h->d_descs, h->descs.data(), sizeof(MemberDesc) * n_members,
                     hipMemcpyHostToDevice, h->stream) != hipSuccess)
    return fail(RLB_E_DEVICE);
  if (copy_fields_in(h, n0, eps0, u0, fields_on_device, &dn, &de, &du) != RLB_OK)
    return fail(RLB_E_DEVICE);
  if (rlb::launch_prepare(h->d_descs, n_members, L.ref_blocks, dn, de, du, L.ncells,
                          planar ? 1 : 0, h->d_partials, h->d_view, h->stream) != hipSuccess)
    return fail(RLB_E_DEVICE);
  const hipError_t ie =
      planar ? rlb::d2q9_launch_init(h->precision, h->buf[0], L.cs, h->d_descs, n_members, dn,
                                     de, du, L.ncells, h->stream)
             : rlb::launch_init(h->precision, h->buf[0], L.lay, h->d_descs, n_members, dn, de, du,
                                L.ncells, h->stream);
  if (ie != hipSuccess) return fail(RLB_E_DEVICE);
  if (opt->ckpt_every > 0) {  // reads the caller's fields too: ahead of the wait
    rlb_status ts = rlb::tape_init(h->tape, L.tape, h->ws + L.off_tape, h->precision, L.ncells,
                                   L.cs, opt->ckpt_every, opt->tape_steps, dn, de, du,
                                   h->buf[0], h->stream);
    if (ts != RLB_OK) return fail(ts);
  }
  // The default's segments too, so that no step of a fresh handle waits.
  std::vector<rlb::TubeSeg> segs;
  if (is_tube_variant(h, h->variant) || is_strip_variant(h, h->variant)) {
    const rlb_status ts = build_round_segments(h, h->variant, segs);
    if (ts != RLB_OK) return fail(ts);
  }
  rlb::HostView view;
  if (read_view(h, &view) != RLB_OK) return fail(RLB_E_DEVICE);
  if (view.refused) return fail(RLB_E_UNPHYSICAL);
  h->descs[0].ref = view.ref0;
  if (h->lattice) {
    const MemberDesc& d = h->descs[0];
    h->geom.nx = d.nx;
    h->geom.ny = d.ny;
    h->geom.nz = d.nz;
    h->geom.bcx = d.bcx;
    h->geom.bcy = d.bcy;
    h->geom.bcz = d.bcz;
    h->geom.cs = L.cs;
    h->geom.lay = L.lay;
    h->geom.rt = d.rt;
    h->geom.ref = d.ref;
    h->geom.ext = d.ext;
    // Plain stores in the one-step kernels while the double-buffered state is
    // at most 1 GiB (measured on D3Q19 FP32 planar lattices: 25-37 % faster
    // at 80-160 MB, even at 320 MB, 10 % faster at 640 MB; nontemporal stores
    // 4-5 % faster from 1.3 GB up, e.g. the 5.1 GB of 256^3).
    h->geom.cached_store = 2 * (L.off_buf1 - L.off_buf0) <= kCachedStateBytes ? 1 : 0;
  }
  if (h->lattice && can_march(h)) {
    if (!h->d2) h->march = rlb::march_grid(h->precision, h->geom, h->num_cu);
    const MarchDefault md = march_default(h);
    const double use = h->d2 ? rlb::d2q9_march_use(h->precision, md.variant, h->corr, h->ext,
                                                   h->geom, h->num_cu)
                             : h->march.use;
    if (use >= md.least_use) h->variant = march_base(h) + md.variant;
  }
  h->cur = 0;
  h->tape_ok = opt->ckpt_every > 0;
  *out = h;
  return RLB_OK;
}

rlb_status rlb_step(rlb_handle h, int32_t nsteps) {
  if (!h || nsteps < 0) return RLB_E_ARG;
  if (nsteps == 0) return RLB_OK;
  DeviceGuard g(h->device);
  if (!g.ok) return RLB_E_DEVICE;
  if (h->opt.ckpt_every <= 0 || !h->tape_ok) return advance(h, nsteps);
  // With a tape: stop at every checkpoint boundary and keep g.
  const int K = h->opt.ckpt_every;
  int32_t left = nsteps;
  while (left > 0) {
    int32_t chunk = (int32_t)std::min<int64_t>(left, K - (h->steps % K));
    rlb_status st = advance(h, chunk);
    if (st != RLB_OK) return st;
    left -= chunk;
    if (h->steps > h->opt.tape_steps) {
      h->tape_ok = false;
      return advance(h, left);
    }
    if (h->steps % K == 0) {
      st = rlb::tape_checkpoint(h->tape, h->steps / K, state_buf(h), h->stream);
      if (st != RLB_OK) return st;
    }
  }
  return RLB_OK;
}

rlb_status rlb_moments(rlb_handle h, double* n, double* eps, double* P, double* gamma,
                       double* u, double sums[5], int64_t* n_unphysical,
                       int32_t out_on_device) {
  if (!h) return RLB_E_ARG;
  if (out_on_device != 0 && out_on_device != 1) return RLB_E_ARG;
  DeviceGuard g(h->device);
  if (!g.ok) return RLB_E_DEVICE;
  const int64_t nc = h->L.ncells;
  double* s = h->d_stage;
  double *dn = n, *de = eps, *dP = P, *dg = gamma, *du = u;
  if (!out_on_device) {
    dn = n ? s : nullptr;
    de = eps ? s + nc : nullptr;
    dP = P ? s + 2 * nc : nullptr;
    dg = gamma ? s + 3 * nc : nullptr;
    du = u ? s + 4 * nc : nullptr;
  }
  const int nparts = h->L.export_parts;
  if (h->d2)
    RLB_HIP(rlb::d2q9_launch_export(h->precision, state_buf(h), h->L.cs, h->d_descs,
                                    h->n_members, nc, dn, de, dP, dg, du, h->d_xparts, nparts,
                                    nullptr, h->stream));
  else
    RLB_HIP(rlb::launch_export(h->precision, state_buf(h), h->L.lay, h->d_descs, h->n_members,
                               nc, dn, de, dP, dg, du, h->d_xparts, nparts, nullptr, h->stream));
  RLB_HIP(rlb::launch_finish(h->d_xparts, nparts, h->d_bad, h->d_view, h->stream));
  if (!out_on_device) {
    if (n) RLB_HIP(hipMemcpyAsync(n, dn, sizeof(double) * nc, hipMemcpyDeviceToHost, h->stream));
    if (eps)
      RLB_HIP(hipMemcpyAsync(eps, de, sizeof(double) * nc, hipMemcpyDeviceToHost, h->stream));
    if (P) RLB_HIP(hipMemcpyAsync(P, dP, sizeof(double) * nc, hipMemcpyDeviceToHost, h->stream));
    if (gamma)
      RLB_HIP(hipMemcpyAsync(gamma, dg, sizeof(double) * nc, hipMemcpyDeviceToHost, h->stream));
    if (u)
      RLB_HIP(hipMemcpyAsync(u, du, sizeof(double) * 3 * nc, hipMemcpyDeviceToHost, h->stream));
  }
  rlb::HostView view;
  rlb_status st = read_view(h, &view);
  if (st != RLB_OK) return st;
  if (sums) std::memcpy(sums, view.sums, sizeof(view.sums));
  if (n_unphysical) *n_unphysical = (int64_t)view.bad;
  if (view.error) return RLB_E_DEVICE;
  return view.bad ? RLB_E_UNPHYSICAL : RLB_OK;
}

rlb_status rlb_diagnostics(rlb_handle h, double sums[5], int64_t* step, int64_t* n_unphysical) {
  if (!h) return RLB_E_ARG;
  if (h->diag_step < 0) return RLB_E_STATE;
  DeviceGuard g(h->device);
  if (!g.ok) return RLB_E_DEVICE;
  RLB_HIP(rlb::launch_finish(h->d_partials, h->diag_parts, h->d_bad, h->d_view, h->stream));
  rlb::HostView view;
  rlb_status st = read_view(h, &view);
  if (st != RLB_OK) return st;
  if (sums) std::memcpy(sums, view.sums, sizeof(view.sums));
  if (step) *step = h->diag_step;
  if (n_unphysical) *n_unphysical = (int64_t)view.bad;
  return view.error ? RLB_E_DEVICE : RLB_OK;
}

rlb_status rlb_populations(rlb_handle h, double* f, double* g, int32_t out_on_device) {
  if (!h) return RLB_E_ARG;
  if (out_on_device != 0 && out_on_device != 1) return RLB_E_ARG;
  DeviceGuard dg(h->device);
  if (!dg.ok) return RLB_E_DEVICE;
  const int64_t nc = h->L.ncells;
  const int Q = h->q;
  auto planes = [&](int p0, int np, double* out) {
    return h->d2 ? rlb::d2q9_launch_population_planes(h->precision, state_buf(h), h->L.cs,
                                                      h->d_descs, h->n_members, nc, p0, np, out,
                                                      h->stream)
                 : rlb::launch_population_planes(h->precision, state_buf(h), h->L.lay,
                                                 h->d_descs, h->n_members, nc, p0, np, out,
                                                 h->stream);
  };
  if (out_on_device) {
    if (f) RLB_HIP(planes(0, Q, f));
    if (g) RLB_HIP(planes(Q, Q, g));
  } else {
    // staging holds 8 planes: convert f (then g) in chunks of up to 8 planes
    double* s = h->d_stage;
    for (int which = 0; which < 2; ++which) {
      double* hostp = which ? g : f;
      if (!hostp) continue;
      for (int a0 = 0; a0 < Q; a0 += 8) {
        const int na = std::min(8, Q - a0);
        RLB_HIP(planes(which * Q + a0, na, s));
        RLB_HIP(hipMemcpyAsync(hostp + (size_t)a0 * nc, s, sizeof(double) * na * nc,
                               hipMemcpyDeviceToHost, h->stream));
        RLB_HIP(hipStreamSynchronize(h->stream));
      }
    }
  }
  return persistent_error(h);
}

rlb_status rlb_grad(rlb_handle h, const double* dL_du, const double* dL_deps,
                    double dL_dtau[3], double* dL_deps0, double* dL_du0, int32_t io_on_device) {
  if (!h || !dL_du || !dL_deps || !dL_dtau || !dL_deps0 || !dL_du0) return RLB_E_ARG;
  if (io_on_device != 0 && io_on_device != 1) return RLB_E_ARG;
  if (h->opt.ckpt_every <= 0 || !h->tape_ok) return RLB_E_STATE;
  DeviceGuard g(h->device);
  if (!g.ok) return RLB_E_DEVICE;
  rlb::GradContext c{};
  c.precision = h->precision;
  c.ncells = h->L.ncells;
  c.cs = h->L.cs;
  c.desc = h->descs[0];
  c.steps = h->steps;
  c.tau_q_tied = !(h->params[0].tau_q > 0.0);
  c.state = state_buf(h);
  c.stage = h->d_stage;
  c.sums_out = h->d_small + 32;
  c.stream = h->stream;
  return rlb::tape_grad(h->tape, c, dL_du, dL_deps, dL_dtau, dL_deps0, dL_du0, io_on_device);
}

rlb_status rlb_num_variants(rlb_handle h, int32_t* count) {
  if (!h || !count) return RLB_E_ARG;
  if (h->d2)
    *count = h->lattice ? march_base(h) + rlb::d2q9_num_march_variants(h->corr)
                        : cells_base(h) + rlb::kNumCells;
  else
    *count = h->lattice ? march_base(h) + rlb::num_march_variants()
                        : cells_base(h) + rlb::kNumCells;
  return RLB_OK;
}

rlb_status rlb_variant_name(rlb_handle h, int32_t v, char* buf, size_t buflen) {
  int32_t n;
  if (rlb_num_variants(h, &n) != RLB_OK || !buf || buflen == 0) return RLB_E_ARG;
  if (v < 0 || v >= n) return RLB_E_ARG;
  put_name(h, v, buf, buflen);
  return RLB_OK;
}

rlb_status rlb_set_variant(rlb_handle h, int32_t v) {
  int32_t n;
  if (rlb_num_variants(h, &n) != RLB_OK) return RLB_E_ARG;
  if (v < 0 || v >= n) return RLB_E_ARG;
  h->variant = v;
  return RLB_OK;
}

rlb_status rlb_get_variant(rlb_handle h, int32_t* v) {
  if (!h || !v) return RLB_E_ARG;
  *v = h->variant;
  return RLB_OK;
}

rlb_status rlb_tune(rlb_handle h, int32_t trial_steps, int32_t* best_variant,
                    double* ms_per_step) {
  if (!h || trial_steps < 1) return RLB_E_ARG;
  DeviceGuard g(h->device);
  if (!g.ok) return RLB_E_DEVICE;
  int32_t n;
  rlb_num_variants(h, &n);
  hipEvent_t e0, e1;
  RLB_HIP(hipEventCreate(&e0));
  RLB_HIP(hipEventCreate(&e1));
  // trial steps must not count toward the inadmissible-cell total
  RLB_HIP(hipMemcpyAsync(h->d_bad_save, h->d_bad, rlb::kBadBytes, hipMemcpyDeviceToDevice,
                         h->stream));
  const int keep = h->variant;
  int best = keep;
  double best_ms = 1e300;
  rlb_status st = RLB_OK;
  for (int v = 0; v < n && st == RLB_OK; ++v) {
    // whole launches: a part of one would price the variant by its start, or by
    // another's kernel
    const int one = launch_steps(h, v);
    const int steps = (int)std::min<int64_t>((trial_steps + (int64_t)one - 1) / one * one,
                                             INT32_MAX / one * one);
    float ms = 0.0f;
    bool usable = !is_idle_march(h, v);  // else another variant's kernel, timed already
    for (int rep = 0; rep < 2 && st == RLB_OK && usable; ++rep) {  // rep 0 warms up
      if (hipEventRecord(e0, h->stream) != hipSuccess) st = RLB_E_DEVICE;
      if (h->lattice && is_tile_variant(h, v)) {
        bool flip = false;
        st = launch_tile_rounds(h, v, steps, 0, state_buf(h), spare_buf(h), 0, 0, &flip);
        if (st == RLB_E_UNSUPPORTED) {  // a tiled axis leaves no owned cell
          usable = false;
          st = RLB_OK;
        }
      } else if (h->lattice) {
        const bool march = is_march_variant(h, v);
        for (int i = 0; i < steps && st == RLB_OK; i += launch_steps(h, v))
          st = march ? launch_march(h, v, state_buf(h), spare_buf(h))
                     : launch_lattice_step(h, v, false, state_buf(h), spare_buf(h));
      } else if (st == RLB_OK) {
        bool flip = false;
        st = launch_persistent(h, v, steps, 0, state_buf(h), spare_buf(h), 0, 0, &flip);
        if (st == RLB_E_UNSUPPORTED) {  // segments do not all fit at once
          usable = false;
          st = RLB_OK;
        }
      }
      if (st == RLB_OK && usable && hipEventRecord(e1, h->stream) != hipSuccess)
        st = RLB_E_DEVICE;
      if (st == RLB_OK && usable && hipEventSynchronize(e1) != hipSuccess) st = RLB_E_DEVICE;
      if (st == RLB_OK && usable && hipEventElapsedTime(&ms, e0, e1) != hipSuccess)
        st = RLB_E_DEVICE;
    }
    const double per = usable ? (double)ms / steps : HUGE_VAL;
    if (ms_per_step) ms_per_step[v] = per;
    if (st == RLB_OK && usable && per < best_ms) {
      best_ms = per;
      best = v;
    }
  }
  if (st == RLB_OK) st = persistent_error(h);
  (void)hipMemcpyAsync(h->d_bad, h->d_bad_save, rlb::kBadBytes, hipMemcpyDeviceToDevice,
                       h->stream);
  (void)hipStreamSynchronize(h->stream);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  h->variant = (st == RLB_OK) ? best : keep;
  if (best_variant) *best_variant = h->variant;
  return st;
}

rlb_status rlb_info(rlb_handle h, int64_t* steps, char* kernel_name, size_t buflen) {
  if (!h) return RLB_E_ARG;
  if (steps) *steps = h->steps;
  if (kernel_name && buflen) put_name(h, h->variant, kernel_name, buflen);
  return RLB_OK;
}

void rlb_free(rlb_handle h) {
  if (!h) return;
  {
    DeviceGuard g(h->device);
    (void)hipStreamSynchronize(h->stream);
    rlb::tape_release(h->tape);
  }
  delete h;
}

}  // extern "C"
