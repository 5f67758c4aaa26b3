// rlb_run_noalloc (include/rlb.h): the run of rlb_init + rlb_step +
// rlb_moments on one lattice, for callers that cannot allocate. Everything the
// kernels need besides the caller's fields (populations, member descriptor,
// partial sums, counters) lives in one fixed device array of this file.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "../../include/rlb.h"
#include "internal.hpp"

namespace {

// The fixed scratch array. In host code its name is only a stand-in for the
// device symbol: the device address comes from hipGetSymbolAddress, once per
// device, and only that address is handed to kernels and copies.
static __device__ __align__(256) unsigned char scratch[RLB_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
constexpr size_t kAlign = 256;

struct DeviceSlot {
  std::mutex mu;           // one call at a time per device: the array is shared
  unsigned char* ptr = nullptr;  // device address of this device's copy of scratch
};
DeviceSlot g_slots[kMaxDevices];

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// Carving of the scratch array for one lattice of ncells cells.
struct Carve {
  size_t desc, small, bad, parts, xparts, buf0, buf1, total;
  int64_t cs;
  int ref_blocks, export_parts;
};

Carve carve(int64_t ncells, int q, size_t esz) {
  Carve c{};
  c.cs = (ncells + 63) / 64 * 64 + 64;
  c.ref_blocks = rlb::ref_blocks(ncells);
  c.export_parts = rlb::export_blocks(ncells);
  size_t o = 0;
  c.desc = o;
  o = align_up(o + sizeof(rlb::MemberDesc));
  c.small = o;  // the host's view
  o = align_up(o + 1024);
  c.bad = o;
  o = align_up(o + rlb::kBadBytes);
  c.parts = o;
  o = align_up(o + sizeof(double) * 5 * rlb::kRefBlocks);
  c.xparts = o;
  o = align_up(o + sizeof(double) * 5 * (size_t)c.export_parts);
  const size_t buf = 2 * (size_t)q * (size_t)c.cs * esz;
  c.buf0 = o;
  o = align_up(o + buf);
  c.buf1 = o;
  o = align_up(o + buf);
  c.total = o;
  return c;
}

bool paper_eos(const rlb_params& p) {
  return (p.eos_gamma == 0.0 || p.eos_gamma == 4.0 / 3.0) && p.mass == 0.0;
}

bool finite_tau(double t) { return std::isfinite(t) && t > 0.5; }

// The checks rlb_init makes on one member and the options (its make_layout).
rlb_status check(const rlb_params& p, const rlb_options& o) {
  if (o.precision != RLB_FP32 && o.precision != RLB_FP64) return RLB_E_ARG;
  if (o.lattice != RLB_D3Q19 && o.lattice != RLB_D2Q9) return RLB_E_ARG;
  if (o.correction != 0 && o.correction != 1) return RLB_E_ARG;
  if (o.ckpt_every != 0) return RLB_E_UNSUPPORTED;  // no tape: rlb_grad needs a handle
  if (o.correction && o.lattice != RLB_D2Q9) return RLB_E_UNSUPPORTED;
  if (p.nx < 1 || p.ny < 1 || p.nz < 1) return RLB_E_ARG;
  for (int k = 0; k < 3; ++k)
    if (p.bc[k] != RLB_PERIODIC && p.bc[k] != RLB_ZERO_GRADIENT) return RLB_E_ARG;
  if (o.lattice == RLB_D2Q9 && p.nz != 1) return RLB_E_ARG;
  if (!finite_tau(p.tau_f) || !finite_tau(p.tau_v) || !finite_tau(p.tau_e) ||
      !finite_tau(p.tau_eps) || std::isnan(p.tau_q) || (p.tau_q > 0.0 && !finite_tau(p.tau_q)))
    return RLB_E_TAU;
  if (!std::isfinite(p.eta_over_s) || p.eta_over_s < 0.0) return RLB_E_ARG;
  if (!(p.eos_gamma == 0.0 || (p.eos_gamma > 1.0 && p.eos_gamma <= 2.0))) return RLB_E_ARG;
  if (!std::isfinite(p.mass) || p.mass < 0.0) return RLB_E_ARG;
  if (p.eta_over_s > 0.0) {
    if (!std::isfinite(p.kappa) || !(p.kappa > 0.0)) return RLB_E_ARG;
    if (!std::isfinite(p.dof) || !(p.dof > 0.0)) return RLB_E_ARG;
    for (double a : {p.a_f, p.a_e, p.a_eps, p.a_q})
      if (!std::isfinite(a) || a < 0.0) return RLB_E_ARG;
  }
  if (o.correction && !paper_eos(p)) return RLB_E_UNSUPPORTED;
  return RLB_OK;
}

#define NA_HIP(call)                           \
  do {                                         \
    if ((call) != hipSuccess) return RLB_E_DEVICE; \
  } while (0)

// The run itself, with this device's scratch address in ws.
rlb_status run(unsigned char* ws, const rlb_params& p, const rlb_options& o, const double* n0,
               const double* eps0, const double* u0, int32_t nsteps, double* n, double* eps,
               double* P, double* gamma, double* u, double sums[5], int64_t* n_unphysical,
               hipStream_t st) {
  const bool d2 = o.lattice == RLB_D2Q9;
  const int64_t nc = (int64_t)p.nx * p.ny * p.nz;
  const Carve c = carve(nc, d2 ? 9 : 19, o.precision == RLB_FP32 ? 4 : 8);
  rlb::MemberDesc* d_desc = (rlb::MemberDesc*)(ws + c.desc);
  rlb::HostView* d_view = (rlb::HostView*)(ws + c.small);
  unsigned long long* d_bad = (unsigned long long*)(ws + c.bad);
  double* d_parts = (double*)(ws + c.parts);
  double* d_xparts = (double*)(ws + c.xparts);
  void* buf[2] = {ws + c.buf0, ws + c.buf1};
  const rlb::StateLayout lay = rlb::plane_layout(c.cs, (uint32_t)p.nx * (uint32_t)p.ny);

  rlb::MemberDesc desc;
  std::memset(&desc, 0, sizeof(desc));
  desc.offset = 0;
  desc.nx = p.nx;
  desc.ny = p.ny;
  desc.nz = p.nz;
  desc.ncells = (int32_t)nc;
  desc.bcx = p.bc[0];
  desc.bcy = p.bc[1];
  desc.bcz = p.bc[2];
  const double tq = p.tau_q > 0.0 ? p.tau_q : p.tau_v;
  desc.rt.w_f = 1.0 / p.tau_f;
  desc.rt.s_e = 1.0 / p.tau_e;
  desc.rt.s_eps = 1.0 / p.tau_eps;
  desc.rt.s_q = 1.0 / tq;
  desc.rt.s_v = 1.0 / p.tau_v;
  desc.ext.eta_s = p.eta_over_s;
  desc.ext.kappa = p.kappa;
  desc.ext.dof = p.dof;
  desc.ext.visc = 3.0 * p.kappa * p.eta_over_s;
  desc.ext.inv_eq = rlb::kPiSquared / p.dof;
  desc.ext.a_f = p.a_f;
  desc.ext.a_e = p.a_e;
  desc.ext.a_eps = p.a_eps;
  desc.ext.a_q = p.a_q;
  desc.ext.q_tied = p.tau_q > 0.0 ? 0 : 1;
  desc.ext.eos_gamma = p.eos_gamma > 0.0 ? p.eos_gamma : 4.0 / 3.0;
  desc.ext.mass = p.mass;
  desc.ext.general_eos = paper_eos(p) ? 0 : 1;
  const bool ext = p.eta_over_s > 0.0 || desc.ext.general_eos;

  // The whole run is enqueued and its one answer read back at the end (each
  // wait for the device costs what several of these kernels take): the
  // reference state stays on the device, where the step kernels read it, and
  // the export writes nothing when the input pass refused a cell. The array
  // keeps the previous call's contents: the counters are cleared first.
  NA_HIP(rlb::launch_begin((unsigned long long*)d_view,
                           (c.parts - c.small) / sizeof(unsigned long long), nullptr, 0, &desc,
                           d_desc, st));
  NA_HIP(rlb::launch_prepare(d_desc, 1, c.ref_blocks, n0, eps0, u0, nc, d2 ? 1 : 0, d_parts,
                             d_view, st));
  NA_HIP(d2 ? rlb::d2q9_launch_init(o.precision, buf[0], c.cs, d_desc, 1, n0, eps0, u0, nc, st)
            : rlb::launch_init(o.precision, buf[0], lay, d_desc, 1, n0, eps0, u0, nc, st));

  // steps (rlb_step): one launch per step
  const int variant = nc <= 64 * (int64_t)rlb::small_blocks(d2) ? 0 : 1;
  const int blocks = (int)(variant ? (nc + 255) / 256 : (nc + 63) / 64);
  rlb::MemberLaunch m{};
  m.descs = d_desc;
  m.cs = c.cs;
  m.partials = d_parts;
  m.bad = d_bad;
  int cur = 0;
  for (int32_t i = 0; i < nsteps; ++i) {
    m.bufA = buf[cur];
    m.bufB = buf[1 - cur];
    NA_HIP(rlb::launch_step_cells(o.precision, d2, variant, o.correction != 0, ext, false, m, desc,
                                  1, blocks, st));
    cur = 1 - cur;
  }

  // fields and lattice sums of the final state (rlb_moments)
  if (d2)
    NA_HIP(rlb::d2q9_launch_export(o.precision, buf[cur], c.cs, d_desc, 1, nc, n, eps, P, gamma,
                                   u, d_xparts, c.export_parts, &d_view->refused, st));
  else
    NA_HIP(rlb::launch_export(o.precision, buf[cur], lay, d_desc, 1, nc, n, eps, P, gamma, u,
                              d_xparts, c.export_parts, &d_view->refused, st));
  NA_HIP(rlb::launch_finish(d_xparts, c.export_parts, d_bad, d_view, st));
  rlb::HostView view;
  NA_HIP(hipMemcpyAsync(&view, d_view, sizeof(view), hipMemcpyDeviceToHost, st));
  NA_HIP(hipStreamSynchronize(st));
  if (view.refused) return RLB_E_UNPHYSICAL;
  if (sums) std::memcpy(sums, view.sums, sizeof(view.sums));
  if (n_unphysical) *n_unphysical = (int64_t)view.bad;
  return view.bad ? RLB_E_UNPHYSICAL : RLB_OK;
}

}  // namespace

extern "C" rlb_status rlb_run_noalloc(const rlb_params* member, const rlb_options* opt,
                                      const double* n0, const double* eps0, const double* u0,
                                      int32_t nsteps, double* n, double* eps, double* P,
                                      double* gamma, double* u, double sums[5],
                                      int64_t* n_unphysical, void* hip_stream) {
  if (!member || !opt || !n0 || !eps0 || !u0 || nsteps < 0) return RLB_E_ARG;
  rlb_status s = check(*member, *opt);
  if (s != RLB_OK) return s;
  const int64_t nc = (int64_t)member->nx * member->ny * member->nz;
  if (nc >= (int64_t(1) << 31)) return RLB_E_SCRATCH;
  const Carve c = carve(nc, opt->lattice == RLB_D2Q9 ? 9 : 19,
                        opt->precision == RLB_FP32 ? 4 : 8);
  if (c.total > (size_t)RLB_NOALLOC_SCRATCH_BYTES) return RLB_E_SCRATCH;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return RLB_E_DEVICE;
  DeviceSlot& slot = g_slots[dev];
  std::lock_guard<std::mutex> lock(slot.mu);
  if (!slot.ptr) {  // first call on this device (it is current): this copy's address
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr)
      return RLB_E_DEVICE;
    slot.ptr = (unsigned char*)ptr;
  }
  return run(slot.ptr, *member, *opt, n0, eps0, u0, nsteps, n, eps, P, gamma, u, sums,
             n_unphysical, (hipStream_t)hip_stream);
}
