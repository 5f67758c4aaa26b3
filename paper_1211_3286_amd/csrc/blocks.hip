// The fused one-step kernel on lattices stored in blocks of 32 cells
// (step_lattice.hpp; a source of its own, compiled beside kernels.hip).

#include <hip/hip_runtime.h>

#include "step_lattice.hpp"

namespace rlb {

hipError_t launch_step_blocks(int precision, int v, bool diag, bool ext, const void* src,
                              void* dst, const LatticeGeom& g, double* partials,
                              unsigned long long* bad, hipStream_t s) {
  return lat_step<true>(precision, v, diag, ext, src, dst, g, partials, bad, s);
}

}  // namespace rlb
