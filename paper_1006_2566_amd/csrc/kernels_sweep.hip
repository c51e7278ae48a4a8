// Colour-pass kernels: one launch updates every site of one colour (§4's
// checkerboard: sites of one colour share no bond, so they are independent).
//
// Memory: spins and couplings are colour-split structure-of-arrays (six planes of
// N/2 values each), so a wavefront reads one contiguous row segment per plane and
// the six neighbours of a colour-c site are the same xh in the rows y+-1 and planes
// z+-1 of the other colour, plus xh and xh+-1 in its own row.  A pass therefore
// reads the own colour's spins and couplings, the other colour's spins and
// couplings, and writes the own colour's spins: 30 bytes per lattice site in
// binary32.  Neighbour rows shared by adjacent tiles are served from L2, which is
// why tiles are assigned to XCDs in contiguous z ranges (see xcd_tile).
#include <algorithm>

#include "hsg_device.h"
#include "hsg_internal.h"
#include "hsg_site.h"

namespace hsg {

Geometry pass_geometry(int32_t L) {
  Geometry g{};
  g.L = L;
  g.Lh = L / 2;
  g.plane = g.Lh * L;
  g.tiles_p = (g.plane + kPassThreads - 1) / kPassThreads;
  g.slab = std::max(1, std::min(L, kPassThreads / std::max(64, g.plane)));
  g.n_blocks = g.tiles_p * L;
  g.n_partials = std::max(g.n_blocks, L <= kBrickMaxL ? (L / 2) * (L / 2) : 0);
  g.inv_lh = g.Lh > 1 ? 0xFFFFFFFFu / (uint32_t)g.Lh + 1u : 0u;
  g.inv_tp = g.tiles_p > 1 ? (uint32_t)(0x100000000ull / (uint32_t)g.tiles_p) : 0u;
  return g;
}

size_t work_bytes_for(int32_t L) {
  return 256 + sizeof(double) * ((size_t)pass_geometry(L).n_partials + (size_t)kReduceRegion);
}

size_t fused_offset(int32_t L) { return (work_bytes_for(L) + 255) & ~(size_t)255; }

size_t work_bytes_for(int32_t L, int32_t dtype_bytes) {
  BrickPlan plan;
  if (!march_supported(L) && !phase_supported(L) && !brick_plan(L, dtype_bytes, &plan))
    return work_bytes_for(L);
  return fused_offset(L) + (size_t)3 * L * L * L * (size_t)dtype_bytes;
}

// One tile of a colour pass (kPassThreads consecutive sites of one plane of the colour);
// Metropolis and heat-bath passes add the tile's accepted energy changes to partials[tile]
// in a fixed order (wave sums, then the waves in order).  `tile` must be wave-uniform.
template <typename R, PassMode MODE, bool NT>
__device__ __forceinline__ void pass_tile(const PassArgs<R>& a, uint32_t tile) {
  const TileSite ts = tile_site(a.g, tile);
  const HitCtx<R> hc{a.beta, a.sweep, a.phase, a.k_hits, a.seed_lo, a.seed_hi};
  double dE_sum = 0.0;
  if (ts.i < (uint32_t)a.g.plane)
    dE_sum = update_site<R, MODE, NT>(a.spins, a.J, a.colour,
                                      tile_site_offsets<R>(a.g, ts, (uint32_t)a.colour), hc);

  if constexpr (MODE != PassMode::OverRelax) {
    __shared__ double wave_part[kPassThreads / 64];
    const double v = wave_sum(dE_sum);
    if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0)
      atomicAdd(&a.partials[tile],  // its only writer: the sum without waiting for a load
                ((wave_part[0] + wave_part[1]) + (wave_part[2] + wave_part[3])));
  }
}

// Workgroup b of the launch takes tile tile_base + xcd_tile(b) (mirrored when the pass
// walks z backwards); the grid is tile_count workgroups.
template <typename R, PassMode MODE, bool NT>
__global__ __launch_bounds__(kPassThreads) void colour_pass_kernel(PassArgs<R> a) {
  int32_t tile = xcd_tile((int32_t)blockIdx.x, a.tile_count);
  if (a.reverse) tile = a.tile_count - 1 - tile;
  pass_tile<R, MODE, NT>(a, (uint32_t)__builtin_amdgcn_readfirstlane(a.tile_base + tile));
}

template <typename R, bool NT>
void launch_pass_kind(PassMode mode, const PassArgs<R>& a, hipStream_t stream) {
  const dim3 grid((unsigned)a.tile_count), block(kPassThreads);
  switch (mode) {
    case PassMode::Metropolis:
    case PassMode::MetropolisFull:
      if (metropolis_mode(a.k_hits) == PassMode::MetropolisFull)
        hipLaunchKernelGGL((colour_pass_kernel<R, PassMode::MetropolisFull, NT>), grid, block, 0,
                           stream, a);
      else
        hipLaunchKernelGGL((colour_pass_kernel<R, PassMode::Metropolis, NT>), grid, block, 0,
                           stream, a);
      break;
    case PassMode::OverRelax:
      hipLaunchKernelGGL((colour_pass_kernel<R, PassMode::OverRelax, NT>), grid, block, 0, stream,
                         a);
      break;
    case PassMode::HeatBath:
      hipLaunchKernelGGL((colour_pass_kernel<R, PassMode::HeatBath, NT>), grid, block, 0, stream,
                         a);
      break;
  }
}

template <typename R>
hipError_t launch_colour_pass(PassMode mode, const PassArgs<R>& a, hipStream_t stream) {
  if (a.tile_count < 1 || a.tile_base < 0 || a.tile_base + a.tile_count > a.g.n_blocks)
    return hipErrorInvalidValue;
  if (a.nt)
    launch_pass_kind<R, true>(mode, a, stream);
  else
    launch_pass_kind<R, false>(mode, a, stream);
  return hipGetLastError();
}

template hipError_t launch_colour_pass<float>(PassMode, const PassArgs<float>&, hipStream_t);
template hipError_t launch_colour_pass<double>(PassMode, const PassArgs<double>&, hipStream_t);

// Sum of partials[i0], partials[i0 + step], ... below i1 in a fixed order (strided per
// thread, then a fixed tree), each reset to zero; valid in thread 0.
constexpr int kFoldThreads = 1024;
__device__ __forceinline__ double fold_range(double* partials, int32_t i0, int32_t i1,
                                             int32_t step) {
  __shared__ double wave_part[16];
  double acc = 0.0;
  for (int32_t i = i0 + (int32_t)threadIdx.x * step; i < i1; i += kFoldThreads * step) {
    acc += partials[i];
    partials[i] = 0.0;
  }
  return block_sum(acc, wave_part);
}

// First of two folds: workgroup b puts the sum of its chunk in the chunk's first place.
__global__ __launch_bounds__(kFoldThreads) void fold_chunks_kernel(double* partials, int32_t n,
                                                                   int32_t chunk) {
  const int32_t i0 = (int32_t)blockIdx.x * chunk;
  const double total = fold_range(partials, i0, min(n, i0 + chunk), 1);
  if (threadIdx.x == 0) partials[i0] = total;
}

// *E += sum of every step-th partial; the partials are zero afterwards, for the next sweeps.
__global__ __launch_bounds__(kFoldThreads) void fold_partials_kernel(double* partials, int32_t n,
                                                                     int32_t step, double* E) {
  const double total = fold_range(partials, 0, n, step);
  if (threadIdx.x == 0) *E += total;
}

// One workgroup reads the partials at the rate of one compute unit: 17.7 us for the 32768
// of L = 256 and 119 us for the 262144 of L = 512.  Chunks of kFoldChunk are therefore
// folded in parallel first, where one workgroup would need more than eight rounds (below
// that the second launch costs more than it saves).
constexpr int kFoldChunk = 2048;
hipError_t launch_fold_partials(double* partials, int32_t n, double* E, hipStream_t stream) {
  int32_t step = 1;
  if (n > 8 * kFoldThreads) {
    step = kFoldChunk;
    hipLaunchKernelGGL(fold_chunks_kernel, dim3((unsigned)((n + step - 1) / step)),
                       dim3(kFoldThreads), 0, stream, partials, n, step);
  }
  hipLaunchKernelGGL(fold_partials_kernel, dim3(1), dim3(kFoldThreads), 0, stream, partials, n,
                     step, E);
  return hipGetLastError();
}

}  // namespace hsg
