// Batched form: many independent lattices ("chains") of mixed size advanced by one
// launch, plus replica exchange (parallel tempering) and pairwise overlaps over the
// chains of a batch.
//
// One workgroup owns one chain for the whole launch: it runs that chain's colour
// passes with a workgroup barrier between them, so a whole sweep -- and several
// sweeps -- happen inside the launch with no grid-wide synchronisation.  Workgroups
// are dispatched in the caller's order (largest lattices first), which balances
// lattices of uneven L; the launch has no state of its own, so it can be captured in
// a HIP graph and replayed.  The site update is the same function as in the
// single-lattice colour pass.
#include <algorithm>

#include "hsg.h"
#include "hsg_device.h"
#include "hsg_internal.h"
#include "hsg_site.h"

namespace hsg {

namespace {

// Workgroup size of the per-chain reductions (energy, overlaps): one workgroup
// reduces a whole chain, so large chains want the largest workgroup.
constexpr int kChainReduceThreads = 1024;

template <typename R>
struct ChainView {
  Planes<R> S, J;
  int32_t L, Lh;
  int64_t Nh;
};

template <typename R>
__device__ __forceinline__ ChainView<R> chain_view(const hsg_chain& ch, R* spins_base,
                                                   R* J_base) {
  ChainView<R> v;
  v.L = ch.L;
  v.Lh = ch.L / 2;
  v.Nh = (int64_t)v.Lh * v.L * v.L;
  v.S = planes_of<R>(spins_base + ch.spin_offset, v.Nh);
  v.J = planes_of<R>(J_base + ch.J_offset, v.Nh);
  return v;
}

template <typename R>
struct BatchArgs {
  const hsg_chain* chains;
  R* spins;
  R* J;
  const double* beta;
  double* E;
  uint32_t* sweep;
  int32_t* remaining;
  const int32_t* order;
  int32_t n_chains;
  int32_t n_sweeps;
};

// Site ic of colour COLOUR of a chain and its neighbours.
template <typename R, int COLOUR>
__device__ __forceinline__ SiteOffsets chain_site(const ChainView<R>& v, uint32_t ic,
                                                  const SmallDiv& by_lh, const SmallDiv& by_l) {
  const uint32_t row = by_lh.div(ic), z = by_l.div(row);
  return site_offsets<R>((uint32_t)v.L, (uint32_t)v.Lh, COLOUR, ic, ic - row * (uint32_t)v.Lh,
                         row - z * (uint32_t)v.L, z);
}

// One colour pass of mode MODE over a chain, spread over the workgroup.  The colour
// is a compile-time constant, so the site update addresses its planes with constant
// indices (no pointer table in scratch memory, global rather than flat loads).
template <typename R, PassMode MODE, int COLOUR>
__device__ __forceinline__ double chain_pass(const ChainView<R>& v, const HitCtx<R>& hc,
                                             const SmallDiv& by_lh, const SmallDiv& by_l) {
  double dE = 0.0;
  for (uint32_t ic = threadIdx.x; ic < (uint32_t)v.Nh; ic += blockDim.x)
    dE += update_site<R, MODE>(v.S, v.J, COLOUR, chain_site<R, COLOUR>(v, ic, by_lh, by_l), hc);
  return dE;
}

// Value every lane of the wave holds the same copy of, made visibly uniform (scalar)
// for the compiler: loop bounds and exits that contain workgroup barriers must be.
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t uniform(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)v);
}

// Element i (wave-uniform) of a table that no kernel writes while this one runs: read
// through the constant address space, so that it is one scalar load.  A tile's table
// entry, its chain and the chain's state hang on one another; as vector loads these three
// round trips and the fourteen words moved to scalar registers were half of a short pass.
template <typename T>
__device__ __forceinline__ T uniform_ld(const T* table, int32_t i) {
  typedef const T __attribute__((address_space(4))) * ConstPtr;
  return ((ConstPtr)(uintptr_t)table)[i];
}

// The chain table entry, every field scalar.
__device__ __forceinline__ hsg_chain load_chain(const hsg_chain* chains, int32_t ci) {
  hsg_chain u;
  const hsg_chain* c = chains + uniform(ci);
  u.spin_offset = uniform_ld(&c->spin_offset, 0);
  u.J_offset = uniform_ld(&c->J_offset, 0);
  u.seed = uniform_ld(&c->seed, 0);
  u.J_seed = 0;  // read by the initial state only
  u.L = uniform_ld(&c->L, 0);
  u.k_hits = uniform_ld(&c->k_hits, 0);
  u.n_or = uniform_ld(&c->n_or, 0);
  u.renorm_every = uniform_ld(&c->renorm_every, 0);
  u.flags = uniform_ld(&c->flags, 0);
  u.reserved = 0;
  return u;
}

// One workgroup per chain: workgroup b advances chain order[b].  The hardware
// dispatcher hands workgroups to compute units as they free up, in order, so the
// caller's order (largest lattices first) balances chains of uneven size without a
// software queue, and every loop that contains a barrier has uniform bounds.
template <typename R>
__global__ __launch_bounds__(1024) void batch_sweep_kernel(BatchArgs<R> a) {
  __shared__ double s_red[16];
  const int32_t ci = uniform(a.order[blockIdx.x]);
  const hsg_chain ch = load_chain(a.chains, ci);
  const ChainView<R> v = chain_view<R>(ch, a.spins, a.J);
  const SmallDiv by_lh((uint32_t)v.Lh), by_l((uint32_t)v.L);
  int32_t n = a.n_sweeps;
  if (a.remaining) n = uniform(min(n, a.remaining[ci]));
  HitCtx<R> hc;
  hc.beta = (R)a.beta[ci];
  hc.k_hits = ch.k_hits;
  hc.seed_lo = (uint32_t)ch.seed;
  hc.seed_hi = (uint32_t)(ch.seed >> 32);
  const uint32_t sweep0 = uniform(a.sweep[ci]);
  const bool heat = (ch.flags & HSG_HEAT_BATH) != 0;
  double dE = 0.0;
  for (int32_t s = 0; s < n; ++s) {
    hc.sweep = sweep0 + (uint32_t)s;
    for (int32_t phase = 0; phase <= ch.n_or; ++phase) {
      if (phase == 0 && ch.k_hits == 0) continue;
      hc.phase = (uint32_t)phase;
      if (phase > 0) {
        chain_pass<R, PassMode::OverRelax, 0>(v, hc, by_lh, by_l);
        __syncthreads();
        chain_pass<R, PassMode::OverRelax, 1>(v, hc, by_lh, by_l);
      } else if (heat) {
        dE += chain_pass<R, PassMode::HeatBath, 0>(v, hc, by_lh, by_l);
        __syncthreads();
        dE += chain_pass<R, PassMode::HeatBath, 1>(v, hc, by_lh, by_l);
      } else if (ch.k_hits % 4 == 0) {  // every group of four hits complete
        dE += chain_pass<R, PassMode::MetropolisFull, 0>(v, hc, by_lh, by_l);
        __syncthreads();
        dE += chain_pass<R, PassMode::MetropolisFull, 1>(v, hc, by_lh, by_l);
      } else {
        dE += chain_pass<R, PassMode::Metropolis, 0>(v, hc, by_lh, by_l);
        __syncthreads();
        dE += chain_pass<R, PassMode::Metropolis, 1>(v, hc, by_lh, by_l);
      }
      __syncthreads();
    }
    if (ch.renorm_every > 0 && (hc.sweep + 1u) % (uint32_t)ch.renorm_every == 0u) {
      for (uint32_t e = threadIdx.x; e < 2u * (uint32_t)v.Nh; e += blockDim.x) {
        const int c = e >= (uint32_t)v.Nh ? 1 : 0;
        renormalise_spin(v.S, c, (int64_t)e - c * v.Nh);
      }
      __syncthreads();
    }
  }
  const double total = block_sum(dE, s_red);
  if (threadIdx.x == 0) {
    a.E[ci] += total;
    a.sweep[ci] = sweep0 + (uint32_t)n;
    if (a.remaining) a.remaining[ci] -= n;
  }
}

template <typename R>
__global__ __launch_bounds__(256) void batch_init_kernel(const hsg_chain* chains, R* spins,
                                                         R* J) {
  const hsg_chain ch = chains[blockIdx.y];
  const int64_t N = (int64_t)ch.L * ch.L * ch.L;
  R* js = (ch.flags & HSG_CHAIN_INIT_J) ? J + ch.J_offset : nullptr;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < N;
       e += (int64_t)gridDim.x * blockDim.x)
    init_site<R>(ch.L, e, (uint32_t)ch.seed, (uint32_t)(ch.seed >> 32), spins + ch.spin_offset, js,
                 (uint32_t)ch.J_seed, (uint32_t)(ch.J_seed >> 32));
}

// H of a chain, by one workgroup: the colour's index in 32 bits, divided by products.
template <typename R>
__global__ __launch_bounds__(kChainReduceThreads) void batch_energy_kernel(
    const hsg_chain* chains, R* spins, R* J, double* out) {
  __shared__ double s_red[16];
  const ChainView<R> v = chain_view<R>(load_chain(chains, (int32_t)blockIdx.x), spins, J);
  const SmallDiv by_lh((uint32_t)v.Lh), by_l((uint32_t)v.L);
  double acc = 0.0;
  for (uint32_t ic = threadIdx.x; ic < (uint32_t)v.Nh; ic += kChainReduceThreads)
    acc += colour0_bond_sum<R>(v.S, v.J, chain_site<R, 0>(v, ic, by_lh, by_l));
  const double total = block_sum(acc, s_red);
  if (threadIdx.x == 0) out[blockIdx.x] = -total;
}

__host__ __device__ inline uint32_t half_sites(int32_t L) {
  return (uint32_t)(L / 2) * (uint32_t)L * (uint32_t)L;
}

// Overlap of two chains of equal L over the sites [e0, e1) of either colour, reduced by one
// workgroup; its 15 sums divided by `norm` go to out.  A thread takes U sites at a time,
// their loads in flight together (one compute unit reads them all: the loop is bound by the
// latency of its loads, and for large chains by what it can load, 170 GB/s); the waves' sums
// are added in order, all 15 at once.
template <typename R>
__device__ __forceinline__ void pair_overlap(const hsg_chain& ca, const hsg_chain& cb,
                                             const R* spins, uint32_t e0, uint32_t e1,
                                             double norm, double* out) {
  constexpr int kWaves = kChainReduceThreads / 64;
  constexpr int U = sizeof(R) == 4 ? 4 : 2;
  __shared__ double part[kWaves][16];
  const uint32_t Nh = half_sites(ca.L);
  const R* a = spins + ca.spin_offset;
  const R* b = spins + cb.spin_offset;
  double v[15] = {0.0};
  auto add = [&](const R* av, const R* bv) {
    const double x[3] = {(double)av[0], (double)av[1], (double)av[2]};
    const double y[3] = {(double)bv[0], (double)bv[1], (double)bv[2]};
#pragma unroll
    for (int m = 0; m < 3; ++m) {
#pragma unroll
      for (int n = 0; n < 3; ++n) v[3 * m + n] = fma(x[m], y[n], v[3 * m + n]);
      v[9 + m] += x[m];
      v[12 + m] += y[m];
    }
  };
  for (int c = 0; c < 2; ++c) {
    const R* ac = a + 3 * c * Nh;
    const R* bc = b + 3 * c * Nh;
    uint32_t e = e0 + threadIdx.x;
    for (; e + (U - 1) * kChainReduceThreads < e1; e += U * kChainReduceThreads) {
      R av[U][3], bv[U][3];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          av[u][k] = ac[k * Nh + e + u * kChainReduceThreads];
          bv[u][k] = bc[k * Nh + e + u * kChainReduceThreads];
        }
#pragma unroll
      for (int u = 0; u < U; ++u) add(av[u], bv[u]);
    }
    for (; e < e1; e += kChainReduceThreads) {
      const R av[3] = {ac[e], ac[Nh + e], ac[2 * Nh + e]};
      const R bv[3] = {bc[e], bc[Nh + e], bc[2 * Nh + e]};
      add(av, bv);
    }
  }
#pragma unroll
  for (int k = 0; k < 15; ++k) {
    const double t = wave_sum(v[k]);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][k] = t;
  }
  __syncthreads();
  if (threadIdx.x < 15) {
    double t = 0.0;
    for (int w = 0; w < kWaves; ++w) t += part[w][threadIdx.x];
    out[threadIdx.x] = t / norm;
  }
}

template <typename R>
__device__ __forceinline__ void pair_overlap(const hsg_chain& ca, const hsg_chain& cb,
                                             const R* spins, double* out) {
  const uint32_t Nh = half_sites(ca.L);
  pair_overlap<R>(ca, cb, spins, 0u, Nh, 2.0 * (double)Nh, out);
}

template <typename R>
__global__ __launch_bounds__(kChainReduceThreads) void chain_pairs_overlap_kernel(
    const hsg_chain* chains, const R* spins, const int32_t* pairs, double* out) {
  const int32_t p = blockIdx.x;
  pair_overlap<R>(chains[pairs[2 * p]], chains[pairs[2 * p + 1]], spins, out + 15 * (int64_t)p);
}

// The same and H of a chain in parts of 8192 sites of a colour, a workgroup each, whose
// sums are then added in order: a chain's result depends on nothing but the chain.  A
// workgroup alone took 255 us for the overlaps of a few chains of up to L = 96 and 755 for
// the energies of 48 (bound by what its compute unit can load); 54 to a chain take 16 and 84.
// Up to L = 48 a chain is one part: it is read in 10 to 20 us, and served lattices of L <= 32
// lost more to the second launch than the parts gave (20 of them, 8 to 32 sweeps each: 1152 us
// in parts, 1093 without).
__host__ __device__ inline uint32_t part_sites(int32_t L) { return L <= 48 ? 55296u : 8192u; }
__host__ __device__ inline int32_t chain_parts(int32_t L) {
  return (int32_t)((half_sites(L) + part_sites(L) - 1u) / part_sites(L));
}
template <typename R>
__global__ __launch_bounds__(kChainReduceThreads) void chain_pairs_part_kernel(
    const hsg_chain* chains, const R* spins, const int32_t* pairs, double* parts) {
  const int32_t p = (int32_t)blockIdx.y, part = (int32_t)blockIdx.x;
  const hsg_chain& ca = chains[pairs[2 * p]];
  const uint32_t Nh = half_sites(ca.L), n = part_sites(ca.L), e0 = (uint32_t)part * n;
  if (e0 >= Nh) return;
  pair_overlap<R>(ca, chains[pairs[2 * p + 1]], spins, e0, min(e0 + n, Nh), 1.0,
                  parts + 15 * ((int64_t)p * gridDim.x + part));
}
constexpr int kSumThreads = 256;  // 16 partial sums of a record's 15 values, then theirs
__global__ __launch_bounds__(kSumThreads) void chain_pairs_sum_kernel(
    const hsg_chain* chains, const int32_t* pairs, const double* parts, int32_t stride,
    double* out) {
  __shared__ double part[16][16];
  const int32_t p = (int32_t)blockIdx.x, i = (int32_t)threadIdx.x & 15,
                g = (int32_t)threadIdx.x >> 4;
  const int32_t L = chains[pairs[2 * p]].L, n = min(chain_parts(L), stride);
  double t = 0.0;
  if (i < 15)
    for (int32_t k = g; k < n; k += 16) t += parts[15 * ((int64_t)p * stride + k) + i];
  part[g][i] = t;
  __syncthreads();
  if (threadIdx.x < 15) {
    t = 0.0;
    for (int k = 0; k < 16; ++k) t += part[k][threadIdx.x];
    out[15 * (int64_t)p + threadIdx.x] = t / (2.0 * (double)half_sites(L));
  }
}
template <typename R>
__global__ __launch_bounds__(kChainReduceThreads) void batch_energy_part_kernel(
    const hsg_chain* chains, R* spins, R* J, double* parts) {
  __shared__ double s_red[16];
  const int32_t c = (int32_t)blockIdx.y, part = (int32_t)blockIdx.x;
  const ChainView<R> v = chain_view<R>(load_chain(chains, c), spins, J);
  const uint32_t n = part_sites(v.L), e0 = (uint32_t)part * n, e1 = min(e0 + n, (uint32_t)v.Nh);
  if (e0 >= e1) return;
  const SmallDiv by_lh((uint32_t)v.Lh), by_l((uint32_t)v.L);
  double acc = 0.0;
  for (uint32_t ic = e0 + threadIdx.x; ic < e1; ic += kChainReduceThreads)
    acc += colour0_bond_sum<R>(v.S, v.J, chain_site<R, 0>(v, ic, by_lh, by_l));
  const double total = block_sum(acc, s_red);
  if (threadIdx.x == 0) parts[(int64_t)c * gridDim.x + part] = total;
}
__global__ __launch_bounds__(kSumThreads) void batch_energy_sum_kernel(const hsg_chain* chains,
                                                                       const double* parts,
                                                                       int32_t stride,
                                                                       double* out) {
  __shared__ double s_red[16];
  const int32_t c = (int32_t)blockIdx.x, n = min(chain_parts(chains[c].L), stride);
  double t = 0.0;
  for (int32_t k = (int32_t)threadIdx.x; k < n; k += kSumThreads)
    t += parts[(int64_t)c * stride + k];
  const double total = block_sum(t, s_red);
  if (threadIdx.x == 0) out[c] = -total;
}

template <typename R>
__global__ __launch_bounds__(kChainReduceThreads) void ladder_pairs_overlap_kernel(
    const hsg_chain* chains, const R* spins, const int32_t* chain_at_slot, int32_t n_temps,
    const int32_t* ladder_pairs, double* out) {
  const int32_t p = blockIdx.x, t = blockIdx.y;
  const int32_t la = ladder_pairs[2 * p], lb = ladder_pairs[2 * p + 1];
  const int32_t a = chain_at_slot[(int64_t)la * n_temps + t];
  const int32_t b = chain_at_slot[(int64_t)lb * n_temps + t];
  pair_overlap<R>(chains[a], chains[b], spins, out + 15 * ((int64_t)p * n_temps + t));
}

// One exchange round: a thread per slot of every ladder.  Round n pairs the slots (t, t+1)
// with t = n mod 2, t + 2, ...; the pairs of a round share no slot, so the thread of a
// pair's lower slot decides the swap and sets both temperatures, and a slot without a
// partner keeps its own.  With `bump` (one workgroup) the round counter is advanced here,
// after every thread has read it.  (A thread per ladder walked its pairs one dependent
// load after another: 9.6 us for 24 temperatures.)
constexpr int kExchangeThreads = 256;
__global__ __launch_bounds__(kExchangeThreads) void pt_exchange_kernel(
    int32_t n_ladders, int32_t n_temps, int32_t* chain_at_slot, const double* beta_of_slot,
    int32_t* accepted, uint32_t seed_lo, uint32_t seed_hi, uint32_t* round_ctr, const double* E,
    double* beta, int32_t bump) {
  const int64_t i = blockIdx.x * (int64_t)kExchangeThreads + threadIdx.x;
  const uint32_t round = *round_ctr;
  if (bump) {
    __syncthreads();
    if (threadIdx.x == 0) *round_ctr = round + 1u;
  }
  if (i >= (int64_t)n_ladders * n_temps) return;
  const int32_t l = (int32_t)(i / n_temps), t = (int32_t)(i - (int64_t)l * n_temps);
  const int32_t parity = (int32_t)(round & 1u);
  int32_t* slots = chain_at_slot + (int64_t)l * n_temps;
  const bool lower = t >= parity && ((t - parity) & 1) == 0;  // lower slot of a pair, if any
  if (!lower && t > parity) return;                           // upper slot: its partner's work
  int32_t ca = slots[t];
  if (lower && t + 1 < n_temps) {
    int32_t cb = slots[t + 1];
    const double delta = (beta_of_slot[t] - beta_of_slot[t + 1]) * (E[ca] - E[cb]);
    const Word4 w = philox10((uint32_t)t, round, (uint32_t)l, kTagSwap, seed_lo, seed_hi);
    const double u = unit_uniform<double>(w.w0);
    if (delta >= 0.0 || u < exp(delta)) {
      slots[t] = cb;
      slots[t + 1] = ca;
      if (accepted) accepted[(int64_t)l * n_temps + t] += 1;
      const int32_t c = ca;
      ca = cb;
      cb = c;
    }
    beta[cb] = beta_of_slot[t + 1];
  }
  beta[ca] = beta_of_slot[t];
}

__global__ void bump_round_kernel(uint32_t* round_ctr) { *round_ctr += 1u; }

// ------------------------------------------------------------------------------------
// Multi-lattice colour pass: one launch updates colour c of every listed chain.  Tile
// t covers blockDim.x consecutive colour sites of one chain; chains that have used up
// their budget, or do not have this phase, return at once.

template <typename R>
struct MultiPassArgs {
  const hsg_chain* chains;
  R* spins;
  R* J;
  const double* beta;
  double* E;
  const uint32_t* sweep;
  const int32_t* remaining;  // NULL: every chain runs all the call's sweeps
  const int32_t* tiles;
  double* partials;  // a double per tile that takes its energy changes, or NULL: atomics on E
  int32_t n_tiles;
  int32_t s;  // sweep offset within the call
  int32_t phase;
  int32_t colour;
  int32_t reverse;
};

template <typename R, int COLOUR>
__global__ __launch_bounds__(1024) void multi_pass_kernel(MultiPassArgs<R> a) {
  __shared__ double s_red[16];
  int32_t t = xcd_tile((int32_t)blockIdx.x, a.n_tiles);
  if (a.reverse) t = a.n_tiles - 1 - t;
  t = uniform(t);
  const int32_t ci = uniform_ld(a.tiles, 2 * t), ic0 = uniform_ld(a.tiles, 2 * t + 1);
  if (a.remaining && a.s >= uniform_ld(a.remaining, ci)) return;
  const hsg_chain ch = load_chain(a.chains, ci);
  if ((a.phase == 0 && ch.k_hits == 0) || a.phase > ch.n_or) return;
  const ChainView<R> v = chain_view<R>(ch, a.spins, a.J);
  const uint32_t ic = (uint32_t)ic0 + threadIdx.x;
  HitCtx<R> hc;
  hc.beta = (R)uniform_ld(a.beta, ci);
  hc.k_hits = ch.k_hits;
  hc.seed_lo = (uint32_t)ch.seed;
  hc.seed_hi = (uint32_t)(ch.seed >> 32);
  hc.sweep = uniform_ld(a.sweep, ci) + (uint32_t)a.s;
  hc.phase = (uint32_t)a.phase;
  double dE = 0.0;
  if (ic < (uint32_t)v.Nh) {
    const SmallDiv by_lh((uint32_t)v.Lh), by_l((uint32_t)v.L);
    const SiteOffsets o = chain_site<R, COLOUR>(v, ic, by_lh, by_l);
    if (a.phase > 0)
      update_site<R, PassMode::OverRelax>(v.S, v.J, COLOUR, o, hc);
    else if (ch.flags & HSG_HEAT_BATH)
      dE = update_site<R, PassMode::HeatBath>(v.S, v.J, COLOUR, o, hc);
    else if (ch.k_hits % 4 == 0)  // every group of four hits complete
      dE = update_site<R, PassMode::MetropolisFull>(v.S, v.J, COLOUR, o, hc);
    else
      dE = update_site<R, PassMode::Metropolis>(v.S, v.J, COLOUR, o, hc);
  }
  if (a.phase == 0) {
    const double total = block_sum(dE, s_red);
    if (threadIdx.x == 0 && total != 0.0) {
      if (a.partials)
        atomicAdd(&a.partials[t], total);  // its only writer
      else
        atomicAdd(&a.E[ci], total);
    }
  }
}

// Renormalisation after sweep offset s for the chains whose schedule asks for it.
template <typename R>
__global__ __launch_bounds__(1024) void multi_renorm_kernel(const hsg_chain* chains, R* spins,
                                                            const uint32_t* sweep,
                                                            const int32_t* remaining,
                                                            const int32_t* tiles, int32_t s) {
  const int32_t t = blockIdx.x;
  const int32_t ci = uniform_ld(tiles, 2 * t), ic0 = uniform_ld(tiles, 2 * t + 1);
  if (remaining && s >= uniform_ld(remaining, ci)) return;
  const hsg_chain ch = load_chain(chains, ci);
  if (ch.renorm_every <= 0 ||
      (uniform_ld(sweep, ci) + (uint32_t)s + 1u) % (uint32_t)ch.renorm_every != 0u)
    return;
  const int64_t Nh = (int64_t)(ch.L / 2) * ch.L * ch.L;
  const Planes<R> S = planes_of<R>(spins + ch.spin_offset, Nh);
  const int64_t e = (int64_t)ic0 + threadIdx.x;
  if (e < Nh) {
    renormalise_spin(S, 0, e);
    renormalise_spin(S, 1, e);
  }
}

// Advances every chain's sweep counter and budget by the sweeps it ran.
__global__ void multi_finish_kernel(int32_t n_chains, uint32_t* sweep, int32_t* remaining,
                                    int32_t n_sweeps) {
  const int32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n_chains) return;
  const int32_t n = min(n_sweeps, remaining[c]);
  if (n > 0) {
    sweep[c] += (uint32_t)n;
    remaining[c] -= n;
  }
}

// The same with partials: workgroup c also adds the partials of chain c's tiles (a fixed
// order, then zeroed) to its energy.
__global__ __launch_bounds__(256) void tile_finish_kernel(const int32_t* first_tile,
                                                          double* partials, double* E,
                                                          uint32_t* sweep, int32_t* remaining,
                                                          int32_t n_sweeps) {
  __shared__ double s_red[16];
  const int32_t c = (int32_t)blockIdx.x;
  const int32_t t1 = first_tile[c + 1];
  if (t1 == first_tile[c]) return;  // not a chain of this call
  double acc = 0.0;
  for (int32_t t = first_tile[c] + (int32_t)threadIdx.x; t < t1; t += 256) {
    acc += partials[t];
    partials[t] = 0.0;
  }
  const double total = block_sum(acc, s_red);
  if (threadIdx.x == 0) {
    E[c] += total;
    const int32_t n = remaining ? min(n_sweeps, remaining[c]) : n_sweeps;
    if (n > 0) {
      sweep[c] += (uint32_t)n;
      if (remaining) remaining[c] -= n;
    }
  }
}

}  // namespace

template <typename R>
hipError_t launch_batch_init(const hsg_batch* b, hipStream_t st) {
  hipLaunchKernelGGL(batch_init_kernel<R>, dim3(64, (unsigned)b->n_chains), dim3(256), 0, st,
                     b->chains, (R*)b->spins, (R*)b->J);
  hipLaunchKernelGGL(batch_energy_kernel<R>, dim3((unsigned)b->n_chains),
                     dim3(kChainReduceThreads), 0, st,
                     b->chains, (R*)b->spins, (R*)b->J, b->E);
  return hipGetLastError();
}

int32_t batch_parts(int32_t L) { return chain_parts(L); }

template <typename R>
hipError_t launch_batch_init_parts(const hsg_batch* b, int32_t parts, double* scratch,
                                   hipStream_t st) {
  hipLaunchKernelGGL(batch_init_kernel<R>, dim3(64, (unsigned)b->n_chains), dim3(256), 0, st,
                     b->chains, (R*)b->spins, (R*)b->J);
  hipLaunchKernelGGL(batch_energy_part_kernel<R>, dim3((unsigned)parts, (unsigned)b->n_chains),
                     dim3(kChainReduceThreads), 0, st, b->chains, (R*)b->spins, (R*)b->J, scratch);
  hipLaunchKernelGGL(batch_energy_sum_kernel, dim3((unsigned)b->n_chains), dim3(kSumThreads), 0,
                     st, b->chains, (const double*)scratch, parts, b->E);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_batch_overlap_parts(const hsg_batch* b, const int32_t* pairs, int32_t n_pairs,
                                      int32_t parts, double* scratch, double* out,
                                      hipStream_t st) {
  hipLaunchKernelGGL(chain_pairs_part_kernel<R>, dim3((unsigned)parts, (unsigned)n_pairs),
                     dim3(kChainReduceThreads), 0, st, b->chains, (const R*)b->spins, pairs,
                     scratch);
  hipLaunchKernelGGL(chain_pairs_sum_kernel, dim3((unsigned)n_pairs), dim3(kSumThreads), 0, st,
                     b->chains, pairs, (const double*)scratch, parts, out);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_batch_sweep(const hsg_batch* b, int32_t n_sweeps, hipStream_t st) {
  BatchArgs<R> a;
  a.chains = b->chains;
  a.spins = (R*)b->spins;
  a.J = (R*)b->J;
  a.beta = b->beta;
  a.E = b->E;
  a.sweep = b->sweep;
  a.remaining = b->remaining;
  a.order = b->order;
  a.n_chains = b->n_chains;
  a.n_sweeps = n_sweeps;
  const int threads = b->threads > 0 ? b->threads : 256;
  hipLaunchKernelGGL(batch_sweep_kernel<R>, dim3((unsigned)b->n_chains), dim3((unsigned)threads), 0, st,
                     a);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_batch_energy(const hsg_batch* b, double* out, hipStream_t st) {
  hipLaunchKernelGGL(batch_energy_kernel<R>, dim3((unsigned)b->n_chains),
                     dim3(kChainReduceThreads), 0, st,
                     b->chains, (R*)b->spins, (R*)b->J, out);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_batch_overlap(const hsg_batch* b, const int32_t* pairs, int32_t n_pairs,
                                double* out, hipStream_t st) {
  hipLaunchKernelGGL(chain_pairs_overlap_kernel<R>, dim3((unsigned)n_pairs),
                     dim3(kChainReduceThreads), 0, st,
                     b->chains, (const R*)b->spins, pairs, out);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_pt_overlap(const hsg_pt* pt, const hsg_batch* b, const int32_t* ladder_pairs,
                             int32_t n_pairs, double* out, hipStream_t st) {
  hipLaunchKernelGGL(ladder_pairs_overlap_kernel<R>, dim3((unsigned)n_pairs, (unsigned)pt->n_temps),
                     dim3(kChainReduceThreads), 0, st, b->chains, (const R*)b->spins,
                     pt->chain_at_slot,
                     pt->n_temps, ladder_pairs, out);
  return hipGetLastError();
}

hipError_t launch_pt_exchange(const hsg_pt* pt, const hsg_batch* b, hipStream_t st) {
  const int64_t slots = (int64_t)pt->n_ladders * pt->n_temps;
  const unsigned blocks = (unsigned)((slots + kExchangeThreads - 1) / kExchangeThreads);
  const int32_t bump = blocks == 1 ? 1 : 0;
  hipLaunchKernelGGL(pt_exchange_kernel, dim3(blocks), dim3(kExchangeThreads), 0, st,
                     pt->n_ladders, pt->n_temps, pt->chain_at_slot, pt->beta_of_slot, pt->accepted,
                     (uint32_t)pt->seed, (uint32_t)(pt->seed >> 32), pt->round,
                     (const double*)b->E, b->beta, bump);
  if (!bump) hipLaunchKernelGGL(bump_round_kernel, dim3(1), dim3(1), 0, st, pt->round);
  return hipGetLastError();
}

// The colour passes of n_sweeps sweeps, a launch each over the tiles, and the
// renormalisations between them.
template <typename R>
static void launch_tile_passes(const hsg_batch* b, const int32_t* tiles, double* partials,
                               int32_t n_tiles, int32_t tile_sites, int32_t first_phase,
                               int32_t max_n_or, int32_t renorm, int32_t n_sweeps,
                               hipStream_t st) {
  MultiPassArgs<R> a;
  a.chains = b->chains;
  a.spins = (R*)b->spins;
  a.J = (R*)b->J;
  a.beta = b->beta;
  a.E = b->E;
  a.sweep = b->sweep;
  a.remaining = b->remaining;
  a.tiles = tiles;
  a.partials = partials;
  a.n_tiles = n_tiles;
  const dim3 grid((unsigned)n_tiles), block((unsigned)tile_sites);
  int32_t pass = 0;
  for (int32_t s = 0; s < n_sweeps; ++s) {
    a.s = s;
    for (int32_t phase = first_phase; phase <= max_n_or; ++phase) {
      a.phase = phase;
      for (int32_t colour = 0; colour < 2; ++colour) {
        a.colour = colour;
        a.reverse = pass++ & 1;
        if (colour == 0)
          hipLaunchKernelGGL((multi_pass_kernel<R, 0>), grid, block, 0, st, a);
        else
          hipLaunchKernelGGL((multi_pass_kernel<R, 1>), grid, block, 0, st, a);
      }
    }
    if (renorm)
      hipLaunchKernelGGL(multi_renorm_kernel<R>, grid, block, 0, st, b->chains, (R*)b->spins,
                         (const uint32_t*)b->sweep, (const int32_t*)b->remaining, tiles, s);
  }
}

template <typename R>
hipError_t launch_batch_pass_sweep(const hsg_batch* b, const int32_t* tiles, int32_t n_tiles,
                                   int32_t tile_sites, int32_t max_n_or, int32_t renorm,
                                   int32_t n_sweeps, hipStream_t st) {
  launch_tile_passes<R>(b, tiles, nullptr, n_tiles, tile_sites, 0, max_n_or, renorm, n_sweeps, st);
  hipLaunchKernelGGL(multi_finish_kernel, dim3((unsigned)((b->n_chains + 255) / 256)), dim3(256), 0,
                     st, b->n_chains, b->sweep, b->remaining, n_sweeps);
  return hipGetLastError();
}

// A workgroup writes the tiles of one chain: a million of them for 12288 chains, which took
// 4 ms to make on the host and as long to send.
__global__ __launch_bounds__(256) void tile_table_kernel(const int32_t* first_tile,
                                                         int32_t tile_sites, int32_t* tiles,
                                                         double* partials) {
  const int32_t c = (int32_t)blockIdx.x, t0 = first_tile[c], t1 = first_tile[c + 1];
  for (int32_t t = t0 + (int32_t)threadIdx.x; t < t1; t += 256) {
    reinterpret_cast<int2*>(tiles)[t] = make_int2(c, (t - t0) * tile_sites);
    partials[t] = 0.0;
  }
}
hipError_t launch_tile_table(const int32_t* first_tile, int32_t n_chains, int32_t tile_sites,
                             int32_t* tiles, double* partials, hipStream_t st) {
  hipLaunchKernelGGL(tile_table_kernel, dim3((unsigned)n_chains), dim3(256), 0, st, first_tile,
                     tile_sites, tiles, partials);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_batch_tile_sweep(const hsg_batch* b, const int32_t* tiles,
                                   const int32_t* first_tile, const int32_t* groups,
                                   int32_t n_groups, int32_t tile_sites, double* partials,
                                   int32_t first_phase, int32_t max_n_or, int32_t renorm,
                                   int32_t n_sweeps, hipStream_t st) {
  for (int32_t g = 0; g < n_groups; ++g)
    launch_tile_passes<R>(b, tiles + 2 * (int64_t)groups[g], partials + groups[g],
                          groups[g + 1] - groups[g], tile_sites, first_phase, max_n_or, renorm,
                          n_sweeps, st);
  hipLaunchKernelGGL(tile_finish_kernel, dim3((unsigned)b->n_chains), dim3(256), 0, st, first_tile,
                     partials, b->E, b->sweep, b->remaining, n_sweeps);
  return hipGetLastError();
}

#define HSG_BATCH_INSTANTIATE(R)                                                              \
  template hipError_t launch_batch_init<R>(const hsg_batch*, hipStream_t);                    \
  template hipError_t launch_batch_init_parts<R>(const hsg_batch*, int32_t, double*,          \
                                                 hipStream_t);                                 \
  template hipError_t launch_batch_overlap_parts<R>(const hsg_batch*, const int32_t*, int32_t, \
                                                    int32_t, double*, double*, hipStream_t);   \
  template hipError_t launch_batch_sweep<R>(const hsg_batch*, int32_t, hipStream_t);           \
  template hipError_t launch_batch_energy<R>(const hsg_batch*, double*, hipStream_t);         \
  template hipError_t launch_batch_overlap<R>(const hsg_batch*, const int32_t*, int32_t,      \
                                              double*, hipStream_t);                          \
  template hipError_t launch_pt_overlap<R>(const hsg_pt*, const hsg_batch*, const int32_t*,   \
                                           int32_t, double*, hipStream_t);                     \
  template hipError_t launch_batch_pass_sweep<R>(const hsg_batch*, const int32_t*, int32_t,   \
                                                 int32_t, int32_t, int32_t, int32_t, hipStream_t); \
  template hipError_t launch_batch_tile_sweep<R>(const hsg_batch*, const int32_t*,             \
                                                 const int32_t*, const int32_t*, int32_t,       \
                                                 int32_t, double*, int32_t, int32_t, int32_t,   \
                                                 int32_t, hipStream_t);
HSG_BATCH_INSTANTIATE(float)
HSG_BATCH_INSTANTIATE(double)

}  // namespace hsg
