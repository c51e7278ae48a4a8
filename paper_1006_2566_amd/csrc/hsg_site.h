// One colour-pass update of one site: gather the local field of eq. (2) from the six
// other-colour neighbours, then apply k Metropolis hits, k heat-bath draws or one
// over-relaxation step.  Shared by the single-lattice colour-pass kernel and the
// batched kernel, so a lattice gives the same bits alone or inside a batch.
#pragma once

#include "hsg_device.h"
#include "hsg_internal.h"

namespace hsg {

// Position of internal element e (0 <= e < N) of the colour-split layout.
struct SiteOf {
  int32_t c, xh, y, z, x;
  int64_t ic;         // index within the colour's planes
  uint32_t canon;     // x + L*y + L*L*z
};

__device__ __forceinline__ SiteOf site_of(int64_t e, int32_t L) {
  const int32_t Lh = L / 2;
  const int64_t Nh = (int64_t)Lh * L * L;
  SiteOf s;
  s.c = e >= Nh ? 1 : 0;
  s.ic = e - (int64_t)s.c * Nh;
  s.xh = (int32_t)(s.ic % Lh);
  const int64_t r = s.ic / Lh;
  s.y = (int32_t)(r % L);
  s.z = (int32_t)(r / L);
  s.x = 2 * s.xh + ((s.y + s.z + s.c) & 1);
  s.canon = (uint32_t)s.x + (uint32_t)L * ((uint32_t)s.y + (uint32_t)L * (uint32_t)s.z);
  return s;
}

// Random initial state of internal element e (0 <= e < N) of an L^3 lattice:
// spin uniform on the sphere from Philox tag 1; couplings (when J is not NULL) by
// Box-Muller from tag 2: (u0,u1) -> Jx, Jy; (u2,u3) -> Jz.  Counter (0, site, 0, tag).
template <typename R>
__device__ __forceinline__ void init_site(int32_t L, int64_t e, uint32_t k0, uint32_t k1,
                                          R* spins, R* J, uint32_t jk0, uint32_t jk1) {
  const int64_t Nh = (int64_t)L * L * L / 2;
  const SiteOf st = site_of(e, L);
  const Word4 ws = philox10(0u, st.canon, 0u, kTagInitSpin, k0, k1);
  const Vec3<R> s = sphere_point(unit_uniform<R>(ws.w0), unit_uniform<R>(ws.w1));
  const int64_t base = (int64_t)3 * st.c * Nh + st.ic;
  spins[base] = s.x;
  spins[base + Nh] = s.y;
  spins[base + 2 * Nh] = s.z;
  if (!J) return;
  const Word4 wj = philox10(0u, st.canon, 0u, kTagInitJ, jk0, jk1);
  R sn, cs;
  const R r01 = dev_sqrt((R)-2 * own_log(unit_uniform<R>(wj.w0)));
  sincos_2pi(unit_uniform<R>(wj.w1), sn, cs);
  J[base] = r01 * cs;
  J[base + Nh] = r01 * sn;
  const R r23 = dev_sqrt((R)-2 * own_log(unit_uniform<R>(wj.w2)));
  sincos_2pi(unit_uniform<R>(wj.w3), sn, cs);
  J[base + 2 * Nh] = r23 * cs;
}

// A site and its six neighbours as offsets into the planes of its colour (own) and of the
// other one: bytes in binary32, where a plane of N/2 <= 2^30 values spans less than 2^32
// bytes for every L the library accepts and the loads take a wave-uniform base and a
// 32-bit offset; elements in binary64.
struct SiteOffsets {
  uint32_t own, px, mx, py, my, pz, mz;
  uint32_t site;  // x + L y + L^2 z
};

template <typename R>
struct OffsetUnit {
  static constexpr uint32_t value = sizeof(R) == 4 ? 4 : 1;
};

// The colour-c site at column xh of row y, plane z, its index in the colour ic = xh +
// Lh (y + L z).  Every neighbour is a step from ic: none or one column in x (which of the
// two depends on the row's parity), a row in y, a plane in z, or back across the lattice at
// its faces; and x + L y + L^2 z = 2 ic + p, since a row holds L = 2 Lh sites.  So a site
// costs a dozen vector operations where forming the rows of its neighbours took forty.
template <typename R>
__device__ __forceinline__ SiteOffsets site_offsets(uint32_t L, uint32_t Lh, uint32_t c,
                                                    uint32_t ic, uint32_t xh, uint32_t y,
                                                    uint32_t z) {
  constexpr uint32_t U = OffsetUnit<R>::value;
  const uint32_t p = (y + z + c) & 1u;  // x = 2 xh + p
  const uint32_t row = Lh * U, plane = Lh * L * U;  // steps in y and z
  const uint32_t odd = 0u - p;                      // all ones when p = 1
  SiteOffsets o;
  o.own = ic * U;
  o.px = o.own + (odd & (xh == Lh - 1 ? U - row : U));
  o.mx = o.own + (~odd & (xh == 0 ? row - U : 0u - U));
  o.py = o.own + (y == L - 1 ? row - plane : row);
  o.my = o.own + (y == 0 ? plane - row : 0u - row);
  o.pz = o.own + (z == L - 1 ? plane - plane * L : plane);
  o.mz = o.own + (z == 0 ? plane * L - plane : 0u - plane);
  o.site = 2u * ic + p;
  return o;
}

// Tile `tile` (wave-uniform) of a colour's sites: its plane z and thread threadIdx.x's site
// i of that plane (none when i >= g.plane).
struct TileSite {
  uint32_t z, i;
};
__device__ __forceinline__ TileSite tile_site(const Geometry& g, uint32_t tile) {
  const uint32_t tp = (uint32_t)g.tiles_p;
  uint32_t z = tile;  // tile / tp: the product with floor(2^32 / tp) is at most one short
  if (tp > 1) {
    z = __umulhi(tile, g.inv_tp);
    z += tile - z * tp >= tp ? 1u : 0u;
  }
  return TileSite{z, (tile - z * tp) * (uint32_t)kPassThreads + threadIdx.x};
}
template <typename R>
__device__ __forceinline__ SiteOffsets tile_site_offsets(const Geometry& g, const TileSite& s,
                                                         uint32_t colour) {
  const uint32_t y = SmallDiv{(uint32_t)g.Lh, g.inv_lh}.div(s.i);
  return site_offsets<R>((uint32_t)g.L, (uint32_t)g.Lh, colour, s.i + s.z * (uint32_t)g.plane,
                         s.i - y * (uint32_t)g.Lh, y, s.z);
}

// Monte Carlo stream of the site: Philox key and the uniform counter words.
template <typename R>
struct HitCtx {
  R beta;
  uint32_t sweep, phase;
  int32_t k_hits;
  uint32_t seed_lo, seed_hi;
};

// Draws of a Monte Carlo update that need neither the site's spin nor its field.
//
// Uniforms: the site's stream in a phase is the words of the Philox blocks b = 0, 1,
// ... with counter (sweep, site, phase << 16 | b, tag), in word order.  Metropolis hit
// j takes uniforms 3j, 3j+1, 3j+2 (polar, azimuth, acceptance), heat-bath draw j takes
// 2j, 2j+1: four hits share three blocks, two draws one block.  The hits are taken in
// such groups (kHits).  A heat-bath draw is always taken and does not depend on the spin
// it replaces, so of k draws only the last counts and only that one is computed.
constexpr int kHits = 4;
template <typename R, PassMode MODE>
struct Draws {
  Vec3<R> trial[kHits];  // trial points of a group of Metropolis hits
  R u[kHits];            // their acceptance uniforms
};
template <typename R>
struct Draws<R, PassMode::OverRelax> {};
template <typename R>
struct Draws<R, PassMode::HeatBath> {
  uint32_t w0, w1;
};

// The words of Metropolis group b0 / 3 (nh >= 1 hits of it taken).
template <bool FULL, typename R>
__device__ __forceinline__ void hit_words(uint32_t (&w)[3 * kHits], uint32_t site, uint32_t b0,
                                          int32_t nh, const HitCtx<R>& hc) {
  constexpr int NB = 3;  // Philox blocks per group
  if (FULL) {
    // a full group: its NB blocks advanced together (philox10_n)
    uint32_t c2[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) c2[i] = (hc.phase << 16) | (b0 + (uint32_t)i);
    Word4 x[NB];
    philox10_n<NB>(hc.sweep, site, c2, kTagMetropolis, hc.seed_lo, hc.seed_hi, x);
    // all words complete here (an empty statement that takes them as operands):
    // without it each block's rounds would be sunk to its first use, behind the
    // previous hit's decision, one chain at a time again
#pragma unroll
    for (int i = 0; i < NB; ++i)
      asm volatile("" : "+v"(x[i].w0), "+v"(x[i].w1), "+v"(x[i].w2), "+v"(x[i].w3));
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      w[4 * i] = x[i].w0;
      w[4 * i + 1] = x[i].w1;
      w[4 * i + 2] = x[i].w2;
      w[4 * i + 3] = x[i].w3;
    }
  } else {
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (i == 0 || 4 * i < 3 * nh) {
        const Word4 x = philox10(hc.sweep, site, (hc.phase << 16) | (b0 + (uint32_t)i),
                                 kTagMetropolis, hc.seed_lo, hc.seed_hi);
        w[4 * i] = x.w0;
        w[4 * i + 1] = x.w1;
        w[4 * i + 2] = x.w2;
        w[4 * i + 3] = x.w3;
      }
  }
}

// The first group's draws of a site.
template <typename R, PassMode MODE>
__device__ __forceinline__ Draws<R, MODE> first_draws(uint32_t site, const HitCtx<R>& hc) {
  Draws<R, MODE> d;
  if constexpr (MODE == PassMode::HeatBath) {
    const uint32_t j = (uint32_t)hc.k_hits - 1u;  // the last draw: uniforms 2j, 2j + 1
    const Word4 x = philox10(hc.sweep, site, (hc.phase << 16) | (j >> 1), kTagHeatBath,
                             hc.seed_lo, hc.seed_hi);
    d.w0 = (j & 1u) ? x.w2 : x.w0;
    d.w1 = (j & 1u) ? x.w3 : x.w1;
  } else if constexpr (MODE != PassMode::OverRelax) {
    constexpr bool kFull = MODE == PassMode::MetropolisFull;
    uint32_t w[3 * kHits];
    hit_words<kFull>(w, site, 0u, hc.k_hits, hc);
#pragma unroll
    for (int g = 0; g < kHits; ++g)
      if (kFull || g < hc.k_hits) {
        d.trial[g] = sphere_point_words<R>(w[3 * g], w[3 * g + 1]);
        d.u[g] = unit_uniform<R>(w[3 * g + 2]);
      }
  }
  return d;
}

// One Metropolis decision: sh = s.h of the current spin.
template <typename R>
__device__ __forceinline__ void decide_hit(Vec3<R>& s, R& sh, double& dE_sum, const Vec3<R>& trial,
                                           R th, R u, R beta) {
  const R dE = sh - th;
  // both conditions formed for every trial: a wave has lanes that need the second
  // one in almost every hit, and a branch around it cost more than it skipped
  const bool accept = (dE <= (R)0) | (u < accept_prob(-beta * dE));
  if (accept) {
    s = trial;
    sh = th;
    dE_sum += (double)dE;
  }
}

// The update of one site given its spin s and local field h (eq. 2): reflection about
// h (over-relaxation), or k Metropolis hits / heat-bath draws with h fixed.  s is
// replaced in place; returns the sum of the accepted energy changes.
//
// A hit's draws, trial spin and trial energy do not depend on earlier decisions, only its
// accept/reject step does; with G > 1 a group's trials are formed first (instruction-level
// parallelism for a wave with few neighbours on its SIMD), then its decisions in order;
// with `first` the first group's draws were made before the field was known.  Every
// operation and the order of the energy sum are the same for any of these.
template <typename R, PassMode MODE, int G = 1>
__device__ __forceinline__ double apply_update(Vec3<R>& s, const Vec3<R>& h, uint32_t site,
                                               const HitCtx<R>& hc,
                                               const Draws<R, MODE>* first = nullptr) {
  double dE_sum = 0.0;
  if constexpr (MODE == PassMode::OverRelax) {
    s = reflect(s, h);
  } else if constexpr (MODE == PassMode::HeatBath) {
    const Draws<R, MODE> d = first ? *first : first_draws<R, MODE>(site, hc);
    const Vec3<R> t = heat_bath_point(h, hc.beta, unit_uniform<R>(d.w0), unit_uniform<R>(d.w1));
    const R dE = dot3(s, h) - dot3(t, h);
    s = t;
    dE_sum = (double)dE;
  } else {
    // every group complete (k_hits a multiple of four): no per-group conditions
    constexpr bool kFull = MODE == PassMode::MetropolisFull;
    R sh = dot3(s, h);
    int32_t j0 = 0;
    uint32_t b0 = 0;
    if (first) {
#pragma unroll
      for (int g = 0; g < kHits; ++g)
        if (kFull || g < hc.k_hits)
          decide_hit(s, sh, dE_sum, first->trial[g], dot3(first->trial[g], h), first->u[g],
                     hc.beta);
      j0 = kHits;
      b0 = 3;
    }
    for (; j0 < hc.k_hits; j0 += kHits, b0 += 3) {
      const int32_t nh = hc.k_hits - j0;  // hits left (the group takes min(kHits, nh))
      uint32_t w[3 * kHits];
      hit_words<kFull>(w, site, b0, nh, hc);
      Vec3<R> trial[kHits];
      R th[kHits], u[kHits];
      auto draw = [&](int g) {
        trial[g] = sphere_point_words<R>(w[3 * g], w[3 * g + 1]);
        u[g] = unit_uniform<R>(w[3 * g + 2]);
        th[g] = dot3(trial[g], h);
      };
      auto decide = [&](int g) { decide_hit(s, sh, dE_sum, trial[g], th[g], u[g], hc.beta); };
      if constexpr (G == 1) {
#pragma unroll
        for (int g = 0; g < kHits; ++g) {
          if (kFull || g < nh) {
            draw(g);
            decide(g);
          }
        }
      } else {
#pragma unroll
        for (int g = 0; g < kHits; ++g)
          if (kFull || g < nh) draw(g);
#pragma unroll
        for (int g = 0; g < kHits; ++g)
          if (kFull || g < nh) decide(g);
      }
    }
  }
  return dE_sum;
}

// The value at offset `off` of a plane (see SiteOffsets) whose base is wave-uniform; with
// NT a load of data the pass only reads (couplings, the other colour's spins) carries the
// non-temporal cache hint.
template <typename R>
__device__ __forceinline__ R* plane_at(R* base, uint32_t off) {
  if constexpr (sizeof(R) == 4)
    return (R*)((char*)base + off);
  else
    return base + off;
}
template <bool NT, typename R>
__device__ __forceinline__ R plane_ld(R* base, uint32_t off) {
  if constexpr (NT)
    return __builtin_nontemporal_load(plane_at(base, off));
  else
    return *plane_at(base, off);
}

// Updates the colour-c site at o in place; returns the sum of the accepted energy changes.
template <typename R, PassMode MODE, bool NT = false>
__device__ __forceinline__ double update_site(const Planes<R>& S, const Planes<R>& J, int32_t c,
                                              const SiteOffsets& o, const HitCtx<R>& hc) {
  const int oc = 3 * c, nc = 3 * (1 - c);
  // couplings of the six bonds: +x,+y,+z stored at the site, -x,-y,-z at the neighbour
  const R j_px = plane_ld<NT>(J.p[oc + 0], o.own), j_mx = plane_ld<NT>(J.p[nc + 0], o.mx);
  const R j_py = plane_ld<NT>(J.p[oc + 1], o.own), j_my = plane_ld<NT>(J.p[nc + 1], o.my);
  const R j_pz = plane_ld<NT>(J.p[oc + 2], o.own), j_mz = plane_ld<NT>(J.p[nc + 2], o.mz);
  R hcomp[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    R* sn = S.p[nc + k];
    R acc = j_px * plane_ld<NT>(sn, o.px);
    acc = dev_fma(j_mx, plane_ld<NT>(sn, o.mx), acc);
    acc = dev_fma(j_py, plane_ld<NT>(sn, o.py), acc);
    acc = dev_fma(j_my, plane_ld<NT>(sn, o.my), acc);
    acc = dev_fma(j_pz, plane_ld<NT>(sn, o.pz), acc);
    acc = dev_fma(j_mz, plane_ld<NT>(sn, o.mz), acc);
    hcomp[k] = acc;
  }
  const Vec3<R> h{hcomp[0], hcomp[1], hcomp[2]};
  Vec3<R> s{plane_ld<false>(S.p[oc + 0], o.own), plane_ld<false>(S.p[oc + 1], o.own),
            plane_ld<false>(S.p[oc + 2], o.own)};
  const double dE_sum = apply_update<R, MODE>(s, h, o.site, hc);
  *plane_at(S.p[oc + 0], o.own) = s.x;
  *plane_at(S.p[oc + 1], o.own) = s.y;
  *plane_at(S.p[oc + 2], o.own) = s.z;
  return dE_sum;
}

// s / |s| (length from a fused dot product, correctly rounded root and divisions).
template <typename R>
__device__ __forceinline__ Vec3<R> unit_vector(const Vec3<R>& s) {
  const R n = dev_sqrt(dot3(s, s));
  return Vec3<R>{dev_div(s.x, n), dev_div(s.y, n), dev_div(s.z, n)};
}

// sigma <- sigma / |sigma| for the spin at index e of colour c (N/2 = Nh per colour).
template <typename R>
__device__ __forceinline__ void renormalise_spin(const Planes<R>& S, int c, int64_t e) {
  const Vec3<R> s{S.p[3 * c][e], S.p[3 * c + 1][e], S.p[3 * c + 2][e]};
  const R n = dev_sqrt(dot3(s, s));
  S.p[3 * c][e] = dev_div(s.x, n);
  S.p[3 * c + 1][e] = dev_div(s.y, n);
  S.p[3 * c + 2][e] = dev_div(s.z, n);
}

// sigma_i . h_i of the colour-0 site at o in binary64.  Every bond has exactly one
// colour-0 end (L even), so H = -(sum of this over the colour-0 sites).
template <typename R>
__device__ __forceinline__ double colour0_bond_sum(const Planes<R>& S, const Planes<R>& J,
                                                   const SiteOffsets& o) {
  const double j[6] = {(double)plane_ld<false>(J.p[0], o.own), (double)plane_ld<false>(J.p[3], o.mx),
                       (double)plane_ld<false>(J.p[1], o.own), (double)plane_ld<false>(J.p[4], o.my),
                       (double)plane_ld<false>(J.p[2], o.own), (double)plane_ld<false>(J.p[5], o.mz)};
  const uint32_t nb[6] = {o.px, o.mx, o.py, o.my, o.pz, o.mz};
  double e_site = 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double hk = 0.0;
#pragma unroll
    for (int d = 0; d < 6; ++d) hk = fma(j[d], (double)plane_ld<false>(S.p[3 + k], nb[d]), hk);
    e_site = fma((double)plane_ld<false>(S.p[k], o.own), hk, e_site);
  }
  return e_site;
}

}  // namespace hsg
