// Sweeps of small lattices (§4's checkerboard schedule) with several colour passes per
// launch.  A colour pass of a lattice of up to ~10^5 sites takes 2-4 us of which the
// launch, the drain of the one before and the latency of one chain of loads are nearly
// all; on some hosts the launch calls themselves (4 us each) are slower than the GPU.
//
// tiny_kernel (tiny_supported): the whole lattice in one workgroup, its spins in LDS, each
// thread's couplings and spins in registers, and all sweeps of a call in one launch.
//
// brick_kernel (larger lattices): a phase -- its colour-0 and colour-1 passes -- per launch.
// A workgroup owns whole rows in x, a few in y and z: it loads their spins and couplings and
// those of the two rows around them into LDS at once, updates colour 0 on its rows and the
// ring around them, then colour 1 on its rows, which finds every neighbour it reads already
// updated.  Ring rows belong to other workgroups too, which compute them from the same
// inputs and the same Philox draws, hence to the same bits; workgroups never communicate,
// and read one spin array and write another.  The recomputed ring costs arithmetic that the
// idle compute units of a small lattice have to spare.  (Bricks cut in x as well touched
// five times the cache lines per load instruction, and spent half of the launch on that.)
//
// Site arithmetic (field of eq. 2 in the fixed order, then apply_update) and therefore the
// spins are those of the single passes, bit for bit; only the order of the binary64 sum of
// energy changes differs.
//
// This file defines the launchers: one source includes it, kernels_march.hip.
#pragma once

#include "hsg_device.h"
#include "hsg_internal.h"
#include "hsg_site.h"

namespace hsg {
namespace {

__device__ __forceinline__ int32_t wrap_to(int32_t v, int32_t n) {
  return v < 0 ? v + n : (v >= n ? v - n : v);
}

// Local field of eq. 2 from six neighbour spins in LDS (component stride cs), the fixed
// order of the single-pass kernel.
template <typename R>
struct SiteBonds {
  R px, mx, py, my, pz, mz;
};
struct Neighbours {
  int32_t px, mx, py, my, pz, mz;
};
template <typename R>
__device__ __forceinline__ Vec3<R> lds_field(const R* spins, int32_t cs, const Neighbours& n,
                                             const SiteBonds<R>& j) {
  R h[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const R* s = spins + k * cs;
    R acc = j.px * s[n.px];
    acc = dev_fma(j.mx, s[n.mx], acc);
    acc = dev_fma(j.py, s[n.py], acc);
    acc = dev_fma(j.my, s[n.my], acc);
    acc = dev_fma(j.pz, s[n.pz], acc);
    acc = dev_fma(j.mz, s[n.mz], acc);
    h[k] = acc;
  }
  return Vec3<R>{h[0], h[1], h[2]};
}

// ---------------------------------------------------------------------------- bricks

// Quotient n / d for n < 4096, d < 64 (a region's sites and extents), the multiplier from
// the hardware reciprocal: m = floor(2^20 / d) + 1 is exact for every d, since 2^20 / d is
// 1/d or more from an integer unless d is a power of two, and the reciprocal an ulp from
// it; and n m / 2^20 exceeds n / d by less than 1/d.  (An integer division of uniform
// values is a few hundred cycles, and each stage needs two.)
struct RegionDiv {
  uint32_t m;
  __device__ __forceinline__ explicit RegionDiv(int32_t d)
      : m((uint32_t)__builtin_amdgcn_readfirstlane(
            (int32_t)((uint32_t)(1048576.0f * __builtin_amdgcn_rcpf((float)d)) + 1u))) {}
  __device__ __forceinline__ int32_t div(int32_t n) const {
    return (int32_t)(((uint32_t)n * m) >> 20);
  }
};

template <typename R, PassMode MODE, int T, int LDS_BYTES>
__global__ __launch_bounds__(T) void brick_kernel(BrickArgs<R> a) {
  constexpr int kCap = LDS_BYTES / (6 * (int)sizeof(R));  // sites, both colours
  __shared__ R spins[3 * kCap];  // [component][colour][site of the region]
  __shared__ R bonds[3 * kCap];  // [direction][colour][site]
  __shared__ double s_red[16];
  const int32_t tid = (int32_t)threadIdx.x;
  const int32_t L = a.L, Lh = a.L / 2;
  const uint32_t Nh = (uint32_t)(Lh * L * L);

  // this brick: rows [y0, y0 + ny) of the planes [z0, z0 + nz)
  const uint32_t tile = (uint32_t)xcd_tile((int32_t)blockIdx.x, (int32_t)gridDim.x);
  const SmallDiv dy{(uint32_t)a.n[0], a.inv[0]}, dz{(uint32_t)a.n[1], a.inv[1]};
  const uint32_t bz = dy.div(tile), by = tile - bz * dy.d;
  const int32_t y0 = (int32_t)dy.div(by * (uint32_t)L), z0 = (int32_t)dz.div(bz * (uint32_t)L);
  const int32_t ny = (int32_t)dy.div((by + 1) * (uint32_t)L) - y0,
                nz = (int32_t)dz.div((bz + 1) * (uint32_t)L) - z0;
  // region: two rows and planes more on each side
  const int32_t RY = ny + 4, plane = RY * Lh, NC = plane * (nz + 4);
  const RegionDiv dlh(Lh);
  const HitCtx<R> hc{a.beta, a.sweep, a.phase, a.k_hits, a.seed_lo, a.seed_hi};

  // Sites: colour 0 on the rows and a ring of one (c = 0), then colour 1 on the rows, all
  // numbered in one range, so that where there are threads enough each has one site of the
  // launch and its draws, which need no spin, are made while the loads are on their way.
  struct Place {
    int32_t c, rz, ry, j;  // colour; plane, row and column of the region
    int32_t p;             // x parity of the row's sites of the colour
    uint32_t g;            // index in the colour
    bool own;              // not of the ring
  };
  const int32_t n0 = Lh * (ny + 2) * (nz + 2), n01 = n0 + Lh * ny * nz;
  const RegionDiv dy0(ny + 2), dy1(ny);
  auto place = [&](int32_t i) {
    Place q;
    q.c = i >= n0 ? 1 : 0;
    i -= q.c ? n0 : 0;
    const int32_t row = dlh.div(i), pz = q.c ? dy1.div(row) : dy0.div(row);
    q.j = i - row * Lh;
    q.rz = pz + 1 + q.c;
    q.ry = row - pz * (ny + (q.c ? 0 : 2)) + 1 + q.c;
    q.p = (q.c + y0 + z0 + q.ry + q.rz) & 1;
    const int32_t y = wrap_to(y0 - 2 + q.ry, L), z = wrap_to(z0 - 2 + q.rz, L);
    q.g = (uint32_t)(q.j + Lh * (y + L * z));
    q.own = (uint32_t)(q.rz - 2) < (uint32_t)nz && (uint32_t)(q.ry - 2) < (uint32_t)ny;
    return q;
  };
  Draws<R, MODE> first;
  Place mine{};

  {  // the region's spins and couplings
    const RegionDiv dry(RY);
    constexpr int U = sizeof(R) == 4 ? 4 : 2;  // sites in flight per thread
    for (int32_t e0 = tid; e0 < 2 * NC; e0 += U * T) {
      R v[U][6];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int32_t e = e0 + u * T;
        if (e < 2 * NC) {
          const int32_t c = e >= NC ? 1 : 0, i = e - c * NC;
          const int32_t row = dlh.div(i), rz = dry.div(row);
          const int32_t y = wrap_to(y0 - 2 + row - rz * RY, L), z = wrap_to(z0 - 2 + rz, L);
          const uint32_t g = (c ? 3u * Nh : 0u) + (uint32_t)(i - row * Lh + Lh * (y + L * z));
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            v[u][k] = a.in[g + (uint32_t)k * Nh];
            v[u][3 + k] = a.J[g + (uint32_t)k * Nh];
          }
        }
      }
      if (e0 == tid && tid < n01) {
        mine = place(tid);
        first = first_draws<R, MODE>(2u * mine.g + (uint32_t)mine.p, hc);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int32_t e = e0 + u * T;
        if (e < 2 * NC) {
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            spins[k * kCap + e] = v[u][k];
            bonds[k * kCap + e] = v[u][3 + k];
          }
        }
      }
    }
  }

  double dE = 0.0;
  auto update = [&](const Place& q, const Draws<R, MODE>* d) {
    const int32_t idx = (q.rz * RY + q.ry) * Lh + q.j;
    const int32_t m = q.c * NC + idx, o = NC - q.c * NC + idx;
    const int32_t up = q.p ? (q.j == Lh - 1 ? o + 1 - Lh : o + 1) : o;
    const int32_t down = q.p ? o : (q.j == 0 ? o - 1 + Lh : o - 1);
    const Neighbours n{up, down, o + Lh, o - Lh, o + plane, o - plane};
    const SiteBonds<R> jb{bonds[m],            bonds[n.mx],
                          bonds[kCap + m],     bonds[kCap + n.my],
                          bonds[2 * kCap + m], bonds[2 * kCap + n.mz]};
    const Vec3<R> h = lds_field<R>(spins, kCap, n, jb);
    Vec3<R> sp{spins[m], spins[kCap + m], spins[2 * kCap + m]};
    const double e = apply_update<R, MODE, kHits>(sp, h, 2u * q.g + (uint32_t)q.p, hc, d);
    if (MODE != PassMode::OverRelax) dE += q.own ? e : 0.0;
    if (q.c == 0) {  // for colour 1, before any renormalisation
      spins[m] = sp.x;
      spins[kCap + m] = sp.y;
      spins[2 * kCap + m] = sp.z;
    }
    if (q.own) {
      if (a.renorm) sp = unit_vector(sp);
      R* out = a.out + (q.c ? 3u * Nh : 0u) + q.g;
      out[0] = sp.x;
      out[Nh] = sp.y;
      out[2 * Nh] = sp.z;
    }
  };
  __syncthreads();
  if (tid < n0) update(mine, &first);
  for (int32_t i = tid + T; i < n0; i += T) update(place(i), nullptr);
  __syncthreads();
  if (tid >= n0 && tid < n01) update(mine, &first);
  for (int32_t i = tid + T; i < n01; i += T)
    if (i >= n0) update(place(i), nullptr);
  if constexpr (MODE != PassMode::OverRelax) {
    const double total = block_sum(dE, s_red);
    if (tid == 0) atomicAdd(&a.partials[blockIdx.x], total);  // its only writer: no round trip
  }
}

// ---------------------------------------------------------------------- one workgroup

// The lattice's sweeps in one workgroup, T threads on the sites of colour 0 and T on those of
// colour 1.  A thread owns sites t, t + T, ... (ROUNDS of them) for the whole launch: their
// couplings, their neighbours' places and their spins stay in registers; the other colour is
// read from LDS.  A pass is a chain of dependent steps on one wave per SIMD or two, half of
// it the draws, which need no spin: the colour that waits makes those of its next Monte
// Carlo update.  us a sweep of k = 4 and one over-relaxation phase, each thread on both
// colours / so: L = 8 3.0 / 2.1, 10 3.9 / 3.2, 12 6.5 / 5.8 (binary64 L = 8 4.0 / 3.5); k = 1
// 2.3 / 1.7, 2.8 / 2.2, 4.5 / 4.2.
template <typename R, PassMode MC, int T, int ROUNDS>
__global__ __launch_bounds__(2 * T) void tiny_kernel(TinyArgs<R> a) {
  constexpr int kCap = T * ROUNDS;
  constexpr bool kMetropolis = MC == PassMode::Metropolis || MC == PassMode::MetropolisFull;
  constexpr bool kFull = MC == PassMode::MetropolisFull;
  __shared__ R lds[2][3][kCap];
  __shared__ double s_red[16];
  const uint32_t L = (uint32_t)a.L, Lh = L / 2, Nh = Lh * L * L;
  const int32_t c = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x) >= T ? 1 : 0;
  const uint32_t tid = threadIdx.x - (uint32_t)(c * T);
  SiteBonds<R> jb[ROUNDS];
  Vec3<R> sp[ROUNDS];
  uint32_t site[ROUNDS], at[ROUNDS][6];  // neighbours' places in LDS: px, mx, py, my, pz, mz
  const SmallDiv by_lh(Lh), by_l(L);
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const uint32_t i = tid + (uint32_t)(r * T);
    site[r] = 0;
    if (i >= Nh) continue;
    const uint32_t row = by_lh.div(i), z = by_l.div(row);
    const SiteOffsets q = site_offsets<R>(L, Lh, (uint32_t)c, i, i - row * Lh, row - z * L, z);
    const R* Jo = a.J + 3 * c * Nh;
    const R* Jn = a.J + 3 * (1 - c) * Nh;
    jb[r] = SiteBonds<R>{*plane_at(Jo, q.own),          *plane_at(Jn, q.mx),
                         *plane_at(Jo + Nh, q.own),     *plane_at(Jn + Nh, q.my),
                         *plane_at(Jo + 2 * Nh, q.own), *plane_at(Jn + 2 * Nh, q.mz)};
    const R* S = a.spins + 3 * c * Nh;
    sp[r] = Vec3<R>{S[i], S[Nh + i], S[2 * Nh + i]};
    site[r] = q.site;
    const uint32_t nb[6] = {q.px, q.mx, q.py, q.my, q.pz, q.mz};
#pragma unroll
    for (int k = 0; k < 6; ++k)
      at[r][k] = nb[k] * (uint32_t)(sizeof(R) / OffsetUnit<R>::value) +
                 (uint32_t)((1 - c) * 3 * kCap * (int)sizeof(R));
  }
  auto put = [&](int r) {
    R* own = &lds[c][0][tid + (uint32_t)(r * T)];
    own[0] = sp[r].x;
    own[kCap] = sp[r].y;
    own[2 * kCap] = sp[r].z;
  };
  auto each = [&](auto f) {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
      if (tid + (uint32_t)(r * T) < Nh) f(r);
  };
  auto field = [&](int r) {
    const char* base = (const char*)&lds[0][0][0];
    R h[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      auto s = [&](int d) { return *(const R*)(base + at[r][d] + k * kCap * (int)sizeof(R)); };
      R acc = jb[r].px * s(0);
      acc = dev_fma(jb[r].mx, s(1), acc);
      acc = dev_fma(jb[r].py, s(2), acc);
      acc = dev_fma(jb[r].my, s(3), acc);
      acc = dev_fma(jb[r].pz, s(4), acc);
      acc = dev_fma(jb[r].mz, s(5), acc);
      h[k] = acc;
    }
    return Vec3<R>{h[0], h[1], h[2]};
  };
  // The draws of a sweep's first group of hits at the thread's first site, in two halves
  // (words; trial points) that each fit behind a pass of the other colour.
  uint32_t w[3 * kHits];
  Draws<R, MC> d;
  const bool mc = MC != PassMode::OverRelax && a.k_hits > 0;
  auto ctx = [&](uint32_t sweep) {
    return HitCtx<R>{a.beta, sweep, 0u, a.k_hits, a.seed_lo, a.seed_hi};
  };
  auto words = [&](uint32_t sweep) {
    const HitCtx<R> hc = ctx(sweep);
    if constexpr (kMetropolis)
      hit_words<kFull>(w, site[0], 0u, a.k_hits, hc);
    else
      d = first_draws<R, MC>(site[0], hc);
  };
  auto points = [&] {
    if constexpr (kMetropolis) {
#pragma unroll
      for (int g = 0; g < kHits; ++g)
        if (kFull || g < a.k_hits) {
          d.trial[g] = sphere_point_words<R>(w[3 * g], w[3 * g + 1]);
          d.u[g] = unit_uniform<R>(w[3 * g + 2]);
        }
    }
  };
  each(put);
  if (mc) {
    words(a.sweep);
    if (c == 0) points();
  }
  __syncthreads();
  const double E0 = threadIdx.x == 0 ? *a.E : 0.0;
  double dE = 0.0;
  auto monte_carlo = [&](uint32_t sweep) {
    each([&](int r) {
      dE += apply_update<R, MC, kHits>(sp[r], field(r), site[r], ctx(sweep), r == 0 ? &d : nullptr);
      put(r);
    });
  };
  auto over_relax = [&] {
    each([&](int r) {
      sp[r] = reflect(sp[r], field(r));
      put(r);
    });
  };
  int32_t until_renorm = a.until_renorm;
  for (int32_t n = 0; n < a.n_sweeps; ++n) {
    const uint32_t sweep = a.sweep + (uint32_t)n;
    const bool more = mc && n + 1 < a.n_sweeps;
    if (mc) {
      if (c == 0) {
        monte_carlo(sweep);
      } else {
        if (a.n_or == 0 && n > 0) words(sweep);
        points();
      }
      __syncthreads();
      if (c == 1) {
        monte_carlo(sweep);
      } else if (more) {
        words(sweep + 1u);
        if (a.n_or == 0) points();
      }
      __syncthreads();
    }
    for (int32_t phase = 1; phase <= a.n_or; ++phase) {
      if (c == 0)
        over_relax();
      else if (phase == 1 && more)
        words(sweep + 1u);
      __syncthreads();
      if (c == 1)
        over_relax();
      else if (phase == 1 && more)
        points();
      __syncthreads();
    }
    if (a.renorm_every > 0 && --until_renorm == 0) {
      until_renorm = a.renorm_every;
      each([&](int r) {
        sp[r] = unit_vector(sp[r]);
        put(r);
      });
      __syncthreads();
    }
  }
  each([&](int r) {
    const uint32_t i = tid + (uint32_t)(r * T);
    R* S = a.spins + 3 * c * Nh;
    S[i] = sp[r].x;
    S[Nh + i] = sp[r].y;
    S[2 * Nh + i] = sp[r].z;
  });
  if (mc) {
    const double total = block_sum(dE, s_red);
    if (threadIdx.x == 0) *a.E = E0 + total;
  }
}

// The same with every thread on ROUNDS sites of both colours, for lattices whose 1024 threads
// would have more sites each than registers, or more waves idle than there is to do for them.
template <typename R, PassMode MC, int T, int ROUNDS>
__global__ __launch_bounds__(T) void tiny_both_kernel(TinyArgs<R> a) {
  constexpr int kCap = T * ROUNDS;
  __shared__ R lds[2][3][kCap];
  __shared__ double s_red[16];
  const uint32_t L = (uint32_t)a.L, Lh = L / 2, Nh = Lh * L * L;
  SiteOffsets o[2][ROUNDS];
  SiteBonds<R> jb[2][ROUNDS];
  Vec3<R> sp[2][ROUNDS];
  const SmallDiv by_lh(Lh), by_l(L);
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const uint32_t i = threadIdx.x + (uint32_t)(r * T);
      if (i >= Nh) continue;
      const uint32_t row = by_lh.div(i), z = by_l.div(row);
      SiteOffsets q = site_offsets<R>(L, Lh, (uint32_t)c, i, i - row * Lh, row - z * L, z);
      const R* Jo = a.J + 3 * c * Nh;
      const R* Jn = a.J + 3 * (1 - c) * Nh;
      jb[c][r] = SiteBonds<R>{*plane_at(Jo, q.own),          *plane_at(Jn, q.mx),
                              *plane_at(Jo + Nh, q.own),     *plane_at(Jn + Nh, q.my),
                              *plane_at(Jo + 2 * Nh, q.own), *plane_at(Jn + 2 * Nh, q.mz)};
      const R* S = a.spins + 3 * c * Nh;
      sp[c][r] = Vec3<R>{S[i], S[Nh + i], S[2 * Nh + i]};
      lds[c][0][i] = sp[c][r].x;
      lds[c][1][i] = sp[c][r].y;
      lds[c][2][i] = sp[c][r].z;
      o[c][r] = q;
    }
  __syncthreads();
  const double E0 = threadIdx.x == 0 ? *a.E : 0.0;
  double dE = 0.0;
  int32_t until_renorm = a.until_renorm;
  for (int32_t n = 0; n < a.n_sweeps; ++n) {
    const uint32_t sweep = a.sweep + (uint32_t)n;
    for (int32_t phase = a.k_hits > 0 ? 0 : 1; phase <= a.n_or; ++phase) {
      const HitCtx<R> hc{a.beta, sweep, (uint32_t)phase, a.k_hits, a.seed_lo, a.seed_hi};
#pragma unroll
      for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
          const uint32_t i = threadIdx.x + (uint32_t)(r * T);
          if (i >= Nh) continue;
          const SiteOffsets& q = o[c][r];
          R h[3];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const R* s = lds[1 - c][k];
            R acc = jb[c][r].px * *plane_at(s, q.px);
            acc = dev_fma(jb[c][r].mx, *plane_at(s, q.mx), acc);
            acc = dev_fma(jb[c][r].py, *plane_at(s, q.py), acc);
            acc = dev_fma(jb[c][r].my, *plane_at(s, q.my), acc);
            acc = dev_fma(jb[c][r].pz, *plane_at(s, q.pz), acc);
            acc = dev_fma(jb[c][r].mz, *plane_at(s, q.mz), acc);
            h[k] = acc;
          }
          const Vec3<R> hv{h[0], h[1], h[2]};
          if (phase == 0)
            dE += apply_update<R, MC, kHits>(sp[c][r], hv, q.site, hc);
          else
            apply_update<R, PassMode::OverRelax>(sp[c][r], hv, q.site, hc);
          lds[c][0][i] = sp[c][r].x;
          lds[c][1][i] = sp[c][r].y;
          lds[c][2][i] = sp[c][r].z;
        }
        __syncthreads();
      }
    }
    if (a.renorm_every > 0 && --until_renorm == 0) {
      until_renorm = a.renorm_every;
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
          const uint32_t i = threadIdx.x + (uint32_t)(r * T);
          if (i >= Nh) continue;
          sp[c][r] = unit_vector(sp[c][r]);
          lds[c][0][i] = sp[c][r].x;
          lds[c][1][i] = sp[c][r].y;
          lds[c][2][i] = sp[c][r].z;
        }
      __syncthreads();
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const uint32_t i = threadIdx.x + (uint32_t)(r * T);
      if (i >= Nh) continue;
      R* S = a.spins + 3 * c * Nh;
      S[i] = sp[c][r].x;
      S[Nh + i] = sp[c][r].y;
      S[2 * Nh + i] = sp[c][r].z;
    }
  if (a.k_hits > 0) {
    const double total = block_sum(dE, s_red);
    if (threadIdx.x == 0) *a.E = E0 + total;
  }
}

template <typename R, PassMode MC>
hipError_t launch_tiny_as(const TinyArgs<R>& a, hipStream_t st) {
  const int32_t Nh = a.L * a.L * a.L / 2;
  const dim3 one(1);
  if (Nh <= 256)
    hipLaunchKernelGGL((tiny_kernel<R, MC, 256, 1>), one, dim3(512), 0, st, a);
  // us a sweep of k = 4 (1) by colour / by both: binary32 L = 14, three rounds of sites
  // against two, 8.5 / 8.4 (6.7 / 5.0); binary64 L = 10, two against one, 7.3 / 6.5 (4.6 / 3.9)
  else if constexpr (sizeof(R) == 4) {
    if (Nh <= 512)
      hipLaunchKernelGGL((tiny_kernel<R, MC, 512, 1>), one, dim3(1024), 0, st, a);
    else if (Nh <= 1024)
      hipLaunchKernelGGL((tiny_kernel<R, MC, 512, 2>), one, dim3(1024), 0, st, a);
    else if (Nh <= 1408)
      hipLaunchKernelGGL((tiny_both_kernel<R, MC, 704, 2>), one, dim3(704), 0, st, a);
    else
      return hipErrorInvalidValue;
  } else if (Nh <= 512) {
    hipLaunchKernelGGL((tiny_both_kernel<R, MC, 512, 1>), one, dim3(512), 0, st, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

namespace {

// LDS of a workgroup: four, two or one to a compute unit.
constexpr int kLds[3] = {38400, 79872, 159744};

uint32_t inv_of(int32_t d) { return d > 1 ? 0xFFFFFFFFu / (uint32_t)d + 1u : 0u; }

template <typename R, PassMode MODE>
void launch_brick_as(const BrickArgs<R>& a, const BrickPlan& b, hipStream_t st) {
  constexpr int T0 = 512, T1 = sizeof(R) == 4 ? 1024 : 512;  // threads by LDS size
  const dim3 grid((unsigned)(b.n[0] * b.n[1]));
  if (b.lds == 0)
    hipLaunchKernelGGL((brick_kernel<R, MODE, T0, kLds[0]>), grid, dim3(T0), 0, st, a);
  else if (b.lds == 1)
    hipLaunchKernelGGL((brick_kernel<R, MODE, T1, kLds[1]>), grid, dim3(T1), 0, st, a);
  else
    hipLaunchKernelGGL((brick_kernel<R, MODE, T1, kLds[2]>), grid, dim3(T1), 0, st, a);
}

}  // namespace

// In binary64 a lattice of L = 12 (two rounds of sites a thread) is faster in bricks: 12
// against 10 us a sweep of k = 4 and one over-relaxation phase.
bool tiny_supported(int32_t L, int32_t elem) { return L <= (elem == 4 ? 14 : 10); }

// Rows of a brick, timed against 2 x 2 .. 4 x 8 rows of 256 - 1024 threads: the smallest
// bricks (most workgroups, shortest chains) as long as they are not more than the compute
// units.  A sweep of k = 4 and one over-relaxation phase, pass by pass and so (us, binary32):
// L = 16 13.2 / 8.3, 24 13.8 / 8.6, 32 13.8 / 9.1, 44 15.8 / 12.2, 64 17.5 / 16.5 (over-
// relaxation alone, two phases: 11.0 / 7.1 at L = 24, 15.5 / 12.7 at 64).  Larger lattices
// would need more bricks than compute units at 159 KB of LDS each: pass by pass is faster
// (L = 64: 512 workgroups 22 us).  Binary64 (twice the LDS, half the threads): L = 16
// 16.2 / 10.3, 32 18.1 / 12.3, 40 18.8 / 15.3; L = 48 20.0 / 22.4.
bool brick_plan(int32_t L, int32_t elem, BrickPlan* plan) {
  if (tiny_supported(L, elem) || L > (elem == 4 ? kBrickMaxL : 40)) return false;
  int32_t wy, wz;  // rows in y and z
  if (L <= 32)
    wy = wz = 2;
  else if (elem == 8)
    wy = 2, wz = 4;
  else
    wy = wz = L <= 46 ? 3 : 4;
  BrickPlan b{};
  b.n[0] = (L + wy - 1) / wy;
  b.n[1] = (L + wz - 1) / wz;
  const int32_t bytes = (L / 2) * (wy + 4) * (wz + 4) * 2 * 6 * elem;
  b.lds = bytes <= kLds[0] ? 0 : bytes <= kLds[1] ? 1 : 2;
  *plan = b;
  return true;
}

template <typename R>
hipError_t launch_brick(const BrickArgs<R>& a0, PassMode mode, hipStream_t st) {
  BrickArgs<R> a = a0;
  BrickPlan b;
  if (!brick_plan(a.L, (int32_t)sizeof(R), &b)) return hipErrorInvalidValue;
  for (int k = 0; k < 2; ++k) {
    a.n[k] = b.n[k];
    a.inv[k] = inv_of(b.n[k]);
  }
  if (mode == PassMode::Metropolis) mode = metropolis_mode(a.k_hits);
  if (mode == PassMode::OverRelax) launch_brick_as<R, PassMode::OverRelax>(a, b, st);
  else if (mode == PassMode::HeatBath) launch_brick_as<R, PassMode::HeatBath>(a, b, st);
  else if (mode == PassMode::MetropolisFull) launch_brick_as<R, PassMode::MetropolisFull>(a, b, st);
  else launch_brick_as<R, PassMode::Metropolis>(a, b, st);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_tiny(const TinyArgs<R>& a, PassMode mc, hipStream_t st) {
  if (a.k_hits == 0) return launch_tiny_as<R, PassMode::OverRelax>(a, st);
  if (mc == PassMode::HeatBath) return launch_tiny_as<R, PassMode::HeatBath>(a, st);
  if (metropolis_mode(a.k_hits) == PassMode::MetropolisFull)
    return launch_tiny_as<R, PassMode::MetropolisFull>(a, st);
  return launch_tiny_as<R, PassMode::Metropolis>(a, st);
}

template hipError_t launch_brick<float>(const BrickArgs<float>&, PassMode, hipStream_t);
template hipError_t launch_brick<double>(const BrickArgs<double>&, PassMode, hipStream_t);
template hipError_t launch_tiny<float>(const TinyArgs<float>&, PassMode, hipStream_t);
template hipError_t launch_tiny<double>(const TinyArgs<double>&, PassMode, hipStream_t);

}  // namespace hsg
