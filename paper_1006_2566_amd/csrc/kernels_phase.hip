// One over-relaxation phase of the checkerboard schedule (§4) -- the colour-0 pass and then
// the colour-1 pass -- in one launch, reading the spins once and writing them once: 36 bytes
// a site in binary32 where two passes move 60.  With the colour-0 pass of the next sweep's
// Monte Carlo phase behind it in the same launch, 36 bytes in place of 90.
//
// A workgroup owns a tile of rows in (x, y) and marches through a run of planes in z.  The
// tile is ny whole rows, which need no halo in x and take any L, or ny parts of rows.  A
// thread keeps its column and rows, so that its places in LDS and in a plane are fixed for
// the launch.  With q the plane of a step and H = 1 with a Monte Carlo pass, else 0:
//
//   A  colour 0 of plane q on the tile and a ring of 1 + H: its own spins and couplings in
//      registers, colour 1 of planes q - 1 .. q + 1 in LDS; the result goes to LDS (and, the
//      tile's, to the output when no Monte Carlo pass follows)
//   B  colour 1 of plane q - 1 on the tile and a ring of H, from colour 0 of planes q - 2 .. q
//      as A left them; the tile's goes to the output, all of it to LDS if C follows
//   C  the Monte Carlo update of colour 0 of plane q - 3 on the tile only, from colour 1 of
//      planes q - 4 .. q - 2 as B left them; each site by the thread that ran A for it, which
//      keeps its six couplings in registers for three steps
//
// The ring and the planes next to the run belong to other workgroups, which compute them
// too, from the same inputs, hence to the same bits; workgroups never communicate, read one
// spin array and write another.  Four planes of each array in LDS, B's and C's own spins
// read before the barrier, leave one barrier per step, between A and the two others: A of
// the next step writes over colour 0 of plane q - 3 and colour 1 of plane q - 1, which
// nobody reads any more, and B of the next step over what C read in the step before.
//
// The site arithmetic is the colour passes', so the spins are theirs bit for bit; only the
// order of the binary64 sum of C's energy changes differs.
//
// What a step needs is loaded two steps ahead (with C, one: a step is longer and registers
// are short), by loads without a condition at a scalar base plus a 32-bit offset.  One
// workgroup of up to 1024 threads per compute unit (123 to 163 KB of LDS); with C, two of
// 512 threads were 25 to 50% slower at L >= 256: their tiles are narrower, and what limits
// tiles of part of a row is the number of cache lines they touch.
//
// us per phase, two passes / this: binary32 L = 128 21.2 / 17.3, 160 36.3 / 28.3, 256 182 /
// 132, 512 1649 / 1068 (36 bytes a site at 4.5 TB/s, 0.89 of a copy: bound by HBM from L =
// 230 up, by the caches' far side below 204); binary64 L = 128 39.3 / 30.9, 256 403 / 291.
// With the Monte Carlo pass, its three passes one by one / this, binary32 k = 4: L = 192 97
// / 78, 256 277 / 177, 512 2490 / 1510; k = 1: 192 88 / 55, 256 274 / 146, 512 2460 / 1394.
// At L = 256 and k = 4 that issues 72M vector instructions, 48M of them C's, which take 117
// of the 177 us; only the waves of the tile's own rows, half of them there, have a C.  At
// 512 (three rounds of 11 rows) the clock falls to 1.6 GHz under the load.  Tiles of 64 x 16
// sites with loads behind conditions and three barriers a step, which this replaced, took
// 161 and 215 us at L = 256, 1327 and 1830 at 512.
#include <algorithm>
#include <type_traits>

#include "hsg_device.h"
#include "hsg_internal.h"
#include "hsg_site.h"

namespace hsg {
namespace {

template <typename R>
struct RowStep {  // what A and B of a step need, and the colour-1 plane that follows
  R s0[3];     // A's own colour-0 spin
  R ja[6];     // couplings of A's site
  R jb[6];     // ... and of B's site, one plane below
  R c1[2][3];  // colour-1 spins on their way to LDS (two sites a thread)
};

// Threads of a workgroup and sites of its planes in LDS, at most.
template <typename R, bool MC>
struct RowSize {
  static constexpr int A = sizeof(R) == 4 ? 1024 : 512;  // threads; colour 0
  static constexpr int C1 = MC ? (sizeof(R) == 4 ? 1344 : 672) : (sizeof(R) == 4 ? 1536 : 1024);
  static constexpr int B = MC ? A : 1;  // colour 1 after B
  static constexpr int D = MC ? 1 : 2;  // steps ahead of which a step's values are loaded
};

// MODE: of the Monte Carlo pass behind the phase, OverRelax for the phase alone.  WAVES: a wave
// takes a row of the tile (kByWave below).
template <typename R, PassMode MODE, bool WAVES>
__device__ __forceinline__ void row_march(const PhaseArgs<R>& a) {
  constexpr bool MC = MODE != PassMode::OverRelax;
  // hits whose trials are formed together: a group's registers cost more than they gain
  // where it may be incomplete (L = 256, one hit: 189 us, and 146 one by one)
  [[maybe_unused]] constexpr int kGroup = MODE == PassMode::MetropolisFull ? 4 : 1;
  constexpr int H = MC ? 1 : 0;  // rows (and columns) B goes beyond the tile
  using Size = RowSize<R, MC>;
  constexpr int N0 = Size::A, N1 = Size::C1, D = Size::D;
  __shared__ R lds1[4][3][N1];  // [plane mod 4][component][site] of colour 1, ny + 4 + 2H rows
  __shared__ R lds0[4][3][N0];  // ... of colour 0 after A, ny + 2 + 2H rows
  __shared__ R ldsB[MC ? 4 : 1][3][Size::B];  // ... of colour 1 after B, ny + 2 rows
  const int32_t tid = (int32_t)threadIdx.x, T = (int32_t)blockDim.x;
  const int32_t L = a.L, Lh = L / 2;
  const int64_t zs = (int64_t)Lh * L;  // sites of a colour in a plane
  const int64_t Nh = zs * L;
  const uint32_t tile = (uint32_t)xcd_tile((int32_t)blockIdx.x, (int32_t)gridDim.x);
  const SmallDiv dx{(uint32_t)a.n[0], a.inv[0]}, dy{(uint32_t)a.n[1], a.inv[1]},
      dz{(uint32_t)a.n[2], a.inv[2]};
  const uint32_t r0 = dx.div(tile), bx = tile - r0 * dx.d, bz = dy.div(r0), by = r0 - bz * dy.d;
  const int32_t x0 = (int32_t)dx.div(bx * (uint32_t)Lh), y0 = (int32_t)dy.div(by * (uint32_t)L),
                z0 = (int32_t)dz.div(bz * (uint32_t)L);
  const int32_t nx = (int32_t)dx.div((bx + 1) * (uint32_t)Lh) - x0,
                ny = (int32_t)dy.div((by + 1) * (uint32_t)L) - y0,
                nz = (int32_t)dz.div((bz + 1) * (uint32_t)L) - z0;
  // Columns: a tile of part of a row (several tiles in x) has a halo column of colour 0 on
  // either side and two of colour 1; whole rows have none and wrap around.
  const int32_t hx = a.n[0] > 1 ? 1 : 0;
  const int32_t w0 = nx + 2 * hx, w1 = nx + 4 * hx;
  const int32_t wb = nx + 2 * hx * H;
  [[maybe_unused]] const int32_t n1 = (ny + 4 + 2 * H) * w1;

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  auto wrap = [](int32_t v, int32_t n) { return v < 0 ? v + n : (v >= n ? v - n : v); };
  // n / d for n < 2^14: (n + 1/2) / d is 1/(2d) or more from an integer, the product's error
  // less than n / d 2^-22
  auto quot = [](int32_t n, int32_t d) {
    return (int32_t)(((float)n + 0.5f) * __builtin_amdgcn_rcpf((float)d));
  };
  // Threads and slots past the last site load the last site's: loads without a condition are
  // what lets the wait for one step's values leave the next steps' in flight (with a branch
  // around any of them the compiler has to wait for all).
  // item i of a window of n rows of w columns, h of them halo on either side: its place, or
  // the last one's for threads past the last
  struct Place {
    int32_t r, j;
    bool has;
  };
  auto item = [&](int32_t i, int32_t n, int32_t w, int32_t h) {
    Place p;
    if constexpr (!WAVES) {
      const int32_t s = min(i, n * w - 1);
      p.has = i < n * w;
      p.r = quot(s, w);
      p.j = s - p.r * w;
    } else if ((i >> 6) < n) {  // the tile's 64 columns
      p = Place{i >> 6, h + (i & 63), true};
    } else {  // 2 h halo columns (h = 1 or 2) of a row after the other
      const int32_t e = i - 64 * n, s = min(e, 2 * h * n - 1), c = s & (2 * h - 1);
      p.has = e < 2 * h * n;
      p.r = s >> h;
      p.j = c < h ? c : 64 + c;
    }
    return p;
  };
  const Place itA = item(tid, ny + 2 + 2 * H, w0, hx), itB = item(tid, ny + 2 * H, wb, hx * H);
  const bool hasA = itA.has, hasB = itB.has;
  const int32_t rA = itA.r, jA = itA.j, rB = itB.r, jB = itB.j;
  // in the planes of their results
  const int32_t oA = WAVES ? rA * w0 + jA : tid, oB = WAVES ? rB * wb + jB : tid;
  const int32_t xA = wrap(x0 - hx + jA, Lh), xB = wrap(x0 - hx * H + jB, Lh);
  const int32_t yA = wrap(y0 - 1 - H + rA, L), yB = wrap(y0 - H + rB, L);
  const bool ownA = hasA && rA > H && rA <= ny + H && jA >= hx && jA < hx + nx;
  const bool ownB = hasB && rB >= H && rB < ny + H && jB >= hx * H && jB < hx * H + nx;
  // The neighbour in +x is a column on when the site's x parity p is 1, the one in -x a column
  // back when it is 0; p alternates from plane to plane.  A of plane q has p = (yA + q) & 1, B
  // of plane q - 1 p = (yB + q) & 1.
  const int32_t q0 = z0 - 1 - H;  // A's plane at step 0
  const int32_t pA = (yA + q0) & 1, pB = (yB + q0) & 1;  // at step 0
  // places in LDS of the other colour's site in the same column and row, and in its -+x columns
  const int32_t iA = (rA + 1) * w1 + jA + hx, iB = (rB + 1) * w0 + jB + (MC ? 0 : hx);
  const int32_t mA = hx || xA > 0 ? -1 : Lh - 1, lA = hx || xA < Lh - 1 ? 1 : 1 - Lh;
  const int32_t mB = hx || xB > 0 ? -1 : Lh - 1, lB = hx || xB < Lh - 1 ? 1 : 1 - Lh;
  const int32_t iA_px[2] = {iA + (pA ? lA : 0), iA + (pA ? 0 : lA)},
                iA_mx[2] = {iA + (pA ? 0 : mA), iA + (pA ? mA : 0)};
  const int32_t iB_px[2] = {iB + (pB ? lB : 0), iB + (pB ? 0 : lB)},
                iB_mx[2] = {iB + (pB ? 0 : mB), iB + (pB ? mB : 0)};
  const int32_t iB1 = (rB + 2) * w1 + jB + (MC ? hx : 2 * hx);  // B's own site
  // places in a plane, as byte offsets from its (wave-uniform) first site
  constexpr uint32_t E = sizeof(R);
  const uint32_t ga = (uint32_t)(yA * Lh + xA) * E, gb = (uint32_t)(yB * Lh + xB) * E;
  const uint32_t gam = (uint32_t)(wrap(yA - 1, L) * Lh + xA) * E,
                 gbm = (uint32_t)(wrap(yB - 1, L) * Lh + xB) * E;
  const uint32_t dA = (uint32_t)(xA > 0 ? -1 : Lh - 1) * E, dB = (uint32_t)(xB > 0 ? -1 : Lh - 1) * E;
  const uint32_t gax[2] = {ga + (pA ? 0u : dA), ga + (pA ? dA : 0u)};
  const uint32_t gbx[2] = {gb + (pB ? 0u : dB), gb + (pB ? dB : 0u)};
  uint32_t g1[2];  // colour-1 sites of the region: items tid and tid + T
  [[maybe_unused]] int32_t o1[2];  // with WAVES their places in LDS, or -1
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const Place it = item(tid + u * T, ny + 4 + 2 * H, w1, 2 * hx);
    g1[u] = (uint32_t)(wrap(y0 - 2 - H + it.r, L) * Lh + wrap(x0 - 2 * hx + it.j, Lh)) * E;
    if constexpr (WAVES) o1[u] = it.has ? it.r * w1 + it.j : -1;
  }

  // The twelve component arrays and six outputs have fixed (scalar) bases, and a load's
  // 32-bit offset is its place in the plane plus the plane's: one vector addition for the
  // loads that share it.  (Scalar addresses per load were 300 scalar instructions a step and
  // wave, more than a compute unit issues in the time of the vector ones.)
  const char* in[6];
  const char* Jp[6];
  char* out[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    in[k] = (const char*)(a.in + k * Nh);
    Jp[k] = (const char*)(a.J + k * Nh);
    out[k] = (char*)(a.out + k * Nh);
  }
  const uint32_t zb = (uint32_t)zs * E;  // bytes of a plane
  auto at = [](const char* base, uint32_t off) { return *(const R*)(base + off); };
  auto load_c1 = [&](R (&c1)[2][3], int32_t q) {
    const uint32_t zo = zb * (uint32_t)wrap(q, L);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t o = g1[u] + zo;
#pragma unroll
      for (int k = 0; k < 3; ++k) c1[u][k] = at(in[3 + k], o);
    }
  };
  auto put_c1 = [&](const R (&c1)[2][3], R (&d)[3][N1]) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int32_t i = WAVES ? o1[u] : tid + u * T;
      if (WAVES ? i >= 0 : i < n1) {
#pragma unroll
        for (int k = 0; k < 3; ++k) d[k][i] = c1[u][k];
      }
    }
  };
  // what A of plane q needs (q of step parity U & 1), and colour 1 of plane q + 2
  auto load_a = [&](auto U, RowStep<R>& s, int32_t q) {
    constexpr int par = decltype(U)::value & 1;
    const uint32_t z = (uint32_t)wrap(q, L), zo = zb * z;
    const uint32_t o = ga + zo, om = ga + (z == 0 ? zb * (uint32_t)(L - 1) : zo - zb);
#pragma unroll
    for (int k = 0; k < 3; ++k) s.s0[k] = at(in[k], o);
    s.ja[0] = at(Jp[0], o);
    s.ja[1] = at(Jp[3], gax[par] + zo);
    s.ja[2] = at(Jp[1], o);
    s.ja[3] = at(Jp[4], gam + zo);
    s.ja[4] = at(Jp[2], o);
    s.ja[5] = at(Jp[5], om);
    load_c1(s.c1, q + 2);
  };
  // the couplings of B's site on plane q - 1
  auto load_b = [&](auto U, RowStep<R>& s, int32_t q) {
    constexpr int par = decltype(U)::value & 1;
    const uint32_t z = (uint32_t)wrap(q - 1, L), zo = zb * z;
    const uint32_t o = gb + zo, om = gb + (z == 0 ? zb * (uint32_t)(L - 1) : zo - zb);
    s.jb[0] = at(Jp[3], o);
    s.jb[1] = at(Jp[0], gbx[par] + zo);
    s.jb[2] = at(Jp[4], o);
    s.jb[3] = at(Jp[1], gbm + zo);
    s.jb[4] = at(Jp[5], o);
    s.jb[5] = at(Jp[2], om);
  };
  auto store = [&](auto K0, uint32_t off, const Vec3<R>& s) {
    constexpr int k0 = decltype(K0)::value;
    *(R*)(out[k0] + off) = s.x;
    *(R*)(out[k0 + 1] + off) = s.y;
    *(R*)(out[k0 + 2] + off) = s.z;
  };
  // the field at place i (rows w apart) from planes cur, up and dn of the other colour
  auto field = [&](const auto& cur, const auto& up, const auto& dn, int32_t i, int32_t w,
                   int32_t ipx, int32_t imx, const R (&jj)[6]) {
    R h[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      R acc = jj[0] * cur[k][ipx];
      acc = dev_fma(jj[1], cur[k][imx], acc);
      acc = dev_fma(jj[2], cur[k][i + w], acc);
      acc = dev_fma(jj[3], cur[k][i - w], acc);
      acc = dev_fma(jj[4], up[k][i], acc);
      acc = dev_fma(jj[5], dn[k][i], acc);
      h[k] = acc;
    }
    return Vec3<R>{h[0], h[1], h[2]};
  };
  [[maybe_unused]] R jc[3][6];  // couplings of A's site on planes q - 1, q - 2 and q - 3
  [[maybe_unused]] double dE = 0.0;
  // step t = 4 m + U on plane q = q0 + t; colour-1 plane q sits in slot (t + 1) mod 4,
  // colour-0 plane q in slot t mod 4, plane q - 1 of colour 1 after B too
  auto step = [&](auto Uc, RowStep<R>& s, int32_t q) {
    constexpr int U = decltype(Uc)::value, par = U & 1;
    const bool doC = MC && ownA && q - 3 >= z0;
    Vec3<R> sc{};
    if (doC)
      sc = Vec3<R>{lds0[(U + 1) & 3][0][oA], lds0[(U + 1) & 3][1][oA], lds0[(U + 1) & 3][2][oA]};
    if (hasA) {
      const Vec3<R> h = field(lds1[(U + 1) & 3], lds1[(U + 2) & 3], lds1[U], iA, w1, iA_px[par],
                              iA_mx[par], s.ja);
      const Vec3<R> r = reflect(Vec3<R>{s.s0[0], s.s0[1], s.s0[2]}, h);
      lds0[U][0][oA] = r.x;
      lds0[U][1][oA] = r.y;
      lds0[U][2][oA] = r.z;
      if constexpr (!MC)
        if (ownA && q >= z0 && q < z0 + nz) store(I0{}, ga + zb * (uint32_t)q, r);
    }
    R jn[6];
    if constexpr (MC) {
#pragma unroll
      for (int k = 0; k < 6; ++k) jn[k] = s.ja[k];
    }
    const bool doB = hasB && q > z0 - H;
    Vec3<R> sb{};
    if (doB) sb = Vec3<R>{lds1[U][0][iB1], lds1[U][1][iB1], lds1[U][2][iB1]};
    put_c1(s.c1, lds1[(U + 3) & 3]);
    const int32_t next = min(q + D, z0 + nz + H);  // (past the last step: values nobody uses)
    load_a(std::integral_constant<int, (U + D) & 3>{}, s, next);
    __syncthreads();
    if (doB) {
      const Vec3<R> h = field(lds0[(U + 3) & 3], lds0[U], lds0[(U + 2) & 3], iB, w0, iB_px[par],
                              iB_mx[par], s.jb);
      Vec3<R> r = reflect(sb, h);
      if constexpr (MC) {
        if (a.renorm) r = unit_vector(r);
        ldsB[U][0][oB] = r.x;
        ldsB[U][1][oB] = r.y;
        ldsB[U][2][oB] = r.z;
        if (ownB && q > z0 && q <= z0 + nz) store(I3{}, gb + zb * (uint32_t)(q - 1), r);
      } else {
        store(I3{}, gb + zb * (uint32_t)(q - 1), r);
      }
    }
    load_b(std::integral_constant<int, (U + D) & 3>{}, s, next);
    if constexpr (MC) {
      if (doC) {
        const int32_t ic = oA - w0, p = (pA + par + 1) & 1;
        const Vec3<R> h = field(ldsB[(U + 2) & 3], ldsB[(U + 3) & 3], ldsB[(U + 1) & 3], ic, w0,
                                ic + (p ? lA : 0), ic + (p ? 0 : mA), jc[2]);
        if (a.renorm) sc = unit_vector(sc);
        const int32_t z = q - 3;
        const uint32_t site = (uint32_t)(2 * xA + p) + (uint32_t)L * (uint32_t)(yA + L * z);
        dE += apply_update<R, MODE, kGroup>(
            sc, h, site, HitCtx<R>{a.beta, a.mc_sweep, 0u, a.k_hits, a.seed_lo, a.seed_hi});
        store(I0{}, ga + zb * (uint32_t)z, sc);
      }
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        jc[2][k] = jc[1][k];
        jc[1][k] = jc[0][k];
        jc[0][k] = jn[k];
      }
    }
  };

  // steps q = q0 .. z0 + nz + 2H; colour 1 of planes q0 - 1 .. q0 + 1 first
  RowStep<R> s0, s1;
  {
    R c[3][2][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) load_c1(c[k], q0 - 1 + k);
    load_a(I0{}, s0, q0);
    if constexpr (D == 2) load_a(I1{}, s1, q0 + 1);
    load_b(I0{}, s0, q0);
    if constexpr (D == 2) load_b(I1{}, s1, q0 + 1);
#pragma unroll
    for (int k = 0; k < 3; ++k) put_c1(c[k], lds1[k]);
  }
  __syncthreads();
  const int32_t last = z0 + nz + 2 * H;
  for (int32_t q = q0; q <= last; q += 4) {
    step(I0{}, s0, q);
    if (q + 1 > last) break;
    step(I1{}, D == 2 ? s1 : s0, q + 1);
    if (q + 2 > last) break;
    step(I2{}, s0, q + 2);
    if (q + 3 > last) break;
    step(I3{}, D == 2 ? s1 : s0, q + 3);
  }
  if constexpr (MC) {
    __shared__ double s_red[16];
    const double total = block_sum(dE, s_red);
    if (tid == 0) atomicAdd(&a.partials[blockIdx.x], total);
  }
}

// Two over-relaxation phases in one launch: 36 bytes a site for both.  A thread has one place
// (row r, column j of a window of ny + 8 rows) for the whole march and both colours; with q
// the plane of a step:
//
//   A  phase 1, colour 0, plane q      on the tile and a ring of 3
//   B  phase 1, colour 1, plane q - 1  ... of 2
//   C  phase 2, colour 0, plane q - 3  ... of 1
//   D  phase 2, colour 1, plane q - 4  on the tile
//
// A and C, then a barrier, B and D, then a barrier.  C and B replace what they update in
// LDS, six planes of colour 0 and seven of colour 1 (160 KB); the couplings of A and B wait
// three steps in registers for C and D.  The rings cost a third to a half of the arithmetic
// and nz + 10 steps for nz planes, which stays less than the second reading and writing of
// the lattice: us for two phases, alone / together, binary32 L = 98 23.4 / 23.0, 128 34.7 /
// 28.0, 150 52 / 44, 208 149 / 130, 256 272 / 256, 320 515 / 435, 512 2130 / 1850; binary64
// 128 63 / 63, 180 213 / 180, 256 588 / 529, 384 1970 / 1669.  At L = 128 a step takes 1.8
// us: 44 waves' worth of sites, two barriers and the latency between them on 16 waves.
template <typename R>
constexpr int kPairThreads = sizeof(R) == 4 ? 1024 : 512;
template <typename R>
__global__ __launch_bounds__(kPairThreads<R>) void phase_pair_kernel(PhaseArgs<R> a) {
  constexpr int N = kPairThreads<R>, K0 = 6, K1 = 7;
  constexpr uint32_t E = sizeof(R);
  __shared__ R l0[K0 * 3 * N], l1[K1 * 3 * N];
  const int32_t tid = (int32_t)threadIdx.x;
  const int32_t L = a.L, Lh = L / 2;
  const int64_t zs = (int64_t)Lh * L, Nh = zs * L;
  const uint32_t tile = (uint32_t)xcd_tile((int32_t)blockIdx.x, (int32_t)gridDim.x);
  const SmallDiv dx{(uint32_t)a.n[0], a.inv[0]}, dy{(uint32_t)a.n[1], a.inv[1]},
      dz{(uint32_t)a.n[2], a.inv[2]};
  const uint32_t r0 = dx.div(tile), bx = tile - r0 * dx.d, bz = dy.div(r0), by = r0 - bz * dy.d;
  const int32_t x0 = (int32_t)dx.div(bx * (uint32_t)Lh), y0 = (int32_t)dy.div(by * (uint32_t)L),
                z0 = (int32_t)dz.div(bz * (uint32_t)L);
  const int32_t nx = (int32_t)dx.div((bx + 1) * (uint32_t)Lh) - x0,
                ny = (int32_t)dy.div((by + 1) * (uint32_t)L) - y0,
                nz = (int32_t)dz.div((bz + 1) * (uint32_t)L) - z0;
  const int32_t hx = a.n[0] > 1 ? 3 : 0, w = nx + 2 * hx, rows = ny + 8;
  auto wrap = [](int32_t v, int32_t n) { return v < 0 ? v + n : (v >= n ? v - n : v); };
  const int32_t s = min(tid, rows * w - 1);
  const int32_t r = (int32_t)(((float)s + 0.5f) * __builtin_amdgcn_rcpf((float)w)), j = s - r * w;
  const bool has = tid < rows * w;
  const int32_t x = wrap(x0 - hx + j, Lh), y = wrap(y0 - 4 + r, L);
  // whether a stage that leaves out m rows and c columns on either side has the place
  auto in = [&](int32_t m, int32_t c) {
    return has && r >= m && r < rows - m && (hx == 0 || (j >= c && j < w - c));
  };
  const bool inA = in(1, 1), inB = in(2, 2), inC = in(3, 2), inD = in(4, 3);
  const int32_t q0 = z0 - 3;
  const int32_t p = (y + q0) & 1;  // A's x parity at step 0; B's is the same, C's and D's not
  const int32_t lx = hx || x < Lh - 1 ? 1 : 1 - Lh, mx = hx || x > 0 ? -1 : Lh - 1;
  // bytes from a plane's start in LDS to the site's place and its neighbours'
  constexpr int32_t B = (int32_t)E;
  const int32_t is = s * B, ipy = (s + w) * B, imy = (s - w) * B;
  const int32_t ipx[2] = {is + (p ? lx : 0) * B, is + (p ? 0 : lx) * B};
  const int32_t imx[2] = {is + (p ? 0 : mx) * B, is + (p ? mx : 0) * B};
  const uint32_t g = (uint32_t)(y * Lh + x) * E, gm = (uint32_t)(wrap(y - 1, L) * Lh + x) * E;
  const uint32_t d = (uint32_t)(x > 0 ? -1 : Lh - 1) * E;
  const uint32_t gx[2] = {g + (p ? 0u : d), g + (p ? d : 0u)};
  const char* sp[6];
  const char* Jp[6];
  char* out[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    sp[k] = (const char*)(a.in + k * Nh);
    Jp[k] = (const char*)(a.J + k * Nh);
    out[k] = (char*)(a.out + k * Nh);
  }
  const uint32_t zb = (uint32_t)zs * E;
  auto at = [](const char* base, uint32_t off) { return *(const R*)(base + off); };
  R s0[3], c1[3], ja[4][6], jb[4][6];  // couplings of four steps, step t's in set t mod 4
  // bonds of the site on the plane at byte offset zo, the plane below it at zm
  auto load_bonds = [&](auto C, auto Par, R (&jj)[6], uint32_t zo, uint32_t zm) {
    constexpr int o = 3 * decltype(C)::value, n = 3 - o, par = decltype(Par)::value;
    const uint32_t own = g + zo;
    jj[0] = at(Jp[o], own);
    jj[1] = at(Jp[n], gx[par] + zo);
    jj[2] = at(Jp[o + 1], own);
    jj[3] = at(Jp[n + 1], gm + zo);
    jj[4] = at(Jp[o + 2], own);
    jj[5] = at(Jp[n + 2], g + zm);
  };
  auto load_spin = [&](int c, R (&v)[3], uint32_t zo) {
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] = at(sp[3 * c + k], g + zo);
  };
  auto store = [&](auto C, uint32_t zo, const Vec3<R>& v) {
    constexpr int o = 3 * decltype(C)::value;
    *(R*)(out[o] + (g + zo)) = v.x;
    *(R*)(out[o + 1] + (g + zo)) = v.y;
    *(R*)(out[o + 2] + (g + zo)) = v.z;
  };
  auto field = [&](const char* cur, const char* up, const char* dn, int32_t px, int32_t mxp,
                   const R (&jj)[6]) {
    R h[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      auto ld = [&](const char* plane, int32_t i) { return *(const R*)(plane + i + k * N * B); };
      R acc = jj[0] * ld(cur, px);
      acc = dev_fma(jj[1], ld(cur, mxp), acc);
      acc = dev_fma(jj[2], ld(cur, ipy), acc);
      acc = dev_fma(jj[3], ld(cur, imy), acc);
      acc = dev_fma(jj[4], ld(up, is), acc);
      acc = dev_fma(jj[5], ld(dn, is), acc);
      h[k] = acc;
    }
    return Vec3<R>{h[0], h[1], h[2]};
  };
  auto get = [&](const char* plane) {
    const R* v = (const R*)(plane + is);
    return Vec3<R>{v[0], v[N], v[2 * N]};
  };
  auto put = [&](char* plane, const Vec3<R>& v) {
    R* o = (R*)(plane + is);
    o[0] = v.x;
    o[N] = v.y;
    o[2 * N] = v.z;
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  // Where planes q, q - 1, ... (colour 1: q + 2, q + 1, ...) are in LDS and planes q + 3, q +
  // 2, ... in the arrays, in bytes: turned by one place a step.  (Indices modulo 6, 7 and L at
  // each use were 250 scalar instructions a step and wave, more than a compute unit issues
  // while it issues the vector ones.)
  int32_t o0[K0], o1[K1];
#pragma unroll
  for (int k = 0; k < K0; ++k) o0[k] = k * 3 * N * B;
#pragma unroll
  for (int k = 0; k < K1; ++k) o1[k] = k * 3 * N * B;
  uint32_t zo[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) zo[k] = zb * (uint32_t)wrap(wrap(q0 + 3 - k, L), L);
  auto P0 = [&](int o) { return (char*)l0 + o0[-o]; };
  auto P1 = [&](int o) { return (char*)l1 + o1[2 - o]; };
  const int32_t end = z0 + nz;
  auto step = [&](auto Uc, int32_t q) {
    constexpr int U = decltype(Uc)::value, V = (U + 1) & 3, par = U & 1;
    using Other = std::integral_constant<int, 1 - par>;
    if (inA) put(P0(0), reflect(Vec3<R>{s0[0], s0[1], s0[2]},
                                field(P1(0), P1(1), P1(-1), ipx[par], imx[par], ja[U])));
    if (inC && q >= z0 + 2) {
      const Vec3<R> v = reflect(get(P0(-3)), field(P1(-3), P1(-2), P1(-4), ipx[1 - par],
                                                   imx[1 - par], ja[V]));
      put(P0(-3), v);
      if (inD && q >= z0 + 3 && q < end + 3) store(I0{}, zo[6], v);
    }
    // for the next step (past the last one: values nobody uses)
    load_spin(0, s0, zo[2]);
    load_bonds(I0{}, Other{}, ja[V], zo[2], zo[3]);
    __syncthreads();
    if (inB && q >= z0 - 1)
      put(P1(-1), reflect(get(P1(-1)), field(P0(-1), P0(0), P0(-2), ipx[par], imx[par], jb[U])));
    if (inD && q >= z0 + 4)
      store(I1{}, zo[7], reflect(get(P1(-4)), field(P0(-4), P0(-3), P0(-5), ipx[1 - par],
                                                    imx[1 - par], jb[V])));
    if (has) put(P1(2), Vec3<R>{c1[0], c1[1], c1[2]});
    load_spin(1, c1, zo[0]);
    load_bonds(I1{}, Other{}, jb[V], zo[3], zo[4]);
    __syncthreads();
    const int32_t t0 = o0[K0 - 1], t1 = o1[K1 - 1];
#pragma unroll
    for (int k = K0 - 1; k > 0; --k) o0[k] = o0[k - 1];
#pragma unroll
    for (int k = K1 - 1; k > 0; --k) o1[k] = o1[k - 1];
    o0[0] = t0;
    o1[0] = t1;
#pragma unroll
    for (int k = 7; k > 0; --k) zo[k] = zo[k - 1];
    zo[0] = zo[1] + zb;
    if (zo[0] == zb * (uint32_t)L) zo[0] = 0;
  };
  {
    R c[3][3];  // colour 1 of planes q0 - 1, q0, q0 + 1
#pragma unroll
    for (int k = 0; k < 3; ++k) load_spin(1, c[k], zo[4 - k]);
    load_spin(0, s0, zo[3]);
    load_bonds(I0{}, I0{}, ja[0], zo[3], zo[4]);
    load_spin(1, c1, zo[1]);
    load_bonds(I1{}, I0{}, jb[0], zo[4], zo[5]);
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (has) put(P1(k - 1), Vec3<R>{c[k][0], c[k][1], c[k][2]});
  }
  __syncthreads();
  const int32_t last = end + 3;
  for (int32_t q = q0; q <= last; q += 4) {
    step(I0{}, q);
    if (q + 1 > last) break;
    step(I1{}, q + 1);
    if (q + 2 > last) break;
    step(std::integral_constant<int, 2>{}, q + 2);
    if (q + 3 > last) break;
    step(std::integral_constant<int, 3>{}, q + 3);
  }
}

template <typename R>
__global__ __launch_bounds__((RowSize<R, false>::A)) void phase_kernel(PhaseArgs<R> a) {
  row_march<R, PassMode::OverRelax, false>(a);
}

template <typename R, PassMode MC>
__global__ __launch_bounds__((RowSize<R, true>::A)) void phase_mc_kernel(PhaseArgs<R> a) {
  row_march<R, MC, false>(a);
}

template <typename R, PassMode MC>
__global__ __launch_bounds__((RowSize<R, true>::A)) void phase_mc_wave_kernel(PhaseArgs<R> a) {
  row_march<R, MC, true>(a);
}

}  // namespace

bool phase_supported(int32_t L) {
  return L <= kPhaseMaxL && ((L >= kPhaseMinL && L % 2 == 0) || phase_always(L));
}

bool phase_always(int32_t L) { return L >= 64 && L <= kPhaseMaxL && L % 64 == 0; }

namespace {

uint32_t row_inv(int32_t d) { return d > 1 ? 0xFFFFFFFFu / (uint32_t)d + 1u : 0u; }

// Tiles of 64 columns, all of them (the kernel deals 64 columns and the halo's to a row): a
// wave per row and the halo columns on the waves behind those, so that a load of the tile's
// columns is two cache lines, not three or four.  us of the launch with four hits (one), items
// row by row / a wave per row: L = 512 1587 / 1510 (1564 / 1394), 1024 14038 / 13751 (14083 /
// 12668).  With fewer columns lanes are idle: 448, 56 columns, 1056 / 1221.  The estimate
// below does not weigh the form, so these two lattices are the only ones cut so.
template <typename R, bool MC>
constexpr bool kByWave = MC && sizeof(R) == 4;

// Threads of tiles of that many columns and rows (hx: tiles narrower than the lattice; even:
// all of them nx columns), 0 if the kernel does not hold them.
template <typename R, bool MC>
int32_t row_threads(int32_t nx, int32_t ny, int32_t hx, bool even, bool* waves) {
  using Size = RowSize<R, MC>;
  const int32_t H = MC ? 1 : 0, r0 = ny + 2 + 2 * H, r1 = r0 + 2;
  const int32_t n0 = r0 * (nx + 2 * hx), n1 = r1 * (nx + 4 * hx);
  *waves = kByWave<R, MC> && hx && even && nx == 64;
  const int32_t T = (*waves ? 64 * r0 + 2 * r0 + 63 : n0 + 63) & ~63;
  return T <= Size::A && n0 <= Size::A && n1 <= Size::C1 &&
                 (*waves ? 64 * r1 + 4 * r1 : n1) <= 2 * T
             ? T
             : 0;
}

template <typename R>
int32_t pair_threads(int32_t nx, int32_t ny, int32_t hx, bool, bool* waves) {
  *waves = false;
  const int32_t T = ((ny + 8) * (nx + 6 * hx) + 63) & ~63;
  return T <= kPairThreads<R> ? T : 0;
}

// The tiles for an L^3 lattice: the smallest of an estimate fitted to 5000 timed plans of 60
// lattices (its choice is 1 to 1.5% behind the best of them on average, 15% at worst): the
// steps of a workgroup, nz and `fill` for the pipeline, times its threads and a fixed part,
// and the bytes of its planes, more where the tile is cut in x.  `most` workgroups per
// compute unit, one after the other: one is the longest run in z; with more stages two or
// three sometimes leave fewer units idle, and up to eight where a plane has more tiles than
// there are units.  `ragged`: what a cut that is not on a cache line costs, as columns.
struct PlanFit {
  float fill, fixed, bytes, ends, cut, edge;
  int32_t most, narrow;  // narrow: the fewest columns of a tile that does not have them all
  float ragged = 0.0f;
};
template <class Threads>
bool row_plan(const PlanFit& f, int32_t L, int32_t line, Threads threads, int32_t (&n)[3]) {
  constexpr int kCUs = 256;
  const int32_t Lh = L / 2;
  float best = 0.0f;
  for (int32_t px = 1; px <= 16; ++px) {
    const int32_t nx = (Lh + px - 1) / px, hx = px > 1 ? 1 : 0;
    if (px > 1 && nx < f.narrow) break;
    bool waves;
    for (int32_t ny = 2;; ++ny) {
      const int32_t T = threads(nx, ny, hx, Lh % px == 0, &waves);
      if (!T) break;
      const int32_t ty = (L + ny - 1) / ny;
      if ((L + ty - 1) / ty != ny) continue;  // no fewer tiles than with the next smaller ny
      for (int32_t k = 1; k <= f.most; ++k) {
        const int32_t tz = std::max(1, std::min(L / 3, k * kCUs / (ty * px)));
        const int32_t nz = (L + tz - 1) / tz, rounds = (tz * ty * px + kCUs - 1) / kCUs;
        const float edge = f.edge + (nx % line || Lh % px ? f.ragged : 0.0f);
        const float halo = (float)hx * (f.cut + edge / (float)nx);
        const float cost =
            (float)rounds * (((float)nz + f.fill) * ((float)T + f.fixed) +
                             f.bytes * (float)(nx * ny) * ((float)nz + f.ends) * (1.0f + halo));
        if (best == 0.0f || cost < best) {
          best = cost;
          n[0] = px;
          n[1] = ty;
          n[2] = tz;
        }
      }
    }
  }
  return best > 0.0f;
}

template <class Threads>
bool plan_tiles(const PlanFit& f, int32_t L, int32_t elem, Threads threads, PhasePlan* p) {
  if (!phase_supported(L) || !row_plan(f, L, 128 / elem, threads, p->n)) return false;
  const int32_t Lh = L / 2, px = p->n[0], py = p->n[1];
  p->threads = threads((Lh + px - 1) / px, (L + py - 1) / py, px > 1 ? 1 : 0, Lh % px == 0,
                       &p->waves);
  return p->threads > 0;
}

template <typename R, bool MC>
bool plan_rows(int32_t L, PhasePlan* p) {
  constexpr bool F32 = sizeof(R) == 4;
  // The phase alone, us before / now that runs in z are also cut to fill the last round of
  // workgroups and x is cut on cache lines: binary64 L = 288 465 / 431, 448 1877 / 1540, 512
  // 2526 / 2350, 544 5307 / 3051, 576 4220 / 3330; binary32 416 701 / 623, 544 1740 / 1426,
  // 576 2049 / 1595, 700 3581 / 3121, 900 7894 / 6977, 1024 13586 / 10847.  Binary32 up to L =
  // 400, whose planes have fewer tiles than there are units, keeps the first estimate (352:
  // 363 and 389).
  const bool tall = L > 400;
  const PlanFit f = MC ? (F32 ? PlanFit{2.0f, 500.0f, 2.0f, 4.0f, 0.0f, 32.0f, 3, 14}
                              : PlanFit{4.0f, 200.0f, 1.0f, 0.0f, 0.2f, 8.0f, 3, 14})
                       : (!F32   ? PlanFit{5.0f, 200.0f, 2.0f, 1.0f, 0.1f, 8.0f, 8, 24, 2.0f}
                          : tall ? PlanFit{10.0f, 1000.0f, 8.0f, 1.0f, 0.0f, 16.0f, 8, 24, 12.0f}
                                 : PlanFit{2.5f, 200.0f, 4.0f, 1.0f, 0.2f, 16.0f, 1, 24});
  return plan_tiles(f, L, (int32_t)sizeof(R), row_threads<R, MC>, p);
}

template <typename R>
bool plan_pair(int32_t L, PhasePlan* p) {
  constexpr PlanFit f = sizeof(R) == 4 ? PlanFit{12.0f, 2000.0f, 4.0f, 4.0f, 0.0f, 32.0f, 3, 14}
                                       : PlanFit{12.0f, 500.0f, 1.0f, 0.0f, 0.0f, 32.0f, 3, 14};
  return plan_tiles(f, L, (int32_t)sizeof(R), pair_threads<R>, p);
}

template <typename R>
dim3 set_tiles(PhaseArgs<R>& a, const PhasePlan& p) {
  for (int k = 0; k < 3; ++k) {
    a.n[k] = p.n[k];
    a.inv[k] = row_inv(p.n[k]);
  }
  return dim3((unsigned)(p.n[0] * p.n[1] * p.n[2]));
}

template <typename R, PassMode MODE>
hipError_t launch_rows(PhaseArgs<R> a, hipStream_t st) {
  constexpr bool MC = MODE != PassMode::OverRelax;
  PhasePlan p;
  if (!plan_rows<R, MC>(a.L, &p) || (MC && !a.partials)) return hipErrorInvalidValue;
  const dim3 grid = set_tiles(a, p), block((unsigned)p.threads);
  if constexpr (!MC)
    hipLaunchKernelGGL((phase_kernel<R>), grid, block, 0, st, a);
  else if constexpr (!kByWave<R, MC>)
    hipLaunchKernelGGL((phase_mc_kernel<R, MODE>), grid, block, 0, st, a);
  else if (p.waves)
    hipLaunchKernelGGL((phase_mc_wave_kernel<R, MODE>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((phase_mc_kernel<R, MODE>), grid, block, 0, st, a);
  return hipGetLastError();
}

}  // namespace

bool phase_plan(int32_t L, int32_t elem, int32_t passes, PhasePlan* p) {
  if (passes == 2) return elem == 4 ? plan_rows<float, false>(L, p) : plan_rows<double, false>(L, p);
  if (passes == 3) return elem == 4 ? plan_rows<float, true>(L, p) : plan_rows<double, true>(L, p);
  return passes == 4 && (elem == 4 ? plan_pair<float>(L, p) : plan_pair<double>(L, p));
}

template <typename R>
hipError_t launch_phase_pair(const PhaseArgs<R>& a0, hipStream_t st) {
  PhaseArgs<R> a = a0;
  PhasePlan p;
  if (!plan_pair<R>(a.L, &p)) return hipErrorInvalidValue;
  const dim3 grid = set_tiles(a, p);
  hipLaunchKernelGGL(phase_pair_kernel<R>, grid, dim3((unsigned)p.threads), 0, st, a);
  return hipGetLastError();
}
template hipError_t launch_phase_pair<float>(const PhaseArgs<float>&, hipStream_t);
template hipError_t launch_phase_pair<double>(const PhaseArgs<double>&, hipStream_t);

template <typename R>
hipError_t launch_phase(const PhaseArgs<R>& a, PassMode mc, hipStream_t st) {
  switch (mc == PassMode::Metropolis ? metropolis_mode(a.k_hits) : mc) {
    case PassMode::OverRelax: return launch_rows<R, PassMode::OverRelax>(a, st);
    case PassMode::HeatBath: return launch_rows<R, PassMode::HeatBath>(a, st);
    case PassMode::MetropolisFull: return launch_rows<R, PassMode::MetropolisFull>(a, st);
    case PassMode::Metropolis: return launch_rows<R, PassMode::Metropolis>(a, st);
  }
  return hipErrorInvalidValue;
}

template hipError_t launch_phase<float>(const PhaseArgs<float>&, PassMode, hipStream_t);
template hipError_t launch_phase<double>(const PhaseArgs<double>&, PassMode, hipStream_t);

}  // namespace hsg
