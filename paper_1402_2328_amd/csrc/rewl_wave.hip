// One wavefront per walker: the Wang-Landau sweep of batches of few walkers,
// and the initialisation of every batch (further down).
//
// The sweep.
// With one walker per lane (rewl_sweep.hip) an attempt is a serial chain of
// two LDS round trips and some eighty dependent instructions, about 300 to
// 430 ns, and a batch of few walkers leaves most of the chip idle.  Here the
// 64 lanes of a wavefront work for one walker:
//   * Everything about an attempt that does not depend on the attempts
//     before it is done for 64 attempts at once, one per lane: the Philox
//     block (a function of the attempt number), the site and its
//     neighbours, the energy change on the lattice as it stands at the start
//     of the 64, and the acceptance test turned round: instead of
//     u < exp(delta), delta > ln u, with ln u known in advance.
//   * ln g and the histogram of the 64 bins around the walker sit in
//     registers, one bin per lane.
//   * The attempts are then made one after the other in wave-uniform code:
//     the energy change and ln g at the proposed bin come out of the lanes by
//     v_readlane, so no memory is touched and an attempt costs one
//     subtraction, two compares and some twenty cheap instructions.
//   * An accepted move changes the lattice under the attempts still to be
//     made.  A mask per site of the lanes that pick it (or, where the masks
//     would not fit in LDS, a count) tells a lane beforehand whether its move
//     concerns a later attempt, or any other on the same site; only then (one
//     accepted move in seven at L = 32) are the other lanes' neighbours and
//     energy changes updated.  Against counts alone the masks took 8 Ising L =
//     32 instances from 122 to 115 ns per attempt, q = 10 Potts L = 20 from
//     168 to 149.
// What bounds it: a lone wavefront issues one instruction every four cycles
// and the attempts of one walker are a chain, so the time is the number of
// instructions per attempt (37 at Ising L = 32, of them 18 vector: 160 of 256
// cycles) and the waits between dependent scalar and vector ones; the chip
// is busy from 1024 walkers, one per SIMD.  Branches cost more than what they
// skip: with early exits for rejected moves the attempt had 37 instructions,
// 7 branches and took 327 cycles, without them and 40 instructions 295.
// Measured per attempt against one lane per walker in the default shape, on
// 1024 walkers: Ising L = 32 115 against 453 ns, L = 64 110 against 591,
// q = 10 Potts L = 20 152 against 554.
// The accepted sites are written back to the lattice (bytes in LDS) after
// the 64.  The page of 64 bins moves when the walker comes near its edge:
// stored and reloaded whole, a coalesced row segment each way.
#include <math.h>

#include <type_traits>

#include "rewl_device.h"
#include "rewl_internal.h"

namespace rewl {

namespace {

constexpr int kWave = 64;

// Orders LDS accesses of different lanes of the one wavefront of a
// workgroup: the hardware executes a wavefront's LDS instructions in order,
// so only the compiler has to keep them so (no instruction is emitted).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int lane_of(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ float lane_of(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ uint64_t lane_of(uint64_t v, int lane) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane) << 32 |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
}
__device__ __forceinline__ double lane_of(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Number of bytes of x that are not zero, each below 128.
__device__ __forceinline__ int nonzero_bytes(uint32_t x) {
  return __builtin_popcount((x + 0x7F7F7F7Fu) & 0x80808080u);
}

// The lattice around one attempt's site, per lane.  `same(s)` and
// `change(s, v)` keep it up to date when another attempt sets site s to v.
template <int MODEL>
struct Around;

// Ising: bits 0..3 the right, left, lower and upper neighbour, bit 4 the
// site's own spin (1 = up).
template <>
struct Around<kIsing> {
  uint32_t n;
  __device__ __forceinline__ void load(const uint8_t* lat, int site, int nr, int nl, int nd, int nu,
                                       uint32_t, int) {
    auto up = [&](int s) { return (uint32_t)(lat[s] >> 7) ^ 1u; };  // +1 -> 1, -1 (0xFF) -> 0
    n = up(nr) | up(nl) << 1 | up(nd) << 2 | up(nu) << 3 | up(site) << 4;
  }
  static constexpr int kUnit = 4;  // energy of a bin step with bshift = 0
  // bin step of the flip: agreeing neighbours - 2 (Delta E = 2 s sum, bins of 4)
  __device__ __forceinline__ int step(int, int) const {
    const uint32_t own = (uint32_t)((int32_t)(n << 27) >> 31);  // all ones when up
    return __builtin_popcount(~(n ^ own) & 15u) - 2;
  }
  __device__ __forceinline__ int proposed() const { return (int)((n >> 4) & 1u) ^ 1; }
  __device__ __forceinline__ int own() const { return (int)((n >> 4) & 1u); }
  __device__ __forceinline__ void change(int s, int, int site, int nr, int nl, int nd, int nu, int) {
    n ^= (nr == s ? 1u : 0u) | (nl == s ? 2u : 0u) | (nd == s ? 4u : 0u) | (nu == s ? 8u : 0u) |
         (site == s ? 16u : 0u);
  }
  static __device__ __forceinline__ uint8_t byte_of(int v) { return v ? (uint8_t)1 : (uint8_t)0xFF; }
};

// Potts: the four neighbours' values in the bytes of n, the site's own value
// s0, the draw u among the q - 1 others and the proposed value v.
template <>
struct Around<kPotts> {
  uint32_t n;
  int s0, u, v;
  __device__ __forceinline__ void propose(int q) {
    const int t = s0 + 1 + u;
    v = (int)min((uint32_t)t, (uint32_t)(t - q));  // t - q wraps round when t < q
  }
  __device__ __forceinline__ void load(const uint8_t* lat, int site, int nr, int nl, int nd, int nu,
                                       uint32_t draw, int q) {
    n = (uint32_t)lat[nr] | (uint32_t)lat[nl] << 8 | (uint32_t)lat[nd] << 16 | (uint32_t)lat[nu] << 24;
    s0 = lat[site];
    u = (int)__umulhi(draw, (uint32_t)(q - 1));
    propose(q);
  }
  static constexpr int kUnit = 1;
  // bin step: (neighbours equal to s0) - (neighbours equal to v)
  __device__ __forceinline__ int step(int, int bshift) const {
    return (nonzero_bytes(n ^ ((uint32_t)v * 0x01010101u)) -
            nonzero_bytes(n ^ ((uint32_t)s0 * 0x01010101u))) >> bshift;
  }
  __device__ __forceinline__ int proposed() const { return v; }
  __device__ __forceinline__ int own() const { return s0; }
  __device__ __forceinline__ void change(int s, int val, int site, int nr, int nl, int nd, int nu, int q) {
    const uint32_t m = (nr == s ? 0xFFu : 0u) | (nl == s ? 0xFF00u : 0u) | (nd == s ? 0xFF0000u : 0u) |
                       (nu == s ? 0xFF000000u : 0u);
    n = (n & ~m) | (((uint32_t)val * 0x01010101u) & m);
    s0 = site == s ? val : s0;
    propose(q);
  }
  static __device__ __forceinline__ uint8_t byte_of(int v) { return (uint8_t)v; }
};

// The site that one attempt picks, its neighbours and the lattice around
// them, per lane; and whether another of the wavefront's attempts picks one
// of the five.
template <int MODEL, bool MASKS>
struct Pick {
  int site, nr, nl, nd, nu;
  Around<MODEL> ar;
  // r: the attempt's random numbers
  __device__ __forceinline__ void look(const uint8_t* lat, uint4 r, int side, int N, int q) {
    site = (int)__umulhi(r.x, (uint32_t)N);
    // site = floor(r.x L^2 / 2^32), so its row is floor(r.x L / 2^32)
    const int y = (int)__umulhi(r.x, (uint32_t)side);
    const int x = site - __mul24(y, side);
    nr = site + (x + 1 == side ? 1 - side : 1);
    nl = site + (x == 0 ? side - 1 : -1);
    nd = site + (y + 1 == side ? side - N : side);
    nu = site + (y == 0 ? N - side : -side);
    ar.load(lat, site, nr, nl, nd, nu, r.y, q);
  }
  // live: the lane makes an attempt; picked: zero before and after, a byte
  // per site that counts the lanes that pick it, or (MASKS) their mask.
  // Returns the lanes whose five sites another lane picks one of; with masks
  // only those that a later lane picks next to, or any other the same.
  __device__ __forceinline__ uint64_t compare(uint8_t* picked, bool live) const {
    if constexpr (MASKS) {
      uint64_t* const masks = reinterpret_cast<uint64_t*>(picked);
      const uint64_t me = 1ull << threadIdx.x;
      if (live) atomicOr(reinterpret_cast<unsigned long long*>(masks + site), (unsigned long long)me);
      wave_order();
      const uint64_t same = masks[site], next_to = masks[nr] | masks[nl] | masks[nd] | masks[nu];
      wave_order();
      masks[site] = 0;
      return __ballot(((next_to & ~(me | (me - 1))) | (same & ~me)) != 0);
    }
    if (live) atomicAdd(reinterpret_cast<uint32_t*>(picked) + (site >> 2), 1u << ((site & 3) * 8));
    wave_order();
    const bool others = picked[site] > 1 || (picked[nr] | picked[nl] | picked[nd] | picked[nu]) != 0;
    wave_order();
    picked[site] = 0;
    return __ballot(others);
  }
  __device__ __forceinline__ uint64_t load(const uint8_t* lat, uint8_t* picked, uint4 r, bool live,
                                           int side, int N, int q) {
    look(lat, r, side, N, q);
    return compare(picked, live);
  }
  __device__ __forceinline__ int step(int q, int bshift) const { return ar.step(q, bshift); }
  // attempt i was accepted: every lane's view follows
  __device__ __forceinline__ void follow(int i, int q) {
    ar.change(lane_of(site, i), lane_of(ar.proposed(), i), site, nr, nl, nd, nu, q);
  }
  // the accepted lanes' sites (moved) back to the lattice: a site that other
  // lanes touch (shared) was kept up to date in every lane that holds it
  __device__ __forceinline__ void settle(uint8_t* lat, uint64_t moved, uint64_t shared, int lane) const {
    if ((moved >> lane) & 1) {
      const int val = ((shared >> lane) & 1) ? ar.own() : ar.proposed();
      lat[site] = Around<MODEL>::byte_of(val);
    }
    wave_order();
  }
};

// The same for Ising lattices (L >= 3) with the masks kept in registers: an
// accepted move updates the bin steps of the lanes in two masks (7 vector
// instructions and no compare, against 20 for looking every lane's five sites
// over).
struct PickIsing {
  int site, sgn, st;       // sgn: the site's spin, +1 or -1; st: bin step of its flip
  uint64_t same, next_to;  // lanes that pick this site, or a neighbour of it
  __device__ __forceinline__ uint64_t load(const uint8_t* lat, uint8_t* picked, uint4 r, bool live,
                                           int side, int N, int) {
    uint64_t* const masks = reinterpret_cast<uint64_t*>(picked);
    site = (int)__umulhi(r.x, (uint32_t)N);
    const int y = (int)__umulhi(r.x, (uint32_t)side);
    const int x = site - __mul24(y, side);
    const int nr = site + (x + 1 == side ? 1 - side : 1), nl = site + (x == 0 ? side - 1 : -1);
    const int nd = site + (y + 1 == side ? side - N : side), nu = site + (y == 0 ? N - side : -side);
    const uint64_t me = 1ull << threadIdx.x;
    if (live) atomicOr(reinterpret_cast<unsigned long long*>(masks + site), (unsigned long long)me);
    auto spin = [&](int s) { return (int)(int8_t)lat[s]; };
    sgn = spin(site);
    st = sgn * (spin(nr) + spin(nl) + spin(nd) + spin(nu)) / 2;  // agreeing neighbours - 2
    wave_order();
    same = masks[site];
    next_to = masks[nr] | masks[nl] | masks[nd] | masks[nu];
    wave_order();
    masks[site] = 0;
    return __ballot(((next_to & ~(me | (me - 1))) | (same & ~me)) != 0);
  }
  __device__ __forceinline__ int step(int, int) const { return st; }
  // attempt i was accepted: with s the flipped spin's old value, the step
  // (site's spin times neighbours' sum) / 2 falls by sgn s next to it and
  // changes sign where it is the site
  __device__ __forceinline__ void follow(int i, int) {
    const int lane = threadIdx.x;
    const int t = sgn * lane_of(sgn, i);
    st -= (lane_of(next_to, i) >> lane) & 1 ? t : 0;
    const bool s = (lane_of(same, i) >> lane) & 1;
    st = s ? -st : st;
    sgn = s ? -sgn : sgn;
  }
  __device__ __forceinline__ void settle(uint8_t* lat, uint64_t moved, uint64_t shared, int lane) const {
    if ((moved >> lane) & 1) lat[site] = (uint8_t)(((shared >> lane) & 1) ? sgn : -sgn);
    wave_order();
  }
};

// ln g of one bin, the walker's running value, and the acceptance test in
// both precisions.
template <int PREC>
struct LnG;

template <>
struct LnG<kFP64> {
  double v;
  using Bound = double;
  __device__ __forceinline__ void load(const DevPtrs& P, int64_t e, bool in) { v = in ? P.lng[e] : INFINITY; }
  __device__ __forceinline__ void store(const DevPtrs& P, int64_t e) const { P.lng[e] = v; }
  __device__ __forceinline__ LnG at(int lane) const { return LnG{lane_of(v, lane)}; }
  __device__ __forceinline__ void put(bool here, const LnG& o) { v = here ? o.v : v; }
  __device__ __forceinline__ double minus(const LnG& o) const { return v - o.v; }
  // this (or o) plus ln f; frozen walkers add 0.0: ln g >= +0, so x + 0.0 is
  // x bit for bit
  __device__ __forceinline__ void choose(bool other, const LnG& o, double lnf, bool) {
    double a = o.v + lnf, b = v + lnf;
    asm("" : "+v"(a), "+v"(b));  // keeps the compiler from choosing first
    v = other ? a : b;
  }
  // The uniform u = u53 2^-53 lies in [hi, hi + 1) 2^-32.  delta >= yes
  // makes u < exp(delta) certain, delta < no rules it out; both bounds keep a
  // distance of 2^-12 from ln(hi + 1) - 32 ln 2 and ln(hi) - 32 ln 2, against
  // less than 2e-5 for the roundings of hi, the hardware base-2 logarithm
  // (values up to 32, one ulp 4e-6) and the product with ln 2.  Between them
  // (probability below 1e-3) accept64_flat decides.  hi = 0 gives no =
  // -inf; for delta < -40 and hi >= 1 delta < no holds, a rejection as in
  // accept64.
  static __device__ __forceinline__ void bounds(uint4 r, double& yes, double& no) {
    const float h = (float)r.z;
    yes = (double)((__builtin_amdgcn_logf(h + 1.0f) - 32.0f) * 0x1.62e430p-1f + 0x1p-12f);
    no = (double)((__builtin_amdgcn_logf(h) - 32.0f) * 0x1.62e430p-1f - 0x1p-12f);
  }
  static __device__ __forceinline__ bool accept(uint32_t hi, uint32_t lo, double delta) {
    return accept64_flat(hi, lo, delta);
  }
};

template <>
struct LnG<kFP32C> {
  float h, l;
  using Bound = float;
  __device__ __forceinline__ void load(const DevPtrs& P, int64_t e, bool in) {
    h = in ? P.lhi[e] : INFINITY;
    l = in ? P.llo[e] : 0.0f;
  }
  __device__ __forceinline__ void store(const DevPtrs& P, int64_t e) const {
    P.lhi[e] = h;
    P.llo[e] = l;
  }
  __device__ __forceinline__ LnG at(int lane) const { return LnG{lane_of(h, lane), lane_of(l, lane)}; }
  __device__ __forceinline__ void put(bool here, const LnG& o) {
    h = here ? o.h : h;
    l = here ? o.l : l;
  }
  __device__ __forceinline__ float minus(const LnG& o) const { return (h - o.h) + (l - o.l); }
  // a two-float add of 0 could renormalise the pair: frozen walkers skip it
  __device__ __forceinline__ void choose(bool other, const LnG& o, double lnf, bool frozen) {
    if (other) *this = o;
    if (!frozen) df_add1(h, l, (float)lnf, h, l);
  }
  // the same for the 24-bit uniform u exactly; u = 0 (no = -inf) is left to
  // the exact test, which knows the window
  static __device__ __forceinline__ void bounds(uint4 r, float& yes, float& no) {
    const float t = (__builtin_amdgcn_logf((float)(r.z >> 8)) - 24.0f) * 0x1.62e430p-1f;
    yes = r.z >> 8 ? t + 0x1p-12f : INFINITY;
    no = t - 0x1p-12f;
  }
  static __device__ __forceinline__ bool accept(uint32_t hi, uint32_t, float delta) {
    return accept32_flat(hi >> 8, delta);
  }
};

}  // namespace

// ---------------------------------------------------------------------------
// Initialisation: random spins (one Philox block per 4 sites), full energy,
// then warm-up into the window: greedy moves that never increase the
// distance of E to the window, budget 1000 N; on failure one restart from an
// extreme state (ground state below the middle of the range, checkerboard
// above) and a second budget.
//
// One wavefront per walker.  The slowest walker of a batch decides: in the
// ordered phase it makes up to a million attempts, of which few are
// accepted.  The distance of E + dE to the window decides a greedy move, so
// 64 attempts are judged at once and only the accepted ones (found by a
// ballot) go one after the other, each moving E and, where another attempt
// shares its site or a neighbour, the view of the lanes behind it.  The
// 64-instance mix (17455 walkers) is set up in 7.9 ms; one lane per walker on
// a lattice in device memory took 494 ms.
// ---------------------------------------------------------------------------
template <int MODEL>
__device__ __forceinline__ int32_t wave_energy(const uint8_t* lat, int side, int N, int lane) {
  int32_t e = 0;
  for (int s = lane; s < N; s += kWave) {
    const int y = s / side, x = s - y * side;
    const uint8_t s0 = lat[s], sr = lat[x + 1 == side ? s + 1 - side : s + 1],
                  sd = lat[y + 1 == side ? s + side - N : s + side];
    const int same = (s0 == sr) + (s0 == sd);
    e -= MODEL == kIsing ? 2 * same - 2 : same;
  }
  return wave_reduce(e, [](int32_t a, int32_t b) { return a + b; });
}

__device__ __forceinline__ int32_t dist_to(int32_t E, int32_t elo, int32_t ehi) {
  return max(max(elo - E, E - ehi), 0);
}

template <int MODEL>
__device__ __forceinline__ void init_walker(const DevPtrs& P, const InstDesc& I, int g, uint8_t* lat,
                                            uint8_t* picked) {
  const int lane = threadIdx.x;
  const int loc = g - I.slot_base;
  const int w = loc / I.m;
  const WinDesc W = P.win[I.win_base + w];
  const int side = I.L, N = I.N, q = I.q;
  const int words = I.npad >> 2;
  for (int i = lane; i < words; i += kWave) {
    const uint4 r = draw(I, (uint64_t)i, (uint32_t)loc, kTagInit);
    const uint32_t rv[4] = {r.x, r.y, r.z, r.w};
    uint32_t word = 0;
    for (int j = 0; j < 4; ++j) {
      const uint32_t v = MODEL == kIsing ? (rv[j] >> 31 ? 1u : 0xFFu) : __umulhi(rv[j], (uint32_t)q);
      if (4 * i + j < N) word |= v << (8 * j);
    }
    reinterpret_cast<uint32_t*>(lat)[i] = word;
    reinterpret_cast<uint32_t*>(picked)[i] = 0u;
  }
  wave_order();
  const int32_t elo = I.emin + W.lo * I.binw, ehi = I.emin + W.hi * I.binw;
  // in registers: behind the lattice stores the descriptor would be read anew
  const uint32_t k0 = I.key0, k1 = I.key1, tag = kTagWarm | ((uint32_t)I.inst << 8);
  int32_t E = __builtin_amdgcn_readfirstlane(wave_energy<MODEL>(lat, side, N, lane));
  uint64_t wa = 0;
  for (int phase = 0; phase < 2; ++phase) {
    const int budget = 1000 * N;
    for (int it = 0; it < budget && dist_to(E, elo, ehi) > 0;) {
      const int n = budget - it < kWave ? budget - it : kWave;
      const uint64_t a = wa + (uint64_t)lane;
      const uint4 r = philox10(make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)loc, tag), k0, k1);
      Pick<MODEL, false> pick;
      pick.look(lat, r, side, N, q);
      int dE = pick.ar.step(q, 0) * Around<MODEL>::kUnit;
      uint64_t left = n < kWave ? (1ull << n) - 1 : ~0ull, moved = 0, shared = 0;
      int made = n;
      while (left) {
        const int d = dist_to(E, elo, ehi);
        const uint64_t ok = __ballot(dist_to(E + dE, elo, ehi) <= d) & left;
        if (!ok) break;
        if (!moved) shared = pick.compare(picked, lane < n);
        // Moves without a change of energy that no other attempt shares a
        // site with leave everything that decides about the rest as it is:
        // all of them up to the first other one are accepted together.
        const uint64_t stop = ok & (__ballot(dE != 0) | shared);
        moved |= stop ? ok & ((stop & -stop) - 1) : ok;
        if (!stop) break;
        const int i = __builtin_ctzll(stop);
        moved |= 1ull << i;
        E += lane_of(dE, i);
        if ((shared >> i) & 1) {
          pick.follow(i, q);
          dE = pick.ar.step(q, 0) * Around<MODEL>::kUnit;
        }
        if (dist_to(E, elo, ehi) == 0) {
          made = i + 1;
          break;
        }
        left &= i < kWave - 1 ? ~0ull << (i + 1) : 0ull;
      }
      pick.settle(lat, moved, shared, lane);
      it += made;
      wa += (uint64_t)made;
    }
    if (dist_to(E, elo, ehi) == 0) break;
    if (phase == 0) {
      const uint4 r = draw(I, wa++, (uint32_t)loc, kTagWarm);
      const bool below = (W.lo + W.hi) < (I.nbins - 1);
      int a, b;
      if (MODEL == kIsing) {
        a = (r.x >> 31) ? 1 : 0xFF;
        b = a ^ 0xFE;
      } else {
        a = (int)__umulhi(r.x, (uint32_t)q);
        b = a + 1 + (int)__umulhi(r.y, (uint32_t)(q - 1));
        b = (b >= q) ? b - q : b;
      }
      for (int s = lane; s < N; s += kWave) {
        const int y = s / side, x = s - y * side;
        lat[s] = (uint8_t)((below || ((x + y) & 1) == 0) ? a : b);
      }
      wave_order();
      E = __builtin_amdgcn_readfirstlane(wave_energy<MODEL>(lat, side, N, lane));
    }
  }
  uint32_t* const gsp = reinterpret_cast<uint32_t*>(P.spins + I.spin_base + (int64_t)loc * I.npad);
  for (int i = lane; i < words; i += kWave) gsp[i] = reinterpret_cast<const uint32_t*>(lat)[i];
  if (lane == 0) {
    P.cfg[g] = g;
    P.E[g] = E;
    P.att[g] = 0;
    P.watt[g] = wa;
    if (dist_to(E, elo, ehi) != 0) atomicMin(&P.ist[I.inst].error, -7);
  }
}

// LATER: a slice after the first, of walkers from `first` on.  With an offset
// that is not the constant 0 the whole kernel comes out 4 % slower (7.28
// against 7.01 ms for the 64-instance mix).
template <bool LATER>
__global__ __launch_bounds__(kWave) void k_init(DevPtrs P, int32_t lat_bytes, int32_t first) {
  extern __shared__ __align__(16) uint8_t wlds[];
  const int g = (LATER ? first : 0) + (int)blockIdx.x;
  int lo = 0, hi = P.n_inst - 1;  // the instance that owns slot g
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (P.inst[mid].slot_base <= g) lo = mid;
    else hi = mid - 1;
  }
  const InstDesc& I = P.inst[lo];
  if (I.model == kIsing) init_walker<kIsing>(P, I, g, wlds, wlds + lat_bytes);
  else init_walker<kPotts>(P, I, g, wlds, wlds + lat_bytes);
}

hipError_t launch_init(const DevPtrs& P, int32_t lat_bytes, hipStream_t s) {
  return in_slices(P.n_slots, kWave, [&](int32_t first, int32_t n) {
    hipLaunchKernelGGL(first ? k_init<true> : k_init<false>, dim3(n), dim3(kWave), (size_t)2 * lat_bytes, s, P,
                       lat_bytes, first);
  });
}

template <int MODEL, int PREC, bool MASKS>
__global__ __launch_bounds__(kWave) void k_sweep_wave(DevPtrs P, int32_t wg_offset, int32_t lat_bytes,
                                                      int64_t flips) {
  extern __shared__ __align__(16) uint8_t wlds[];
  uint8_t* const lat = wlds;               // [lat_bytes] spins
  // attempts of the 64 that pick a site: a count in a byte, or a 64-bit mask
  uint8_t* const picked = wlds + lat_bytes;
  using L = LnG<PREC>;
  using Bound = typename L::Bound;
  const WgDesc wg = P.wg[wg_offset + (int)blockIdx.x];
  const InstDesc& I = P.inst[wg.inst];
  if (P.ist[wg.inst].done || P.ist[wg.inst].error) return;
  const int lane = threadIdx.x;
  const int g = wg.slot_first;
  const int loc = g - I.slot_base;
  const int w = loc / I.m, k = loc - w * I.m;
  const WinDesc W = P.win[I.win_base + w];
  const WinState WS = P.wst[I.win_base + w];
  const int nb = W.nb, side = I.L, N = I.N, q = I.q, bshift = I.binw_shift;
  const bool frozen = WS.frozen != 0;
  double lnf = frozen ? 0.0 : WS.lnf;
  asm("" : "+v"(lnf));  // in vector registers: the other operand of the sums is scalar
  const uint32_t k0 = I.key0, k1 = I.key1;
  const uint32_t tagw = kTagMC | ((uint32_t)I.inst << 8);
  const int64_t row = W.lng_base + (int64_t)k * nb;  // of bin lo
  const int D = (MODEL == kPotts && bshift == 0) ? 4 : 2;  // largest bin step of one move

  uint64_t att = P.att[g];
  int b0 = ((P.E[g] - I.emin) >> bshift) - W.lo;  // bin counted from the window's lowest
  if (b0 < 0 || b0 >= nb) {
    // only reachable through corrupted state: flag the instance and keep
    // every access inside the window (the instance's results are void)
    if (lane == 0) atomicMin(&P.ist[wg.inst].error, -6);
    b0 = b0 < 0 ? 0 : nb - 1;
  }

  uint32_t* const gsp = reinterpret_cast<uint32_t*>(P.spins + I.spin_base +
                                                    (int64_t)(P.cfg[g] - I.slot_base) * I.npad);
  const int words = I.npad >> 2;  // npad <= lat_bytes
  for (int i = lane; i < words; i += kWave) reinterpret_cast<uint32_t*>(lat)[i] = gsp[i];
  for (int i = lane; i < (MASKS ? 8 : 1) * words; i += kWave) reinterpret_cast<uint32_t*>(picked)[i] = 0u;
  wave_order();

  // ---- the page: lane l holds bin pb + l; c is the walker's bin in page
  // coordinates.  Lanes outside the window (up to D of them beside it) hold
  // +inf, so that a proposal out of the window is rejected by its delta of
  // -inf.  Every U attempts the page is moved if the walker has come within U
  // D bins of an end of it that is not the window's, so a proposed bin is
  // always in the page.
  constexpr int U = MODEL == kPotts ? 2 : 4;
  int pb, c, c_lo, c_span;
  bool in;  // this lane's bin is in the window
  L ln;
  uint32_t hist;  // counts gathered in this lane's bin
  auto load_page = [&](int b) {
    pb = b - kWave / 2;
    pb = pb > nb - kWave + D ? nb - kWave + D : pb;
    pb = pb < -D ? -D : pb;
    c = b - pb;
    c_lo = pb > -D ? U * D : 0;
    c_span = (pb + kWave < nb + D ? kWave - 1 - U * D : kWave - 1) - c_lo;
    in = (uint32_t)(pb + lane) < (uint32_t)nb;
    ln.load(P, row + pb + lane, in);
    hist = 0;
  };
  auto store_page = [&]() {
    if (!frozen && in) {
      ln.store(P, row + pb + lane);
      if (hist) atomicAdd(&P.H[row + pb + lane], hist);
    }
  };
  auto follow = [&]() {
    if (__builtin_expect((uint32_t)(c - c_lo) > (uint32_t)c_span, 0)) {
      store_page();
      __syncthreads();  // other lanes' stores are read back
      load_page(c + pb);
      __syncthreads();
    }
  };
  load_page(b0);
  L cur = ln.at(c);  // ln g at the walker's bin, in every lane

  for (int64_t t = 0; t < flips; t += kWave) {
    const int n = flips - t < kWave ? (int)(flips - t) : kWave;
    // ---- one attempt per lane
    const uint64_t a = att + (uint64_t)lane;
    const uint4 r = philox10(make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)loc, tagw), k0, k1);
    std::conditional_t<MASKS && MODEL == kIsing, PickIsing, Pick<MODEL, MASKS>> pick;
    const uint64_t shared = pick.load(lat, picked, r, lane < n, side, N, q);
    int step = pick.step(q, bshift);
    Bound yes, no;
    L::bounds(r, yes, no);
    uint64_t moved = 0;  // attempts whose move was accepted

    // ---- the attempts in order, wave-uniform and (but for the rare cases)
    // without branches: a branch costs a lone wave more than the few
    // instructions it would skip
    auto attempt = [&](int i) {
      const int cn = c + lane_of(step, i);
      const L next = ln.at(cn);
      const auto delta = cur.minus(next);
      const uint64_t bit = 1ull << i;
      const uint64_t sure = __ballot(delta >= yes);
      const uint64_t open = __ballot(!(delta < no));
      uint64_t acc = sure & bit;
      if (__builtin_expect((((open & ~sure) | (sure & shared)) & bit) != 0, 0)) {
        if (!acc && (uint32_t)(pb + cn) < (uint32_t)nb)
          acc = __ballot(L::accept((uint32_t)lane_of((int)r.z, i), (uint32_t)lane_of((int)r.w, i),
                                   delta)) & bit;  // the same in every lane
        if (acc & shared) {
          pick.follow(i, q);
          step = pick.step(q, bshift);
        }
      }
      moved |= acc;
      c = acc ? cn : c;
      // both outcomes with ln f added, off the chain of the decision
      cur.choose(acc != 0, next, lnf, frozen);
      const bool here = lane == c;
      ln.put(here, cur);
      hist += here ? 1u : 0u;
    };
    int i = 0;
    for (; i + U <= n; i += U) {
      follow();
#pragma unroll
      for (int j = 0; j < U; ++j) attempt(i + j);
    }
    follow();
    for (; i < n; ++i) attempt(i);
    att += (uint64_t)n;
    pick.settle(lat, moved, shared, lane);
  }

  store_page();
  for (int i = lane; i < words; i += kWave) gsp[i] = reinterpret_cast<const uint32_t*>(lat)[i];
  if (lane == 0) {
    P.E[g] = I.emin + ((W.lo + pb + c) << bshift);  // every energy sits on the bin grid
    P.att[g] = att;
  }
}

hipError_t launch_sweep_wave(const DevPtrs& P, int cls, int32_t wg_offset, int32_t n_wg,
                             int32_t lat_bytes, int32_t l_min, int64_t flips, hipStream_t s) {
  if (n_wg <= 0) return hipSuccess;
  const bool masks = wave_masks(cls, lat_bytes, l_min, n_wg);
  using Fn = void (*)(DevPtrs, int32_t, int32_t, int64_t);
  const Fn potts = P.prec == kFP64 ? (masks ? (Fn)k_sweep_wave<kPotts, kFP64, true> : (Fn)k_sweep_wave<kPotts, kFP64, false>)
                                   : (masks ? (Fn)k_sweep_wave<kPotts, kFP32C, true> : (Fn)k_sweep_wave<kPotts, kFP32C, false>);
  const Fn ising = P.prec == kFP64 ? (masks ? (Fn)k_sweep_wave<kIsing, kFP64, true> : (Fn)k_sweep_wave<kIsing, kFP64, false>)
                                   : (masks ? (Fn)k_sweep_wave<kIsing, kFP32C, true> : (Fn)k_sweep_wave<kIsing, kFP32C, false>);
  const Fn f = cls == 2 ? potts : ising;
  const size_t lds = (size_t)wave_lds_bytes(cls, lat_bytes, l_min, n_wg);
  return in_slices(n_wg, kWave, [&](int32_t first, int32_t n) {
    hipLaunchKernelGGL(f, dim3(n), dim3(kWave), lds, s, P, wg_offset + first, lat_bytes, flips);
  });
}

}  // namespace rewl
