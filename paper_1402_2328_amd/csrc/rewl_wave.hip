// The Wang-Landau sweep with one wavefront per walker, for batches of few
// walkers.
//
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
//     made.  A byte per site counts how many of the 64 attempts pick it, so a
//     lane knows beforehand whether its site or a neighbour of it is picked
//     by another attempt; only then (a third of the accepted moves at
//     L = 32 and less) are the other lanes' neighbours and energy changes
//     updated.
// What bounds it: a lone wavefront issues one instruction every four cycles
// and the attempts of one walker are a chain, so the time is the number of
// instructions per attempt (40, of them 20 vector) and the waits between
// dependent scalar and vector ones (295 cycles in all at Ising L = 32; the
// chip is busy from 1024 walkers, one per SIMD).  Branches cost more than
// what they skip: with early exits for rejected moves the attempt had 37
// instructions, 7 branches and took 327 cycles.
// Measured per attempt against one lane per walker in the default shape, on
// 1024 walkers: Ising L = 32 135 against 453 ns, L = 64 122 against 591,
// q = 10 Potts L = 20 173 against 554 (two-float 208 against 622).
// The accepted sites are written back to the lattice (bytes in LDS) after
// the 64.  The page of 64 bins moves when the walker comes near its edge:
// stored and reloaded whole, a coalesced row segment each way.
#include <math.h>

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

// ln g of one bin, the walker's running value, and the acceptance test in
// both precisions.
template <int PREC>
struct LnG;

template <>
struct LnG<kFP64> {
  double v;
  using Bound = double;
  __device__ __forceinline__ void load(const DevPtrs& P, int64_t e) { v = P.lng[e]; }
  __device__ __forceinline__ void store(const DevPtrs& P, int64_t e) const { P.lng[e] = v; }
  __device__ __forceinline__ LnG at(int lane) const { return LnG{lane_of(v, lane)}; }
  __device__ __forceinline__ void put(bool here, const LnG& o) { v = here ? o.v : v; }
  __device__ __forceinline__ double minus(const LnG& o) const { return v - o.v; }
  // frozen walkers add 0.0: ln g >= +0, so x + 0.0 is x bit for bit
  __device__ __forceinline__ void add(double lnf, bool) { v = v + lnf; }
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
  __device__ __forceinline__ void load(const DevPtrs& P, int64_t e) {
    h = P.lhi[e];
    l = P.llo[e];
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
  __device__ __forceinline__ void add(double lnf, bool frozen) {
    if (!frozen) df_add1(h, l, (float)lnf, h, l);
  }
  // the same for the 24-bit uniform u exactly; u = 0 accepts whatever delta
  // is (both bounds -inf)
  static __device__ __forceinline__ void bounds(uint4 r, float& yes, float& no) {
    const float t = (__builtin_amdgcn_logf((float)(r.z >> 8)) - 24.0f) * 0x1.62e430p-1f;
    yes = t + 0x1p-12f;
    no = t - 0x1p-12f;
  }
  static __device__ __forceinline__ bool accept(uint32_t hi, uint32_t, float delta) {
    return accept32_flat(hi >> 8, delta);
  }
};

}  // namespace

template <int MODEL, int PREC>
__global__ __launch_bounds__(kWave) void k_sweep_wave(DevPtrs P, int32_t wg_offset, int32_t lat_bytes,
                                                      int64_t flips) {
  extern __shared__ __align__(16) uint8_t wlds[];
  uint8_t* const lat = wlds;               // [lat_bytes] spins
  uint8_t* const picked = wlds + lat_bytes;  // [lat_bytes] attempts of the 64 that pick a site
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
  const double lnf = frozen ? 0.0 : WS.lnf;
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
  for (int i = lane; i < words; i += kWave) {
    reinterpret_cast<uint32_t*>(lat)[i] = gsp[i];
    reinterpret_cast<uint32_t*>(picked)[i] = 0u;
  }
  wave_order();

  // ---- the page: lane l holds bin pb + l (l <= top); c is the walker's bin
  // in page coordinates.  Every U attempts the page is moved if the walker
  // has come within U D bins of an end of it that is not the window's, so a
  // proposed bin outside [0, top] is outside the window.
  constexpr int U = MODEL == kPotts ? 2 : 4;
  const int top = nb < kWave ? nb - 1 : kWave - 1;
  int pb, c, c_lo, c_span;
  L ln;
  uint32_t hist;  // counts gathered in this lane's bin
  auto load_page = [&](int b) {
    pb = b - kWave / 2;
    pb = pb > nb - kWave ? nb - kWave : pb;
    pb = pb < 0 ? 0 : pb;
    c = b - pb;
    c_lo = pb > 0 ? U * D : 0;
    c_span = (pb + kWave < nb ? kWave - 1 - U * D : kWave - 1) - c_lo;
    ln.load(P, row + pb + (lane <= top ? lane : top));
    hist = 0;
  };
  auto store_page = [&]() {
    if (!frozen && lane <= top) {
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
    const int site = (int)__umulhi(r.x, (uint32_t)N);
    // site = floor(r.x L^2 / 2^32), so its row is floor(r.x L / 2^32)
    const int y = (int)__umulhi(r.x, (uint32_t)side);
    const int x = site - __mul24(y, side);
    const int nr = site + (x + 1 == side ? 1 - side : 1), nl = site + (x == 0 ? side - 1 : -1);
    const int nd = site + (y + 1 == side ? side - N : side), nu = site + (y == 0 ? N - side : -side);
    if (lane < n)
      atomicAdd(reinterpret_cast<uint32_t*>(picked) + (site >> 2), 1u << ((site & 3) * 8));
    Around<MODEL> ar;
    ar.load(lat, site, nr, nl, nd, nu, r.y, q);
    wave_order();
    const bool others = picked[site] > 1 || (picked[nr] | picked[nl] | picked[nd] | picked[nu]) != 0;
    const uint64_t shared = __ballot(others);
    wave_order();
    picked[site] = 0;
    int step = ar.step(q, bshift);
    Bound yes, no;
    L::bounds(r, yes, no);
    uint64_t moved = 0;  // attempts whose move was accepted

    // ---- the attempts in order, wave-uniform and (but for the rare cases)
    // without branches: a branch costs a lone wave more than the few
    // instructions it would skip
    auto attempt = [&](int i) {
      const int cn = c + lane_of(step, i);
      const uint64_t bit = (uint32_t)cn <= (uint32_t)top ? 1ull << i : 0;  // 0: outside the window
      const L next = ln.at(cn & (kWave - 1));
      const auto delta = cur.minus(next);
      const uint64_t sure = __ballot(delta >= yes) & bit;
      const uint64_t open = __ballot(!(delta < no)) & bit;
      uint64_t acc = sure;
      if (__builtin_expect(((sure ^ open) | (sure & shared)) != 0, 0)) {
        if (sure != open)
          acc = __ballot(L::accept((uint32_t)lane_of((int)r.z, i), (uint32_t)lane_of((int)r.w, i),
                                   delta)) & bit;  // the same in every lane
        if (acc & shared) {
          ar.change(lane_of(site, i), lane_of(ar.proposed(), i), site, nr, nl, nd, nu, q);
          step = ar.step(q, bshift);
        }
      }
      moved |= acc;
      c = acc ? cn : c;
      if (acc) cur = next;
      cur.add(lnf, frozen);
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
    // ---- accepted sites back to the lattice: a site that other attempts
    // touch was kept up to date in every lane that holds it
    if ((moved >> lane) & 1) {
      const int val = ((shared >> lane) & 1) ? ar.own() : ar.proposed();
      lat[site] = Around<MODEL>::byte_of(val);
    }
    wave_order();
  }

  store_page();
  for (int i = lane; i < words; i += kWave) gsp[i] = reinterpret_cast<const uint32_t*>(lat)[i];
  if (lane == 0) {
    P.E[g] = I.emin + ((W.lo + pb + c) << bshift);  // every energy sits on the bin grid
    P.att[g] = att;
  }
}

hipError_t launch_sweep_wave(const DevPtrs& P, int cls, int32_t wg_offset, int32_t n_wg,
                             int32_t lat_bytes, int64_t flips, hipStream_t s) {
  if (n_wg <= 0) return hipSuccess;
  const dim3 grid(n_wg), blk(kWave);
  const size_t lds = (size_t)2 * lat_bytes;  // at most 8 KiB
  if (P.prec == kFP64) {
    if (cls == 2) hipLaunchKernelGGL((k_sweep_wave<kPotts, kFP64>), grid, blk, lds, s, P, wg_offset, lat_bytes, flips);
    else hipLaunchKernelGGL((k_sweep_wave<kIsing, kFP64>), grid, blk, lds, s, P, wg_offset, lat_bytes, flips);
  } else {
    if (cls == 2) hipLaunchKernelGGL((k_sweep_wave<kPotts, kFP32C>), grid, blk, lds, s, P, wg_offset, lat_bytes, flips);
    else hipLaunchKernelGGL((k_sweep_wave<kIsing, kFP32C>), grid, blk, lds, s, P, wg_offset, lat_bytes, flips);
  }
  return hipGetLastError();
}

}  // namespace rewl
