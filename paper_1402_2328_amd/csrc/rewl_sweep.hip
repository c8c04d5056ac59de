// The REWL hot path on gfx950: Wang-Landau sweeps, one walker per lane.
//
// Each workgroup is one 64-lane wavefront holding up to 64 walkers of one
// instance.  For the duration of a launch every walker keeps in LDS
//   * its lattice: Ising spins as bit rows (one 32-bit word per row for
//     L <= 32, two for L <= 64), Potts spins as 4-bit nibbles (q <= 16) or
//     bytes;
//   * a page of PG = 2^k bins of its ln g window, direct-mapped (bin b lives
//     in slot b mod PG), with the histogram H (Ising L = 32: the counts; else
//     the increments gathered since the bin entered).  Walkers move at most
//     D bins per attempt (D = 2 for Ising and q = 2 Potts, 4 for q >= 3
//     Potts); the page always covers [bin - 2D, bin + 2D] inside the window
//     and follows the walker by at
//     most D bins per move: the bin that leaves is written back (ln g
//     stored, its H count stored or its increments added to device memory) and
//     the bin that enters shares its slot; the entering ln g is loaded into
//     registers and committed one attempt later, since it cannot be reached
//     before then, so the load has a whole attempt to arrive (the leaving
//     bin is read out of LDS at the shift and written back one attempt
//     later as well).  Windows of at most PG bins live in LDS entirely.
// With nibble Potts lattices the workgroup also keeps, once for all its
// walkers, a table of every site's four neighbours (lattice word and nibble
// offset of each).
// Four compile-time copies of the attempt loop serve any L, L a power of
// two, Ising L = 32 (one word per row, neighbours by word rotation) and
// nibble Potts lattices with the neighbour table.
// LDS is rows of 32-bit words interleaved by lane: row e of lane l sits at
// word e * S + l (S = lanes per workgroup), so the words that one instruction
// touches across the wavefront fall into consecutive banks.  A page slot is
// three rows next to each other (both words of ln g, then H), so one address
// serves all three.
// What bounds it on a full chip is instruction issue, and the clock that the
// power of the wide multiplies and LDS accesses leaves: 109 vector
// instructions per wave-attempt on 1024 Ising L = 32 instances (122 with ln
// g and H as arrays of their own, bins counted from the range's lowest and
// every Philox round in full), 6.2 against 6.9 ms per sweep of 10^4 attempts
// with the wavefronts placed alike, 5.80 with H as counts; 136 against 167 on
// q = 10 Potts L = 20 in two-float FP32, 4.85 against 6.3 ms.  Random numbers come
// from Philox4x32-10 keyed by (walker slot, attempt), so results do not
// depend on the walker-to-lane mapping, page size or launch shape.
#include <math.h>

#include <mutex>
#include <type_traits>

#include "rewl_device.h"
#include "rewl_internal.h"

namespace rewl {

// Pins a Philox block in registers at this point of the program: an empty
// asm statement (no instruction) that takes the four words as in/out
// operands, so the compiler can neither sink the rounds that produce them
// below it nor merge slices across it.
#define REWL_PIN4(v) asm volatile("" : "+v"((v).x), "+v"((v).y), "+v"((v).z), "+v"((v).w))

// Element at a 32-bit byte offset from a wave-uniform base pointer (the
// scalar-base addressing mode of global memory instructions).
template <typename T>
__device__ __forceinline__ T* at_off(T* base, uint32_t byte_off) {
  return reinterpret_cast<T*>(reinterpret_cast<unsigned char*>(base) + byte_off);
}

// The 32-bit LDS word at a byte offset.  The sweep kernels have no static
// LDS, so their dynamic LDS starts at 0 (prepare_sweep_lds checks it), and
// offsets are addresses; through a pointer to the array every access would
// add its base first.
using LdsWord = __attribute__((address_space(3))) uint32_t;
__device__ __forceinline__ LdsWord& lds_word(int off) { return *(LdsWord*)(uintptr_t)(uint32_t)off; }
__device__ __forceinline__ void lds_add(int off, uint32_t v) {  // no return: the lane owns the word
  (void)__hip_atomic_fetch_add((LdsWord*)(uintptr_t)(uint32_t)off, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Potts proposal s0 -> v: the new value s0 + 1 + u (u < q - 1) taken
// modulo q by one unsigned minimum (v - q wraps round when v < q).
__device__ __forceinline__ int potts_wrap(int v, int q) {
  return (int)min((uint32_t)v, (uint32_t)(v - q));
}

// Energy change / J of a Potts move s0 -> v with neighbours a, b, c, d:
// (neighbours equal to s0) - (neighbours equal to v).  The four values are
// packed one per BITS-bit field (BITS = 4 for q <= 16, else 8); XOR with s
// copied into every field leaves a field zero exactly where the neighbour
// equals s, and OR-folding each field into its top bit (shift-or by
// BITS/2, .., 1 within the field) marks the fields that are not zero.  So
// the change is (nonzero fields for v) - (nonzero fields for s0), without
// compares.
template <int BITS>
__device__ __forceinline__ int potts_de(int a, int b, int c, int d, int s0, int v) {
  constexpr uint32_t rep = BITS == 4 ? 0x1111u : 0x01010101u;
  constexpr uint32_t top = BITS == 4 ? 0x8888u : 0x80808080u;
  const uint32_t n = (uint32_t)a | ((uint32_t)b << BITS) | ((uint32_t)c << (2 * BITS)) |
                     ((uint32_t)d << (3 * BITS));
  auto nonzero_fields = [&](uint32_t x) {
    if constexpr (BITS == 8) x |= x << 4;
    x |= x << 2;
    x |= x << 1;
    return __builtin_popcount(x & top);
  };
  // rep has 25 bits for BITS = 8, beyond a 24-bit multiply
  auto spread = [&](int x) { return BITS == 4 ? __mul24((uint32_t)x, rep) : (uint32_t)x * rep; };
  return nonzero_fields(n ^ spread(v)) - nonzero_fields(n ^ spread(s0));
}

// PROD: the workgroup has a second wavefront that computes the Philox
// blocks of the walkers' coming attempts, kRngChunk at a time, into a
// double buffer in LDS (chunk c in half c mod 2) while the walker wavefront
// consumes the previous chunk; one workgroup barrier per chunk hands over.
// This takes the RNG off the walkers' serial chain when few walkers share
// the chip; the blocks are the ones the walkers would compute themselves.
// S64: the workgroup's stride is 64 lanes, so that a row is 256 bytes and
// rows next to each other are reached by offsets in the instruction (one
// ds_read2st64_b32 for both words of an FP64 ln g).
// The sweep of workgroup-table entry wgi, with the launch's dynamic LDS.
// COUNTS: loops that keep whole counts of H in the page, not increments
// (h_in_page).
template <int MODEL, int PREC, int ROWW, bool PROD, bool S64, HCounts COUNTS>
__device__ __forceinline__ void sweep_body(const DevPtrs& P, const SweepShape& sh, int64_t flips, int wgi,
                                           unsigned char* lds) {
  const WgDesc wg = P.wg[wgi];
  const InstDesc& Ig = P.inst[wg.inst];
  const int S = S64 ? kSweepWave : sh.stride;
  const int NWL = sh.nw;   // lattice words per lane
  const int PG = sh.page;  // page slots per lane, a power of two
  const int PM = PG - 1;
  const int tid = threadIdx.x;
  const int lane = tid & (kSweepWave - 1);
  // Potts nibble lattices: a table of every site's four neighbours, shared
  // by the workgroup, 8 bytes per site after the page; then the RNG double
  // buffer [2][kRngChunk][S] at the next 16-byte boundary (its reads are 16
  // bytes wide), then a flag word
  const bool use_tab = MODEL == kPotts && sh.tab != 0;
  const size_t tab_off = ((size_t)4 * NWL * S + (size_t)12 * PG * S + 7) & ~(size_t)7;
  uint2* tab = reinterpret_cast<uint2*>(lds + tab_off);
  const size_t tab_end = tab_off + (use_tab ? (size_t)8 * Ig.N : 0);
  uint4* rbuf = reinterpret_cast<uint4*>(lds + ((tab_end + 15) & ~(size_t)15));
  bool skip = P.ist[wg.inst].done || P.ist[wg.inst].error;
  if (PROD) {
    // one decision for both wavefronts: both must reach every barrier
    int* flag = reinterpret_cast<int*>(rbuf + (size_t)2 * kRngChunk * S);
    if (tid == 0) *flag = skip ? 1 : 0;
    __syncthreads();
    skip = *flag != 0;
  }
  if (skip) return;
  if (use_tab) {
    // entry of site s = y L + x: for its right, left, lower and upper
    // neighbours the lattice word (9 bits, n >> 3) and the bit offset of
    // the nibble (5 bits, 4 (n & 7)), 14 bits each, two per 32-bit word
    const int Lt = Ig.L;
    for (int s = tid; s < Ig.N; s += (int)blockDim.x) {
      const int y = s / Lt, x = s - y * Lt;
      const int nr = y * Lt + (x + 1 == Lt ? 0 : x + 1), nl = y * Lt + (x == 0 ? Lt - 1 : x - 1);
      const int nd = (y + 1 == Lt ? 0 : y + 1) * Lt + x, nu = (y == 0 ? Lt - 1 : y - 1) * Lt + x;
      auto code = [](int n) { return (uint32_t)(n >> 3) | ((uint32_t)(n & 7) << 11); };
      tab[s] = make_uint2(code(nr) | code(nl) << 14, code(nd) | code(nu) << 14);
    }
    __syncthreads();
  }
  const bool active = lane < wg.count;
  const int64_t nchunks = (flips + kRngChunk - 1) / kRngChunk;
  uint32_t* lat = reinterpret_cast<uint32_t*>(lds);                           // [NWL][S]
  unsigned char* latb = lds;                                                   // byte view (Potts)
  // Potts spins: 4-bit nibbles (8 per word; every q <= 16) or bytes
  const int L = Ig.L, N = Ig.N, q = Ig.q, bshift = Ig.binw_shift;
  const bool nib = MODEL == kPotts && sh.nib != 0;
  const uint32_t k0 = Ig.key0, k1 = Ig.key1;
  const uint32_t tagw = kTagMC | ((uint32_t)Ig.inst << 8);
  const int D = (MODEL == kPotts && bshift == 0) ? 4 : 2;  // largest bin step of one move
  const int M = 2 * D;
  // row and column of a site: shifts and masks when L is a power of two
  const bool pow2 = (L & (L - 1)) == 0;
  const int Lm = L - 1;
  const int lgL = 31 - __builtin_clz((unsigned)L);

  if (PROD && tid >= kSweepWave) {
    // ---- RNG producer ----
    const int gp = wg.slot_first + lane;
    const int locp = gp - Ig.slot_base;
    const uint64_t att0 = active ? P.att[gp] : 0;
    auto fill = [&](int64_t c) {
      uint4* dst = rbuf + (size_t)(c & 1) * kRngChunk * S + lane;
      const int n = (flips - c * kRngChunk) < kRngChunk ? (int)(flips - c * kRngChunk) : kRngChunk;
      for (int i = 0; i < n; ++i) {
        const uint64_t a = att0 + (uint64_t)(c * kRngChunk + i);
        dst[(size_t)i * S] = philox10(make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)locp, tagw), k0, k1);
      }
    };
    if (active && nchunks > 0) fill(0);
    __syncthreads();
    for (int64_t c = 0; c < nchunks; ++c) {
      if (active && c + 1 < nchunks) fill(c + 1);
      __syncthreads();
    }
    return;
  }
  if (!active) return;
  const int g = wg.slot_first + lane;
  const int loc = g - Ig.slot_base;
  const int w = loc / Ig.m;
  const int k = loc - w * Ig.m;
  const WinDesc W = P.win[Ig.win_base + w];
  const WinState WS = P.wst[Ig.win_base + w];
  const int nb = W.nb;
  const bool frozen = WS.frozen != 0;
  const double lnf = WS.lnf;
  const float lnf32 = (float)WS.lnf;
  const double lnf_eff = frozen ? 0.0 : lnf;
  const uint32_t h_inc = frozen ? 0u : 1u;

  // The walkers of a workgroup are consecutive slots of one instance, so
  // their ln g / H rows form one span that starts at the row of the first
  // walker; bins are addressed by 32-bit offsets from that base.
  const int loc0 = wg.slot_first - Ig.slot_base;
  const int w0 = loc0 / Ig.m;
  const WinDesc W0 = P.win[Ig.win_base + w0];
  const int64_t gb0 = W0.lng_base + (int64_t)(loc0 - w0 * Ig.m) * W0.nb;
  const uint32_t eoff = (uint32_t)(W.lng_base + (int64_t)k * nb - gb0);  // of the window's lowest bin
  double* const lngw = PREC == kFP64 ? P.lng + gb0 : nullptr;
  float* const lhw = PREC == kFP64 ? nullptr : P.lhi + gb0;
  float* const llw = PREC == kFP64 ? nullptr : P.llo + gb0;
  uint32_t* const Hw = P.H + gb0;

  // the energy is tracked as its bin, counted from the window's lowest:
  // E = emin + (lo + bin) * binw
  const uint64_t att = P.att[g];
  int bin = ((P.E[g] - Ig.emin) >> bshift) - W.lo;
  if (bin < 0 || bin >= nb) {
    // only reachable through corrupted state: flag the instance and keep
    // every access inside the window (the instance's results are void)
    atomicMin(&P.ist[wg.inst].error, -6);
    bin = bin < 0 ? 0 : nb - 1;
  }

  // ---- stage in the lattice ----
  const int cfg = P.cfg[g];
  int8_t* gsp = P.spins + Ig.spin_base + (int64_t)(cfg - Ig.slot_base) * Ig.npad;
  if (MODEL == kIsing) {
    for (int y = 0; y < L; ++y) {
      for (int part = 0; part < ROWW; ++part) {
        uint32_t bits = 0;
        const int x0 = part * 32;
        const int xe = (L - x0) < 32 ? (L - x0) : 32;
        for (int b = 0; b < xe; ++b) bits |= (uint32_t)(gsp[y * L + x0 + b] > 0) << b;
        lat[(y * ROWW + part) * S + lane] = bits;
      }
    }
  } else if (nib) {
    for (int i = 0; i < ((N + 7) >> 3); ++i) {
      uint32_t bits = 0;
      for (int b = 0; b < 8 && 8 * i + b < N; ++b) bits |= (uint32_t)(uint8_t)gsp[8 * i + b] << (4 * b);
      lat[i * S + lane] = bits;
    }
  } else {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(gsp);
    const int nwi = (N + 3) >> 2;
    for (int i = 0; i < nwi; ++i) lat[i * S + lane] = src[i];
  }

  // ---- page: bins [base, base + cnt) of the window, slot of bin b = b & PM.
  // A slot is three rows of 32-bit words: ln g (FP64 low and high half, or
  // FP32C high and low part) and H (counts or increments).
  const int lane4 = lane * 4;
  const int S4 = S * 4;
  // byte offset of this lane's word in a row; addresses stay below 2^24, so
  // 24-bit multiplies (full rate) suffice
  auto prow = [&](int row) { return S64 ? (row << 8) + lane4 : __mul24(row, S4) + lane4; };
  const int pg4 = S4 * NWL + lane4;
  auto pslot = [&](int b) { return __mul24(b & PM, S64 ? 768 : 3 * S4) + pg4; };
  auto word = [&](int off, int row) -> LdsWord& {
    return lds_word(off + (S64 ? 256 * row : S4 * row));
  };
  auto get64 = [&](int off) { return __hiloint2double((int)word(off, 1), (int)word(off, 0)); };
  auto put64 = [&](int off, double v) {
    word(off, 0) = (uint32_t)__double2loint(v);
    word(off, 1) = (uint32_t)__double2hiint(v);
  };
  auto getf = [&](int off, int row) { return __uint_as_float(word(off, row)); };
  auto putf = [&](int off, int row, float v) { word(off, row) = __float_as_uint(v); };
  // H in the page: a bin's whole count, loaded with its ln g and stored back,
  // or the increments since it entered, added to device memory by an atomic
  // when it leaves.  h_in_page says which and why.
  const bool h_load = COUNTS == HCounts::kAllLoops || (COUNTS == HCounts::kRotationLoop && L == 32);
  const int cnt = nb < PG ? nb : PG;
  const int hi_pm = nb - cnt;  // highest page start; 0: the window is in LDS entirely
  int m_pm = __builtin_amdgcn_readfirstlane(M - PM);
  asm("" : "+s"(m_pm));  // one scalar, not taken apart into PG and the rest
  int base = bin - (PG >> 1);
  base = base > hi_pm ? hi_pm : base;
  base = base < 0 ? 0 : base;
  for (int i = 0; i < cnt; ++i) {
    const int b = base + i;
    const int j = pslot(b);
    const uint32_t e = eoff + (uint32_t)b;
    if (PREC == kFP64) {
      put64(j, *at_off(lngw, e << 3));
    } else {
      putf(j, 0, *at_off(lhw, e << 2));
      putf(j, 1, *at_off(llw, e << 2));
    }
    word(j, 2) = h_load ? *at_off(Hw, e << 2) : 0u;
  }
  constexpr int DMAX = (MODEL == kPotts) ? 4 : 2;
  // Bins in flight after a page shift of pend_n bins: slot pend_row[i] holds
  // the leaving bin of element pend_e + i with its ln g and H
  // (read from LDS) and gets the entering bin's ln g (loaded from device
  // memory); both are settled one attempt later, which keeps the LDS read's
  // latency out of the shift.
  int pend_n = 0;
  uint32_t pend_e = 0u;
  int pend_row[DMAX];
  uint32_t pend_h[DMAX], ev_h[DMAX];
  double pend_l[DMAX], ev_l[DMAX];
  float pend_hi[DMAX], pend_lo[DMAX], ev_hi[DMAX], ev_lo[DMAX];
#pragma unroll
  for (int i = 0; i < DMAX; ++i) {
    pend_row[i] = 0;
    pend_h[i] = ev_h[i] = 0u;
    pend_l[i] = ev_l[i] = 0.0;
    pend_hi[i] = pend_lo[i] = ev_hi[i] = ev_lo[i] = 0.0f;
  }
  // Settles the bins in flight: the leaving bins are written back (ln g
  // stored, H counts stored or increments added in device memory) and the
  // entering bins take their slots.
  auto settle = [&](auto counts) {
    // All lanes' loads have arrived here (vmcnt 0).  Waited for inside the
    // branch only, the compiler has to take them as pending after it, and
    // may wait again, then for the stores below as well, where the next
    // shift reuses their registers.
    __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
    for (int i = 0; i < DMAX; ++i) {
      if (i < pend_n) {
        const int j = pend_row[i];
        if (PREC == kFP64) {
          put64(j, pend_l[i]);
        } else {
          putf(j, 0, pend_hi[i]);
          putf(j, 1, pend_lo[i]);
        }
        word(j, 2) = counts ? pend_h[i] : 0u;
        if (PREC == kFP64) {
          *at_off(lngw, (pend_e << 3) + 8u * i) = ev_l[i];
        } else {
          *at_off(lhw, (pend_e << 2) + 4u * i) = ev_hi[i];
          *at_off(llw, (pend_e << 2) + 4u * i) = ev_lo[i];
        }
        if (counts) *at_off(Hw, (pend_e << 2) + 4u * i) = ev_h[i];
        else atomicAdd(at_off(Hw, (pend_e << 2) + 4u * i), ev_h[i]);
      }
    }
    pend_n = 0;
  };

  int jcur = pslot(bin);  // LDS offset of the current bin's slot
  double lcur = 0.0;
  float hcur = 0.0f, lcur_lo = 0.0f;
  if (PREC == kFP64) lcur = get64(jcur);
  else {
    hcur = getf(jcur, 0);
    lcur_lo = getf(jcur, 1);
  }

  auto pbyte = [&](int site) { return prow(site >> 2) + (site & 3); };
  auto pnib = [&](int site) { return prow(site >> 3); };  // word holding a nibble

  // Rest of an attempt once the proposal is known: ln g at the proposed
  // bin, acceptance, lattice and ln g / H update, page follow.  Without a
  // producer, the last two Philox slices of the block in flight (rn) are
  // placed beside the ln g read and the exponential.
  // bn is the proposed bin.  bn & PM always names a slot of the page, so the
  // ln g read stays in bounds when bn lies outside the window; its value is
  // then not used.
  uint2 tab_e = make_uint2(0u, 0u), tab_en = make_uint2(0u, 0u);  // neighbour table entries
  auto complete = [&](const uint4 r, uint4& rn, int bn, int nv, uint32_t wofs, uint32_t wrow,
                      uint32_t fm, int site, auto lkt, auto nbt) -> bool {
    constexpr bool NB = decltype(nbt)::value;
    constexpr bool TAB = decltype(lkt)::value == 3;
    constexpr bool H_LOAD = COUNTS == HCounts::kAllLoops ||
                            (COUNTS == HCounts::kRotationLoop && decltype(lkt)::value == 2);
    const bool inwin = (uint32_t)bn < (uint32_t)nb;
    const int jn = pslot(bn);
    bool acc;
    if (PREC == kFP64) {
      const double ln = get64(jn);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!PROD) {
        rn = philox_rounds<4, 7>(rn, k0, k1);
        REWL_PIN4(rn);
      }
      __builtin_amdgcn_sched_barrier(0);
      const bool a = accept64_fast(r.z, r.w, lcur - ln);
      if constexpr (!PROD) {
        rn = philox_rounds<7, 10>(rn, k0, k1);
        REWL_PIN4(rn);
        // the next attempt's neighbour table entry, read while this
        // attempt finishes
        if constexpr (TAB) tab_en = tab[__umulhi(rn.x, (uint32_t)N)];
      }
      acc = inwin && a;
      lcur = acc ? ln : lcur;
    } else {
      const float nh = getf(jn, 0);
      const float nl = getf(jn, 1);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!PROD) {
        rn = philox_rounds<4, 7>(rn, k0, k1);
        REWL_PIN4(rn);
      }
      __builtin_amdgcn_sched_barrier(0);
      const bool a = accept32_fast(r.z >> 8, (hcur - nh) + (lcur_lo - nl));
      if constexpr (!PROD) {
        rn = philox_rounds<7, 10>(rn, k0, k1);
        REWL_PIN4(rn);
        // the next attempt's neighbour table entry, read while this
        // attempt finishes
        if constexpr (TAB) tab_en = tab[__umulhi(rn.x, (uint32_t)N)];
      }
      acc = inwin && a;
      hcur = acc ? nh : hcur;
      lcur_lo = acc ? nl : lcur_lo;
    }
    if (MODEL == kIsing) {
      // the row word is written back either way (unchanged when rejected)
      lds_word((int)wofs) = acc ? wrow ^ fm : wrow;
    } else if (acc) {
      if constexpr (NB) {
        const int sh4 = (site & 7) * 4;
        lds_word((int)wofs) = (wrow & ~(15u << sh4)) | ((uint32_t)nv << sh4);
      } else {
        latb[pbyte(site)] = (unsigned char)nv;
      }
    }
    bin = acc ? bn : bin;
    jcur = acc ? jn : jcur;
    if (PREC == kFP64) {
      // frozen walkers add 0.0 and count 0: ln g >= +0 always, so x + 0.0
      // is x bit for bit, and the branch-free form needs no exec mask
      lcur = lcur + lnf_eff;
      put64(jcur, lcur);
      lds_add(jcur + (S64 ? 512 : 2 * S4), h_inc);
    } else if (!frozen) {
      // a two-float add of 0 could renormalise the pair, so frozen FP32C
      // walkers skip the update instead
      df_add1(hcur, lcur_lo, lnf32, hcur, lcur_lo);
      putf(jcur, 0, hcur);
      putf(jcur, 1, lcur_lo);
      lds_add(jcur + (S64 ? 512 : 2 * S4), 1u);
    }
    // settle the bins of the last shift, then follow the walker
    settle(std::bool_constant<H_LOAD>{});
    // bin + M - PM is the lowest page start that still covers bin + M,
    // bin - M the highest that covers bin - M (PM >= 2M); the start then
    // stays inside [0, hi_pm] (0 for a window that is in LDS entirely, which
    // never shifts).  Both are integer medians.
    constexpr bool MA = MODEL == kIsing;  // Ising: 2 % faster; Potts: 1-2 % slower
    const int nbase = med3_i32<MA>(med3_i32<MA>(base, bin + m_pm, bin - M), 0, hi_pm);
    if (nbase != base) {
      // up: the bins from the old start to the new one leave and those PG
      // above them enter; down: the bins from the new start to the old one
      // enter and those PG above them leave.  Either way they are counted
      // from the lower start, and each pair shares a slot.  A frozen walker
      // writes back its unchanged ln g and H.
      const bool up = nbase > base;
      const int bot = up ? base : nbase;
      pend_n = (up ? nbase : base) - bot;  // 1..D
      const uint32_t el = eoff + (uint32_t)bot;
      pend_e = el + (up ? 0u : (uint32_t)PG);
      const uint32_t en = el + (up ? (uint32_t)PG : 0u);
      base = nbase;
#pragma unroll
      for (int i = 0; i < DMAX; ++i) {
        if (i == 0 || i < pend_n) {
          const int j = pslot(bot + i);
          if (PREC == kFP64) {
            pend_l[i] = *at_off(lngw, (en << 3) + 8u * i);
            ev_l[i] = get64(j);
          } else {
            pend_hi[i] = *at_off(lhw, (en << 2) + 4u * i);
            pend_lo[i] = *at_off(llw, (en << 2) + 4u * i);
            ev_hi[i] = getf(j, 0);
            ev_lo[i] = getf(j, 1);
          }
          if (H_LOAD) pend_h[i] = *at_off(Hw, (en << 2) + 4u * i);
          ev_h[i] = word(j, 2);
          pend_row[i] = j;
        }
      }
    }
    return acc;
  };

  // Software pipeline: the Philox block of attempt t+1 (it depends only on
  // the attempt counter) is computed in three slices placed in the latency
  // shadows of attempt t -- after the lattice reads are issued, after the
  // ln g read is issued, and beside the exponential.  sched_barrier keeps
  // the compiler from hoisting the slices back together.
  // One attempt with Philox block r; without a producer it also computes
  // rn, the block of the next attempt, in slices.  The lattice form LK
  // (0: any L, 1: L a power of two, 2: Ising with L = 32, one word per row,
  // 3: Potts nibbles with the neighbour table) and NB (Potts nibbles)
  // select compile-time copies of the loop, chosen
  // once per launch, so that no branch splits the attempt's scheduling
  // region.
  auto attempt = [&](const uint4 r, uint4& rn, const PhiloxRun& pr, uint32_t an, auto lkt, auto nbt) {
    constexpr int LK = decltype(lkt)::value;
    constexpr bool P2 = LK >= 1;
    constexpr bool NB = decltype(nbt)::value;
    const int site = LK == 2 ? (int)(r.x >> 22) : (int)__umulhi(r.x, (uint32_t)N);
    if constexpr (LK == 2) {
      // Ising, L = 32: row y = site / 32 is one word, column x = site % 32.
      // Rotating the row right by x puts the spin at bit 0 and its right
      // neighbour at bit 1; one more rotation left puts the left neighbour
      // at bit 0 and the spin at bit 1.  Word shifts and rotations use the
      // low five bits of site, which is x.  The bin step is
      // db = (agreeing neighbours) - 2 (Delta E = 2 s sum, in bins of 4).
      // byte offsets of rows y, y + 1 and y - 1 of this lane
      uint32_t aw, ad, au;
      if constexpr (S64) {
        // r.x holds y in its top five bits; 32 rows are 8 KiB, so the wrap
        // is a mask
        aw = ((r.x >> 19) & 0x1F00u) | (uint32_t)lane4;
        ad = (aw + 0x100u) & 0x1FFFu;
        au = (aw - 0x100u) & 0x1FFFu;
      } else {
        const int y = site >> 5;
        aw = __mul24((uint32_t)y, (uint32_t)S4) + (uint32_t)lane4;
        ad = __mul24((uint32_t)((y + 1) & 31), (uint32_t)S4) + (uint32_t)lane4;
        au = __mul24((uint32_t)((y - 1) & 31), (uint32_t)S4) + (uint32_t)lane4;
      }
      uint32_t awk = aw;
      asm volatile("" : "+v"(awk));  // keep the address for the write-back
      const uint32_t wrow = lds_word((int)awk);
      const uint32_t wd = lds_word((int)ad);
      const uint32_t wu = lds_word((int)au);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!PROD) {
        rn = pr.first4(an);
        REWL_PIN4(rn);
      }
      __builtin_amdgcn_sched_barrier(0);
      const uint32_t fm = 1u << (site & 31);
      const uint32_t tr = __builtin_amdgcn_alignbit(wrow, wrow, (uint32_t)site);
      const uint32_t tl = __builtin_amdgcn_alignbit(tr, tr, 31u);
      const uint32_t hz = ~(tl ^ tr) & 3u;     // left and right agree with the spin
      const uint32_t vd = ~(wd ^ wrow) & fm;   // lower neighbour agrees
      const uint32_t vu = ~(wu ^ wrow) & fm;   // upper neighbour agrees
      const int bn = bin - 2 + __builtin_popcount(hz) + __builtin_popcount(vd) + __builtin_popcount(vu);
      complete(r, rn, bn, 0, awk, wrow, fm, site, lkt, nbt);
      return;
    }
    if constexpr (LK == 3) {
      // Potts nibbles with the neighbour table: the site's word and nibble
      // from the site, its neighbours' from the table entry read one
      // attempt ahead, so no row, column or wrap arithmetic
      const uint2 e = tab_e;
      // byte offset of lattice word wd of this lane: wd * 4S + 4 lane
      auto word_at = [&](uint32_t wd) {
        return lds_word(prow((int)wd));
      };
      const uint32_t wofs = (uint32_t)pnib(site);
      const uint32_t w0 = lds_word((int)wofs);
      const uint32_t w1 = word_at(__builtin_amdgcn_ubfe(e.x, 0, 9));
      const uint32_t w2 = word_at(__builtin_amdgcn_ubfe(e.x, 14, 9));
      const uint32_t w3 = word_at(__builtin_amdgcn_ubfe(e.y, 0, 9));
      const uint32_t w4 = word_at(__builtin_amdgcn_ubfe(e.y, 14, 9));
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!PROD) {
        rn = pr.first4(an);
        REWL_PIN4(rn);
      }
      __builtin_amdgcn_sched_barrier(0);
      const int s0 = (int)__builtin_amdgcn_ubfe(w0, (site & 7) * 4, 4);
      const int a = (int)__builtin_amdgcn_ubfe(w1, __builtin_amdgcn_ubfe(e.x, 9, 5), 4);
      const int b = (int)__builtin_amdgcn_ubfe(w2, __builtin_amdgcn_ubfe(e.x, 23, 5), 4);
      const int c = (int)__builtin_amdgcn_ubfe(w3, __builtin_amdgcn_ubfe(e.y, 9, 5), 4);
      const int d = (int)__builtin_amdgcn_ubfe(w4, __builtin_amdgcn_ubfe(e.y, 23, 5), 4);
      const int v = potts_wrap(s0 + 1 + (int)__umulhi(r.y, (uint32_t)(q - 1)), q);
      const int dE = potts_de<4>(a, b, c, d, s0, v);
      complete(r, rn, bin + (dE >> bshift), v, wofs, w0, 0u, site, lkt, nbt);
      return;
    }
    int y, x, xr, xl, yd, yu;
    if constexpr (P2) {  // shifts and masks
      y = site >> lgL;
      x = site & Lm;
      xr = (x + 1) & Lm;
      xl = (x - 1) & Lm;
      yd = (y + 1) & Lm;
      yu = (y - 1) & Lm;
    } else {
      // site = floor(r.x N / 2^32) with N = L^2, so its row
      // floor(site / L) = floor(r.x L / 2^32): one multiply, off the chain
      // of the site itself
      y = (int)__umulhi(r.x, (uint32_t)L);
      x = site - __mul24(y, L);
      xr = (x + 1 == L) ? 0 : x + 1;
      xl = (x == 0) ? L - 1 : x - 1;
      yd = (y + 1 == L) ? 0 : y + 1;
      yu = (y == 0) ? L - 1 : y - 1;
    }
    int db, nv = 0;
    int widx = 0;
    uint32_t wrow = 0, fm = 0;
    if (MODEL == kIsing) {
      // bit b of a row word: spin at x = 32 * part + b is +1
      int s0, a, b, c, d;
      if (ROWW == 1) {
        widx = prow(y);
        wrow = lds_word(widx);
        const uint32_t wu = lds_word(prow(yu));
        const uint32_t wd = lds_word(prow(yd));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!PROD) {
          rn = pr.first4(an);
          REWL_PIN4(rn);
        }
        __builtin_amdgcn_sched_barrier(0);
        s0 = (wrow >> x) & 1;
        a = (wrow >> xr) & 1;
        b = (wrow >> xl) & 1;
        c = (wd >> x) & 1;
        d = (wu >> x) & 1;
      } else {
        const int px = x >> 5;
        const uint32_t r0 = lds_word(prow(2 * y));
        const uint32_t r1 = lds_word(prow(2 * y + 1));
        const uint32_t wu = lds_word(prow(2 * yu + px));
        const uint32_t wd = lds_word(prow(2 * yd + px));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!PROD) {
          rn = pr.first4(an);
          REWL_PIN4(rn);
        }
        __builtin_amdgcn_sched_barrier(0);
        wrow = px ? r1 : r0;
        s0 = (wrow >> (x & 31)) & 1;
        a = (((xr >> 5) ? r1 : r0) >> (xr & 31)) & 1;
        b = (((xl >> 5) ? r1 : r0) >> (xl & 31)) & 1;
        c = (wd >> (x & 31)) & 1;
        d = (wu >> (x & 31)) & 1;
        widx = prow(2 * y + px);
      }
      // sigma = 2 bit - 1: dE = 2 s0 (sum of neighbours), bin step dE / 4
      db = (2 * s0 - 1) * (a + b + c + d - 2);
      fm = 1u << (x & 31);
    } else {
      const int rowy = __mul24(y, L);
      int s0, a, b, c, d;
      if constexpr (NB) {
        const int sa = rowy + xr, sb = rowy + xl, sc = __mul24(yd, L) + x, sd = __mul24(yu, L) + x;
        widx = pnib(site);
        wrow = lds_word(widx);
        s0 = (int)__builtin_amdgcn_ubfe(wrow, (site & 7) * 4, 4);
        a = (int)__builtin_amdgcn_ubfe(lds_word(pnib(sa)), (sa & 7) * 4, 4);
        b = (int)__builtin_amdgcn_ubfe(lds_word(pnib(sb)), (sb & 7) * 4, 4);
        c = (int)__builtin_amdgcn_ubfe(lds_word(pnib(sc)), (sc & 7) * 4, 4);
        d = (int)__builtin_amdgcn_ubfe(lds_word(pnib(sd)), (sd & 7) * 4, 4);
      } else {
        s0 = (int)latb[pbyte(site)];
        a = (int)latb[pbyte(rowy + xr)];
        b = (int)latb[pbyte(rowy + xl)];
        c = (int)latb[pbyte(__mul24(yd, L) + x)];
        d = (int)latb[pbyte(__mul24(yu, L) + x)];
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!PROD) {
        rn = pr.first4(an);
        REWL_PIN4(rn);
      }
      __builtin_amdgcn_sched_barrier(0);
      const int v = potts_wrap(s0 + 1 + (int)__umulhi(r.y, (uint32_t)(q - 1)), q);
      nv = v;
      db = (NB ? potts_de<4>(a, b, c, d, s0, v) : potts_de<8>(a, b, c, d, s0, v)) >> bshift;
    }
    complete(r, rn, bin + db, nv, (uint32_t)widx, wrow, fm, site, lkt, nbt);
  };


  using T = std::true_type;
  using F = std::false_type;

  auto run = [&](auto lkt, auto nbt) {
    constexpr bool TAB = decltype(lkt)::value == 3;
    if constexpr (!PROD) {
      uint64_t an = att;  // attempt of block r
      uint4 r = philox10(make_uint4((uint32_t)an, (uint32_t)(an >> 32), (uint32_t)loc, tagw), k0, k1);
      if constexpr (TAB) tab_e = tab[__umulhi(r.x, (uint32_t)N)];
      for (int64_t left = flips; left > 0;) {
        // the blocks up to a wrap of the number's lower half share a
        // PhiloxRun; near one (every 2^32 attempts) each gets its own
        ++an;
        const PhiloxRun pr((uint32_t)(an >> 32), (uint32_t)loc, tagw, k0, k1);
        const bool wraps = 0x100000000ull - (uint32_t)an < (uint64_t)left;
        const int64_t n = __ballot(wraps) ? 1 : left;
        uint32_t an_lo = (uint32_t)an;
        for (int64_t t = 0; t < n; ++t) {
          uint4 rn;
          attempt(r, rn, pr, an_lo++, lkt, nbt);
          r = rn;
          if constexpr (TAB) tab_e = tab_en;
        }
        an += (uint64_t)(n - 1);
        left -= n;
      }
    } else {
      __syncthreads();  // chunk 0 is in the buffer
      for (int64_t c = 0; c < nchunks; ++c) {
        const uint4* src = rbuf + (size_t)(c & 1) * kRngChunk * S + lane;
        const int n = (flips - c * kRngChunk) < kRngChunk ? (int)(flips - c * kRngChunk) : kRngChunk;
        uint4 r = src[0];
        if constexpr (TAB) tab_e = tab[__umulhi(r.x, (uint32_t)N)];
        for (int i = 0; i < n; ++i) {
          const uint4 rnext = src[(size_t)(i + 1 < n ? i + 1 : i) * S];
          if constexpr (TAB) tab_en = tab[__umulhi(rnext.x, (uint32_t)N)];
          uint4 unused;
          attempt(r, unused, PhiloxRun(), 0u, lkt, nbt);
          r = rnext;
          if constexpr (TAB) tab_e = tab_en;
        }
        __syncthreads();  // chunk c consumed, chunk c + 1 written
      }
    }
  };
  using L0 = std::integral_constant<int, 0>;
  using L1 = std::integral_constant<int, 1>;
  using L2 = std::integral_constant<int, 2>;
  using L3 = std::integral_constant<int, 3>;
  if (MODEL == kPotts && nib && use_tab) {
    if constexpr (MODEL == kPotts) run(L3{}, T{});
  } else if (MODEL == kPotts && nib) {
    if (pow2) run(L1{}, T{});
    else run(L0{}, T{});
  } else if (MODEL == kIsing && ROWW == 1 && L == 32) {
    if constexpr (MODEL == kIsing && ROWW == 1) run(L2{}, F{});
  } else {
    if (pow2) run(L1{}, F{});
    else run(L0{}, F{});
  }

  // ---- stage out ----
  settle(h_load);
  if (!frozen) {
    for (int i = 0; i < cnt; ++i) {
      const int b = base + i;
      const int j = pslot(b);
      const uint32_t e = eoff + (uint32_t)b;
      if (PREC == kFP64) {
        *at_off(lngw, e << 3) = get64(j);
      } else {
        *at_off(lhw, e << 2) = getf(j, 0);
        *at_off(llw, e << 2) = getf(j, 1);
      }
      const uint32_t h = word(j, 2);
      if (h_load) *at_off(Hw, e << 2) = h;
      else if (h) atomicAdd(at_off(Hw, e << 2), h);
    }
  }
  if (MODEL == kIsing) {
    for (int y = 0; y < L; ++y) {
      for (int part = 0; part < ROWW; ++part) {
        const uint32_t bits = lat[(y * ROWW + part) * S + lane];
        const int x0 = part * 32;
        const int xe = (L - x0) < 32 ? (L - x0) : 32;
        for (int b = 0; b < xe; ++b) gsp[y * L + x0 + b] = ((bits >> b) & 1) ? 1 : -1;
      }
    }
  } else if (nib) {
    for (int i = 0; i < ((N + 7) >> 3); ++i) {
      const uint32_t bits = lat[i * S + lane];
      for (int b = 0; b < 8 && 8 * i + b < N; ++b) gsp[8 * i + b] = (int8_t)((bits >> (4 * b)) & 15);
    }
  } else {
    uint32_t* dst = reinterpret_cast<uint32_t*>(gsp);
    const int nwi = (N + 3) >> 2;
    for (int i = 0; i < nwi; ++i) dst[i] = lat[i * S + lane];
  }
  P.E[g] = Ig.emin + ((W.lo + bin) << bshift);  // every energy sits on the bin grid
  P.att[g] = att + (uint64_t)flips;
}

// One kernel class per launch: the class's workgroups are entries
// [sh.wg_offset, sh.wg_offset + gridDim.x) of the table.
template <int MODEL, int PREC, int ROWW, bool PROD, bool S64, HCounts COUNTS>
__global__ __launch_bounds__(PROD ? 2 * kSweepWave : kSweepWave) void k_sweep(DevPtrs P, SweepShape sh,
                                                                                int64_t flips) {
  extern __shared__ __align__(16) unsigned char lds[];
  sweep_body<MODEL, PREC, ROWW, PROD, S64, COUNTS>(P, sh, flips, sh.wg_offset + (int)blockIdx.x, lds);
}

// Every kernel class of a batch in one launch: workgroup b runs table entry
// b with the loop of its class (all its lanes take the same branch), in
// the LDS size of the largest class.  The table order decides which
// workgroups the hardware dispatches first.
template <int PREC, bool PROD, bool S64>
__global__ __launch_bounds__(PROD ? 2 * kSweepWave : kSweepWave) void k_sweep_fused(DevPtrs P, SweepShape s0,
                                                                                      SweepShape s1,
                                                                                      SweepShape s2,
                                                                                      int64_t flips) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int wgi = (int)blockIdx.x;
  const int cls = P.wg[wgi].cls;
  if (cls == 0) sweep_body<kIsing, PREC, 1, PROD, S64, HCounts::kNone>(P, s0, flips, wgi, lds);
  else if (cls == 1) sweep_body<kIsing, PREC, 2, PROD, S64, HCounts::kNone>(P, s1, flips, wgi, lds);
  else sweep_body<kPotts, PREC, 0, PROD, S64, HCounts::kNone>(P, s2, flips, wgi, lds);
}

namespace {

using SweepFn = void (*)(DevPtrs, SweepShape, int64_t);
using FusedFn = void (*)(DevPtrs, SweepShape, SweepShape, SweepShape, int64_t);

template <int PREC, bool PROD, bool S64>
SweepFn sweep_fn(int cls, bool all) {
  constexpr HCounts kAll = HCounts::kAllLoops, kRot = HCounts::kRotationLoop, kNone = HCounts::kNone;
  if (cls == 0) return all ? k_sweep<kIsing, PREC, 1, PROD, S64, kAll> : k_sweep<kIsing, PREC, 1, PROD, S64, kRot>;
  if (cls == 1) return all ? k_sweep<kIsing, PREC, 2, PROD, S64, kAll> : k_sweep<kIsing, PREC, 2, PROD, S64, kNone>;
  return k_sweep<kPotts, PREC, 0, PROD, S64, kNone>;
}

SweepFn sweep_fn(int prec, bool prod, bool s64, int cls, bool all) {
  if (prec == kFP64)
    return prod ? (s64 ? sweep_fn<kFP64, true, true>(cls, all) : sweep_fn<kFP64, true, false>(cls, all))
                : (s64 ? sweep_fn<kFP64, false, true>(cls, all) : sweep_fn<kFP64, false, false>(cls, all));
  return prod ? (s64 ? sweep_fn<kFP32C, true, true>(cls, all) : sweep_fn<kFP32C, true, false>(cls, all))
              : (s64 ? sweep_fn<kFP32C, false, true>(cls, all) : sweep_fn<kFP32C, false, false>(cls, all));
}

FusedFn fused_fn(int prec, bool prod, bool s64) {
  if (prec == kFP64)
    return prod ? (s64 ? k_sweep_fused<kFP64, true, true> : k_sweep_fused<kFP64, true, false>)
                : (s64 ? k_sweep_fused<kFP64, false, true> : k_sweep_fused<kFP64, false, false>);
  return prod ? (s64 ? k_sweep_fused<kFP32C, true, true> : k_sweep_fused<kFP32C, true, false>)
              : (s64 ? k_sweep_fused<kFP32C, false, true> : k_sweep_fused<kFP32C, false, false>);
}

}  // namespace

hipError_t prepare_sweep_lds(size_t lds_bytes) {
  // once per device: for 48 kernels it is a tenth of the time that a context
  // of a few walkers takes to set up (80 us)
  static std::mutex mu;
  static bool done[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (done[dev]) return hipSuccess;
  for (int i = 0; i < 8; ++i) {
    const int prec = i & 1 ? kFP32C : kFP64;
    const bool prod = (i & 2) != 0, s64 = (i & 4) != 0;
    const void* fns[] = {(const void*)sweep_fn(prec, prod, s64, 0, false), (const void*)sweep_fn(prec, prod, s64, 0, true),
                         (const void*)sweep_fn(prec, prod, s64, 1, false), (const void*)sweep_fn(prec, prod, s64, 1, true),
                         (const void*)sweep_fn(prec, prod, s64, 2, false), (const void*)fused_fn(prec, prod, s64)};
    for (const void* f : fns) {
      hipFuncAttributes at;
      e = hipFuncGetAttributes(&at, f);
      if (e != hipSuccess) return e;
      if (at.sharedSizeBytes != 0) return hipErrorInvalidValue;  // dynamic LDS must start at 0
      e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
      if (e != hipSuccess) return e;
    }
  }
  done[dev] = true;
  return hipSuccess;
}

// One wavefront per compute unit that ends at once.  The wavefronts of a
// launch are dealt to the four SIMDs of a CU from where the launch before
// left off.  After a kernel of larger workgroups (the merge) that is not the
// same place in every CU, and 7 to 10 % of the SIMDs got one wavefront of the
// sweep too many and as many one too few (hardware ids read back: of 1024
// SIMDs with two wavefronts each, 98 had three and 98 one; none after this
// launch).  The sweep waits for the fullest SIMD: 1024 Ising L = 32 instances
// took 7.15 against 5.85 ms, 128 q = 10 Potts L = 20 instances in two-float
// FP32 6.44 against 5.11 ms; this launch takes 3 us.
__global__ __launch_bounds__(kSweepWave) void k_even_out() {}

hipError_t launch_even_out(int32_t n_cu, hipStream_t s) {
  hipLaunchKernelGGL(k_even_out, dim3(n_cu), dim3(kSweepWave), 0, s);
  return hipGetLastError();
}

hipError_t launch_sweep_class(const DevPtrs& P, int cls, SweepShape sh, int32_t n_wg, int64_t flips,
                              size_t lds_bytes, bool producer, bool all_counts, hipStream_t s) {
  if (n_wg <= 0) return hipSuccess;
  const SweepFn f = sweep_fn(P.prec, producer, sh.stride == kSweepWave, cls, all_counts);
  hipLaunchKernelGGL(f, dim3(n_wg), dim3(producer ? 2 * kSweepWave : kSweepWave), lds_bytes, s, P, sh, flips);
  return hipGetLastError();
}

hipError_t launch_sweep_fused(const DevPtrs& P, const SweepShape sh[3], int32_t n_wg, int64_t flips,
                              size_t lds_bytes, bool producer, hipStream_t s) {
  if (n_wg <= 0) return hipSuccess;
  bool s64 = true;  // a class that is absent has stride 0
  for (int cls = 0; cls < 3; ++cls) s64 = s64 && (sh[cls].stride == kSweepWave || sh[cls].stride == 0);
  hipLaunchKernelGGL(fused_fn(P.prec, producer, s64), dim3(n_wg), dim3(producer ? 2 * kSweepWave : kSweepWave),
                     lds_bytes, s, P, sh[0], sh[1], sh[2], flips);
  return hipGetLastError();
}

}  // namespace rewl
