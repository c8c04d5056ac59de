// REWL kernels for gfx950 (MI355X), everything except the sweep (which is
// in rewl_sweep.hip and rewl_wave.hip) and the initialisation (rewl_wave.hip).
//
// Once per cycle: k_merge_windows (flatness and the in-window average) and
// k_cycle_end (finished flags; replica exchange by Eq. 1, which swaps
// configuration indices, never lattice data).  End of run: k_join (Sec. 3
// joining + normalisation in FP64), k_jackknife and k_jackknife_rows (error
// bars from the m pieces per window) and k_thermo (Sec. 5, Eqs. 7-8).
#include <float.h>
#include <math.h>

#include <mutex>

#include "rewl_device.h"
#include "rewl_internal.h"

namespace rewl {

namespace {

// Sum of values pushed one after the other, added pairwise by levels in their
// order (an odd last element is carried): the sum of 2^l values sits in
// acc[l] as long as bit l of the number of values so far is set, like the
// digits of a binary counter.  Every thread pushes the same number of
// values, so the branches are uniform and acc stays in registers.
template <typename T, typename Add, int LEVELS>
struct PairwiseDigits {
  T acc;
  PairwiseDigits<T, Add, LEVELS - 1> up;
  __device__ __forceinline__ void push(T x, int n, Add add) {
    if (n & 1) up.push(add(acc, x), n >> 1, add);
    else acc = x;
  }
  __device__ __forceinline__ T total(T x, bool any, int n, Add add) const {
    if (n & 1) x = any ? add(acc, x) : acc;
    return up.total(x, any || (n & 1), n >> 1, add);
  }
};
template <typename T, typename Add>
struct PairwiseDigits<T, Add, 0> {
  __device__ __forceinline__ void push(T, int, Add) {}
  __device__ __forceinline__ T total(T x, bool, int, Add) const { return x; }
};
template <typename T, typename Add>
struct PairwiseSum {
  PairwiseDigits<T, Add, 7> digits;  // up to 127 values
  int n = 0;
  __device__ __forceinline__ void push(T x, Add add) { digits.push(x, n++, add); }
  __device__ __forceinline__ T total(Add add) const { return digits.total(T(), false, n, add); }
};
static_assert(kMaxWalkersPerWindow < 128, "PairwiseSum holds up to 127 values");

struct AddF64 {
  __device__ __forceinline__ double operator()(double a, double b) const { return a + b; }
};
struct TwoFloat {
  float h, l;
};
struct AddTwoFloat {
  __device__ __forceinline__ TwoFloat operator()(TwoFloat a, TwoFloat b) const {
    TwoFloat r;
    df_add(a.h, a.l, b.h, b.l, r.h, r.l);
    return r;
  }
};

// f(k, value k) for k = 0..n-1, the values loaded eight at a time so that
// their latencies overlap.
template <typename T, typename Load, typename F>
__device__ __forceinline__ void each_of(int n, Load load, F f) {
  int k = 0;
  for (; k + 8 <= n; k += 8) {
    T v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = load(k + i);
#pragma unroll
    for (int i = 0; i < 8; ++i) f(k + i, v[i]);
  }
  for (; k < n; ++k) f(k, load(k));
}

// Mean over the m walkers of the FP64 rows at x (stride nb).
__device__ __forceinline__ double mean_f64(const double* x, int64_t nb, int m) {
  PairwiseSum<double, AddF64> s;
  each_of<double>(m, [&](int k) { return x[k * nb]; }, [&](int, double v) { s.push(v, AddF64()); });
  return s.total(AddF64()) / (double)m;
}

__device__ __forceinline__ TwoFloat mean_two_float(const float* hi, const float* lo, int64_t nb, int m) {
  PairwiseSum<TwoFloat, AddTwoFloat> s;
  each_of<TwoFloat>(m, [&](int k) { return TwoFloat{hi[k * nb], lo[k * nb]}; },
                    [&](int, TwoFloat v) { s.push(v, AddTwoFloat()); });
  const TwoFloat t = s.total(AddTwoFloat());
  TwoFloat r;
  df_div_int(t.h, t.l, m, r.h, r.l);
  return r;
}

}  // namespace

// ---------------------------------------------------------------------------
// Flatness and in-window merge: one 256-thread block per window.
//
// Latency of reading the m histograms bounds it, so the loads of eight
// walkers are in flight at once, and the flatness test takes one walker per
// wavefront (a block reduction per walker took 181 us for 64 walkers of a
// 206-bin window).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_merge_windows(DevPtrs P, int32_t first) {
  __shared__ uint32_t red[8];
  __shared__ int not_ready;
  const int gw = first + (int)blockIdx.x;
  const WinDesc W = P.win[gw];
  const InstDesc& I = P.inst[W.inst];
  const WinState ws0 = P.wst[gw];
  if (P.ist[W.inst].done || P.ist[W.inst].error || ws0.frozen) return;
  const int m = I.m, nb = W.nb;
  const int tid = threadIdx.x;
  uint8_t* U = P.U + W.u_base;
  uint32_t* const H = P.H + W.lng_base;
  if (tid == 0) not_ready = 0;

  // visited union; every walker's H is read here at every check, so the
  // 2^31 guard on the histogram counters sits in this loop
  uint32_t cnt = 0;
  for (int j = tid; j < nb; j += blockDim.x) {
    uint32_t any = 0;
    each_of<uint32_t>(m, [&](int k) { return H[(int64_t)k * nb + j]; },
                      [&](int, uint32_t h) { any |= h; });
    if (any & 0x80000000u) atomicMin(&P.ist[W.inst].error, -5);
    const uint8_t u = any ? 1 : U[j];
    U[j] = u;
    cnt += u;
  }
  cnt = block_reduce(cnt, [](uint32_t a, uint32_t b) { return a + b; }, red);
  const bool one_t = I.schedule == kOneOverT;
  const bool phase_b = one_t && ws0.phase == 1;
  if (cnt == 0) return;
  if (!phase_b) {
    const int lane = tid & 63;
    volatile int* const stop = &not_ready;
    for (int k = tid >> 6; k < m && !*stop; k += (int)blockDim.x >> 6) {
      uint32_t mn = 0xFFFFFFFFu;
      uint64_t sm = 0;
      for (int j = lane; j < nb; j += 64) {
        const uint32_t h = H[(int64_t)k * nb + j];
        sm += h;
        if (U[j] && h < mn) mn = h;
      }
      mn = wave_reduce(mn, [](uint32_t a, uint32_t b) { return a < b ? a : b; });
      sm = wave_reduce(sm, [](uint64_t a, uint64_t b) { return a + b; });
      const bool fails = one_t ? mn == 0
                               : (uint64_t)I.flat_den * cnt * mn < (uint64_t)I.flat_num * sm;
      if (fails && lane == 0) *stop = 1;
    }
    __syncthreads();
    if (not_ready) return;
  }

  // new ln f: halve (phase A / halving schedule), or 1/t with t the attempts
  // per walker over the visited bins; phase A hands over to B once halving
  // would reach 1/t
  const int slot0 = I.slot_base + (gw - I.win_base) * m;
  const double tinv = (double)cnt / (double)P.att[slot0];
  double next = phase_b ? tinv : 0.5 * ws0.lnf;
  const bool to_b = one_t && !phase_b && next <= tinv;
  if (to_b) next = tinv;
  const bool freezing = next <= I.lnf_final;

  for (int j = tid; j < nb; j += blockDim.x) {
    const int64_t e0 = W.lng_base + j;
    if (P.prec == kFP64) {
      if (freezing)
        each_of<double>(m, [&](int k) { return P.lng[e0 + (int64_t)k * nb]; },
                        [&](int k, double v) { P.pieces[e0 + (int64_t)k * nb] = v; });
      const double mean = mean_f64(P.lng + e0, nb, m);
      if (!isfinite(mean)) atomicMin(&P.ist[W.inst].error, -4);
      for (int k = 0; k < m; ++k) P.lng[e0 + (int64_t)k * nb] = mean;
    } else {
      if (freezing)
        each_of<double>(m, [&](int k) { return (double)P.lhi[e0 + (int64_t)k * nb] + (double)P.llo[e0 + (int64_t)k * nb]; },
                        [&](int k, double v) { P.pieces[e0 + (int64_t)k * nb] = v; });
      const TwoFloat mean = mean_two_float(P.lhi + e0, P.llo + e0, nb, m);
      if (!isfinite(mean.h) || !isfinite(mean.l)) atomicMin(&P.ist[W.inst].error, -4);
      for (int k = 0; k < m; ++k) {
        P.lhi[e0 + (int64_t)k * nb] = mean.h;
        P.llo[e0 + (int64_t)k * nb] = mean.l;
      }
    }
    for (int k = 0; k < m; ++k) H[(int64_t)k * nb + j] = 0;
  }
  if (tid == 0) {
    WinState ws = ws0;
    if (!phase_b) {
      if (ws.stage < kMaxStages) P.stage_merge[(int64_t)gw * kMaxStages + ws.stage] = P.ist[W.inst].merges;
      ws.stage += 1;
    }
    ws.lnf = next;
    if (to_b) ws.phase = 1;
    if (freezing) ws.frozen = 1;
    P.wst[gw] = ws;
  }
}

// ---------------------------------------------------------------------------
// End of a cycle, one block per instance: the instance's merge counter and
// finished flag (merged), then a replica exchange round over its window pairs
// (exchange).  One launch in place of three: each costs 10 us or so of a small
// batch's cycle, whose sweep takes 130 us (Ising L = 8).
// Latency bounds it.  The permutations are drawn by one thread per pair (rows
// padded to an odd number of words, else the threads' accesses meet in four
// LDS banks), then one thread takes each proposal of all pairs, so an
// instance of many windows needs a large block (cycle_end_threads): a round of
// 300 windows of 8 walkers takes 6.8 us, of 64 walkers 28.9, with 256 threads
// and a wavefront per pair 48.9 and 76.9; 48 windows of 16 walkers 6.3 and 9.4.
// ---------------------------------------------------------------------------
constexpr int kPairs = 256;  // window pairs at a time; no more than threads
static_assert(kPairs <= kCycleEndThreads, "a thread draws each pair's permutation");

__global__ __launch_bounds__(kCycleEndMaxThreads) void k_cycle_end(DevPtrs P, int32_t first, int32_t merged,
                                                                   int32_t exchange) {
  __shared__ uint8_t pi[kPairs][kMaxWalkersPerWindow + 4];
  __shared__ uint32_t n_inr[kPairs], n_acc[kPairs];
  __shared__ int open;
  const int inst = first + (int)blockIdx.x;
  const int tid = threadIdx.x, nt = blockDim.x;
  const InstDesc& I = P.inst[inst];
  const InstState st = P.ist[inst];
  // thread 0 writes the counters below, in a round without window pairs with
  // no other barrier between: every wavefront has to have read them
  __syncthreads();
  if (st.done || st.error) return;
  if (merged) {
    if (tid == 0) open = 0;
    __syncthreads();
    for (int w = tid; w < I.h; w += nt)
      if (!P.wst[I.win_base + w].frozen) open = 1;
    __syncthreads();
    if (tid == 0) {
      if (!open) {
        P.ist[inst].done = 1;
        P.ist[inst].done_merge = st.merges;
      }
      P.ist[inst].merges = st.merges + 1;
    }
    if (!open) return;
  }
  if (!exchange) return;
  const uint64_t t = st.rounds;
  const int m = I.m;
  for (int base = (int)(t & 1); base + 1 < I.h; base += 2 * kPairs) {
    const int pairs = min((I.h - base) / 2, kPairs);
    if (tid < pairs) {
      const int w = base + 2 * tid;
      uint8_t* const p = pi[tid];
      for (int k = 0; k < m; ++k) p[k] = (uint8_t)k;
      uint4 r = make_uint4(0, 0, 0, 0);
      int used = 4, call = 0;
      for (int i = m - 1; i >= 1; --i) {
        if (used == 4) {
          r = draw(I, t, ((uint32_t)w << 8) | (uint32_t)call++, kTagPerm);
          used = 0;
        }
        const uint32_t rv = used == 0 ? r.x : used == 1 ? r.y : used == 2 ? r.z : r.w;
        ++used;
        const int j = (int)__umulhi(rv, (uint32_t)(i + 1));
        const uint8_t tmp = p[i];
        p[i] = p[j];
        p[j] = tmp;
      }
      n_inr[tid] = n_acc[tid] = 0;
    }
    __syncthreads();
    // proposal e: walker k of the lower window of pair q
    for (int e = tid; e < pairs * m; e += nt) {
      const int q = e / m, k = e - q * m;
      const int w = base + 2 * q, gw = I.win_base + w;
      const WinDesc W = P.win[gw], Wn = P.win[gw + 1];
      const int kn = pi[q][k];
      const int li = w * m + k, lj = (w + 1) * m + kn;
      const int si = I.slot_base + li, sj = I.slot_base + lj;
      const int32_t EX = P.E[si], EY = P.E[sj];
      const int bx = (EX - I.emin) >> I.binw_shift, by = (EY - I.emin) >> I.binw_shift;
      if (by < W.lo || by > W.hi || bx < Wn.lo || bx > Wn.hi) continue;
      atomicAdd(&n_inr[q], 1u);
      const int64_t bi = W.lng_base + (int64_t)k * W.nb;
      const int64_t bj = Wn.lng_base + (int64_t)kn * Wn.nb;
      const int ix = bx - W.lo, iy = by - W.lo, jx = bx - Wn.lo, jy = by - Wn.lo;
      const uint4 r = draw(I, t, (uint32_t)li, kTagAcc);
      bool acc;
      if (P.prec == kFP64) {
        const double lnP = (P.lng[bi + ix] - P.lng[bi + iy]) + (P.lng[bj + jy] - P.lng[bj + jx]);
        acc = accept64(u53(r.z, r.w), lnP);
      } else {
        const float x1 = (P.lhi[bi + ix] - P.lhi[bi + iy]) + (P.llo[bi + ix] - P.llo[bi + iy]);
        const float x2 = (P.lhi[bj + jy] - P.lhi[bj + jx]) + (P.llo[bj + jy] - P.llo[bj + jx]);
        acc = accept32(r.z >> 8, x1 + x2);
      }
      if (!acc) continue;
      atomicAdd(&n_acc[q], 1u);
      const int32_t ci = P.cfg[si];
      P.cfg[si] = P.cfg[sj];
      P.cfg[sj] = ci;
      P.E[si] = EY;
      P.E[sj] = EX;
    }
    __syncthreads();
    if (tid < pairs) {
      uint64_t* const xs = P.xstats + 3 * (int64_t)(I.win_base + base + 2 * tid);
      xs[0] += (uint64_t)m;
      xs[1] += (uint64_t)n_inr[tid];
      xs[2] += (uint64_t)n_acc[tid];
    }
    __syncthreads();
  }
  if (tid == 0) P.ist[inst].rounds = t + 1;
}

// ---------------------------------------------------------------------------
// Joining (Sec. 3, Eq. 2) and normalisation, FP64, one 1024-thread block per
// joined curve.
//
// Nothing here moves more than a few megabytes; what costs is latency.  So
// the representatives of all windows that fit in LDS (a chunk; all of them
// unless the windows are huge) are computed at once, every thread a bin; the
// best join bin of a window pair does not depend on the other pairs and takes
// one wavefront each; only the shifts (one addition chain over the windows)
// are serial.  Window after window in one 256-thread block with
// representatives in device memory, the join took 116 us (Ising L = 32,
// 16 windows x 8 walkers) to 290 us (q = 10 Potts L = 20, 32 x 16).
// ---------------------------------------------------------------------------
constexpr int kJoinThreads = 1024;
constexpr int kChunkWindows = 256;

struct JoinShared {
  double red[kJoinThreads / 64];
  double a[kChunkWindows], b[kChunkWindows], shift[kChunkWindows];
  int best[kChunkWindows];
};

__device__ __forceinline__ double beta5(const double* l, int j) {
  return (((l[j - 2] - 8.0 * l[j - 1]) + 8.0 * l[j + 1]) - l[j + 2]) / 12.0;
}

// Joins the window representatives into R (Sec. 3, Eq. 2): the
// first window as it is, then window w from the bin of (w-1, w) where the
// five-point slopes agree best (lowest such bin on ties; the middle of the
// overlap if no bin qualifies), shifted to continue the joined curve: a bin
// belongs to the last window whose range from its join bin up holds it.
// normalise: Ising sum g = 2^N, Potts g(E_min) = q.  Whole block.
// rep_of(W, j): representative of window W at its bin j; rep: LDS for cap of
// them, at least two windows' worth.
template <typename RepOf>
__device__ void join_windows(const DevPtrs& P, const InstDesc& I, RepOf rep_of, double* rep, int cap,
                             double* R, int normalise, bool record_joins, JoinShared& S) {
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6, waves = nt >> 6;
  const WinDesc* const win = P.win + I.win_base;
  for (int b = tid; b < I.nbins; b += nt) R[b] = -INFINITY;
  double carry = 0.0;  // shift of the chunk's first window
  for (int w0 = 0;;) {
    // windows w0..w1-1 of this chunk; the next one starts with its last
    int w1 = w0 + 1;
    while (w1 < I.h && w1 - w0 < kChunkWindows && win[w1].rep_off + win[w1].nb - win[w0].rep_off <= cap) ++w1;
    const int off0 = win[w0].rep_off;
    const int items = win[w1 - 1].rep_off + win[w1 - 1].nb - off0;
    for (int e = tid; e < items; e += nt) {
      int lo = w0, hi = w1 - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (win[mid].rep_off - off0 <= e) lo = mid;
        else hi = mid - 1;
      }
      rep[e] = rep_of(win[lo], e - (win[lo].rep_off - off0));
    }
    __syncthreads();
    for (int w = w0 + 1 + wave; w < w1; w += waves) {
      const WinDesc Wa = win[w - 1], Wb = win[w];
      const double* la = rep + (Wa.rep_off - off0);
      const double* lb = rep + (Wb.rep_off - off0);
      const uint8_t* Ua = P.U + Wa.u_base;
      const uint8_t* Ub = P.U + Wb.u_base;
      double bestd = INFINITY;
      int best = INT32_MAX;
      for (int b = Wb.lo + 2 + lane; b <= Wa.hi - 2; b += 64) {
        bool ok = true;
        for (int d = -2; d <= 2; ++d) ok = ok && Ua[b + d - Wa.lo] && Ub[b + d - Wb.lo];
        if (!ok) continue;
        const double db = fabs(beta5(la, b - Wa.lo) - beta5(lb, b - Wb.lo));
        if (db < bestd) {
          bestd = db;
          best = b;
        }
      }
      const double least = wave_reduce(bestd, [](double x, double y) { return x < y ? x : y; });
      if (bestd != least) best = INT32_MAX;
      best = wave_reduce(best, [](int x, int y) { return x < y ? x : y; });
      if (best == INT32_MAX) best = (Wb.lo + Wa.hi) / 2;
      if (lane == 0) {
        S.best[w - w0] = best;
        S.a[w - w0] = la[best - Wa.lo];
        S.b[w - w0] = lb[best - Wb.lo];
        if (record_joins) P.joins[I.win_base + w] = best;
      }
    }
    __syncthreads();
    if (tid == 0) {
      double s = carry;
      S.shift[0] = s;
      for (int w = 1; w < w1 - w0; ++w) {
        s = (S.a[w] + s) - S.b[w];
        S.shift[w] = s;
      }
    }
    __syncthreads();
    const int from = w0 == 0 ? win[0].lo : win[w0 + 1].lo;
    for (int b = from + tid; b <= win[w1 - 1].hi; b += nt) {
      int lo = w0, hi = w1 - 1;  // last window of the chunk that starts at or below b
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (win[mid].lo <= b) lo = mid;
        else hi = mid - 1;
      }
      for (int w = lo; w >= w0 && win[w].hi >= b; --w) {
        if (w == w0 && w0 > 0) break;  // the chunk before wrote these
        if (w > w0 && S.best[w - w0] > b) continue;
        const WinDesc W = win[w];
        const int j = b - W.lo;
        if (j >= 0)
          R[b] = P.U[W.u_base + j] ? (w == 0 ? rep[W.rep_off - off0 + j]
                                             : rep[W.rep_off - off0 + j] + S.shift[w - w0])
                                   : -INFINITY;
        break;
      }
    }
    carry = S.shift[w1 - 1 - w0];
    __syncthreads();
    if (w1 >= I.h) break;
    w0 = w1 - 1;
  }
  if (!normalise) return;
  double c;
  if (I.model == kIsing) {
    double mx = -INFINITY;
    for (int b = tid; b < I.nbins; b += nt) mx = fmax(mx, R[b]);
    mx = block_reduce(mx, [](double a, double b) { return a > b ? a : b; }, S.red);
    double acc = 0.0;
    for (int b = tid; b < I.nbins; b += nt)
      if (isfinite(R[b])) acc += exp(R[b] - mx);
    acc = block_reduce(acc, [](double a, double b) { return a + b; }, S.red);
    c = (double)I.N * log(2.0) - (mx + log(acc));
  } else {
    c = log((double)I.q) - R[0];
  }
  __syncthreads();
  for (int b = tid; b < I.nbins; b += nt)
    if (isfinite(R[b])) R[b] += c;
}

// Window representatives: mean over walkers, same tree as the merge.
__global__ __launch_bounds__(kJoinThreads) void k_join(DevPtrs P, int32_t instance, int32_t normalise,
                                                       int32_t cap, double* packed) {
  extern __shared__ __align__(16) double join_rep[];
  __shared__ JoinShared S;
  const InstDesc& I = P.inst[instance];
  const int m = I.m;
  double* const R = P.R + I.r_base;
  join_windows(
      P, I,
      [&](const WinDesc& W, int j) {
        const int64_t e0 = W.lng_base + j;
        if (P.prec == kFP64) return mean_f64(P.lng + e0, W.nb, m);
        const TwoFloat r = mean_two_float(P.lhi + e0, P.llo + e0, W.nb, m);
        return (double)r.h + (double)r.l;
      },
      join_rep, cap, R, normalise, true, S);
  // the curve and the join bins next to each other, for one copy to the host
  if (!packed) return;
  __syncthreads();
  for (int b = threadIdx.x; b < I.nbins; b += blockDim.x) packed[b] = R[b];
  int32_t* const joins = reinterpret_cast<int32_t*>(packed + I.nbins);
  for (int w = 1 + (int)threadIdx.x; w < I.h; w += blockDim.x) joins[w - 1] = P.joins[I.win_base + w];
}

// Jackknife over the m pieces per window (Sec. 3): block k joins and
// normalises the pairwise means of the pieces without walker k into row k of
// jk ((m + 2) x nbins doubles).  A block per k: one block for all of them
// took 25 ms at Ising L = 32, 16 windows x 64 walkers.
__global__ __launch_bounds__(kJoinThreads) void k_jackknife(DevPtrs P, int32_t instance, double* jk,
                                                            int32_t cap) {
  extern __shared__ __align__(16) double join_rep[];
  __shared__ JoinShared S;
  const InstDesc& I = P.inst[instance];
  const int m = I.m, out = blockIdx.x;
  join_windows(
      P, I,
      [&](const WinDesc& W, int j) {
        const double* const x = P.pieces + W.lng_base + j;
        const int64_t nb = W.nb;
        PairwiseSum<double, AddF64> s;
        each_of<double>(m - 1, [&](int k) { return x[(k + (k >= out ? 1 : 0)) * nb]; },
                        [&](int, double v) { s.push(v, AddF64()); });
        return s.total(AddF64()) / (double)(m - 1);
      },
      join_rep, cap, jk + (int64_t)out * I.nbins, 1, false, S);
}

// Per bin the mean of the m rows of jk and sqrt((m-1)/m * sum (R_k - mean)^2)
// into rows m and m + 1 (-inf and 0 where any row is not finite).
__global__ __launch_bounds__(64) void k_jackknife_rows(DevPtrs P, int32_t instance, double* jk) {
  const InstDesc& I = P.inst[instance];
  const int m = I.m, nbins = I.nbins;
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbins) return;
  bool fin = true;
  double acc = 0.0;
  each_of<double>(m, [&](int k) { return jk[(int64_t)k * nbins + b]; },
                  [&](int, double r) {
                    fin = fin && isfinite(r);
                    acc += r;
                  });
  double mu = -INFINITY, e = 0.0;
  if (fin) {
    mu = acc / (double)m;
    double v = 0.0;
    each_of<double>(m, [&](int k) { return jk[(int64_t)k * nbins + b]; },
                    [&](int, double r) {
                      const double d = r - mu;
                      v += d * d;
                    });
    e = sqrt((double)(m - 1) / (double)m * v);
  }
  jk[(int64_t)m * nbins + b] = mu;
  jk[(int64_t)(m + 1) * nbins + b] = e;
}

// Device memory of the allocation-free jackknife (rewl_jackknife_noalloc):
// the leave-one-out rows of one instance.  Every GPU the library runs on holds
// its own copy until the process ends; calls that overlap on one GPU share it.
static __device__ __align__(256) double scratch[kScratchDoubles];

hipError_t scratch_address(double** out) {
  static std::mutex mu;
  static double* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = static_cast<double*>(p);
  }
  *out = addr[dev];
  return hipSuccess;
}

// Canonical <E> and C_V (Sec. 5, Eqs. 7-8) from the joined ln g: one
// wavefront per temperature, the bins over its lanes (one thread per
// temperature took 403 us for 2000 temperatures of 801 bins).
__global__ __launch_bounds__(256) void k_thermo(DevPtrs P, int32_t instance, int32_t nT) {
  const int i = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
  if (i >= nT) return;
  const InstDesc& I = P.inst[instance];
  const double* lng = P.R + I.r_base;
  const double t = P.thermo[i];
  auto sum = [](double a, double b) { return a + b; };
  double mx = -INFINITY;
  for (int b = lane; b < I.nbins; b += 64) {
    if (!isfinite(lng[b])) continue;
    const double a = lng[b] - (double)(I.emin + b * I.binw) / t;
    if (a > mx) mx = a;
  }
  mx = wave_reduce(mx, [](double a, double b) { return a > b ? a : b; });
  double z = 0.0, e1 = 0.0;
  for (int b = lane; b < I.nbins; b += 64) {
    if (!isfinite(lng[b])) continue;
    const double E = (double)(I.emin + b * I.binw);
    const double wgt = exp(lng[b] - E / t - mx);
    z += wgt;
    e1 += wgt * E;
  }
  z = wave_reduce(z, sum);
  const double em = wave_reduce(e1, sum) / z;
  double v = 0.0;
  for (int b = lane; b < I.nbins; b += 64) {
    if (!isfinite(lng[b])) continue;
    const double E = (double)(I.emin + b * I.binw);
    const double wgt = exp(lng[b] - E / t - mx);
    v += wgt * (E - em) * (E - em);
  }
  v = wave_reduce(v, sum);
  if (lane == 0) {
    P.thermo[kMaxTemps + i] = em;
    P.thermo[kMaxTemps + nT + i] = (v / z) / (t * t);
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static hipError_t merge_windows(const DevPtrs& P, hipStream_t s) {
  return in_slices(P.n_win, 256, [&](int32_t first, int32_t n) {
    hipLaunchKernelGGL(k_merge_windows, dim3(n), dim3(256), 0, s, P, first);
  });
}

static hipError_t cycle_end(const DevPtrs& P, int32_t merged, int32_t exchange, hipStream_t s) {
  return in_slices(P.n_inst, P.cycle_end_threads, [&](int32_t first, int32_t n) {
    hipLaunchKernelGGL(k_cycle_end, dim3(n), dim3(P.cycle_end_threads), 0, s, P, first, merged, exchange);
  });
}

hipError_t launch_merge(const DevPtrs& P, hipStream_t s) {
  const hipError_t e = merge_windows(P, s);
  return e == hipSuccess ? cycle_end(P, 1, 0, s) : e;
}

hipError_t launch_exchange(const DevPtrs& P, hipStream_t s) { return cycle_end(P, 0, 1, s); }

hipError_t launch_merge_exchange(const DevPtrs& P, hipStream_t s) {
  const hipError_t e = merge_windows(P, s);
  return e == hipSuccess ? cycle_end(P, 1, 1, s) : e;
}

// LDS representatives of an instance: all of them up to 128 KiB, and always
// two of its largest windows (8193 bins at most, 128 KiB + 16 B).
static int join_cap(int reps, int nbmax) {
  const int most = (128 << 10) / (int)sizeof(double);
  return reps <= most ? (reps > 2 ? reps : 2) : (2 * nbmax > most ? 2 * nbmax : most);
}

hipError_t prepare_join_lds() {
  const int bytes = join_cap(1 << 30, 8193) * (int)sizeof(double);
  hipError_t e = hipFuncSetAttribute((const void*)k_join, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)k_jackknife, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  return e;
}

hipError_t launch_join(const DevPtrs& P, const InstDesc& I, int32_t reps, int32_t normalise, double* packed,
                       hipStream_t s) {
  const int cap = join_cap(reps, I.nbmax);
  hipLaunchKernelGGL(k_join, dim3(1), dim3(kJoinThreads), (size_t)cap * sizeof(double), s, P, I.inst,
                     normalise, cap, packed);
  return hipGetLastError();
}

hipError_t launch_jackknife(const DevPtrs& P, const InstDesc& I, int32_t reps, double* jk, hipStream_t s) {
  const int cap = join_cap(reps, I.nbmax);
  hipLaunchKernelGGL(k_jackknife, dim3(I.m), dim3(kJoinThreads), (size_t)cap * sizeof(double), s, P, I.inst,
                     jk, cap);
  hipLaunchKernelGGL(k_jackknife_rows, dim3((I.nbins + 63) / 64), dim3(64), 0, s, P, I.inst, jk);
  return hipGetLastError();
}

hipError_t launch_thermo(const DevPtrs& P, int32_t instance, int32_t nT, hipStream_t s) {
  hipLaunchKernelGGL(k_thermo, dim3((nT + 3) / 4), dim3(256), 0, s, P, instance, nT);
  return hipGetLastError();
}

}  // namespace rewl
