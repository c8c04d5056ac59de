// Internal layout shared by the REWL kernels and the host-side C-ABI.
//
// All simulation state lives in one caller-provided device workspace.  The
// host computes the layout once (rewl_init) and passes device pointers to the
// kernels in a DevPtrs block.  Walker slots, windows and configurations are
// numbered globally over the batch of instances; instance i owns slots
// [slot_base, slot_base + h*m) and windows [win_base, win_base + h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rewl {

constexpr int kMaxStages = 64;    // stage bookkeeping per window
constexpr int kMaxWalkersPerWindow = 64;
constexpr int kMaxL = 64;
constexpr int kSweepWave = 64;    // walkers' wavefront of a sweep workgroup
constexpr int kRngChunk = 16;     // attempts per hand-over of the RNG producer
constexpr int kSimds = 1024;
// Walkers up to which a class of a batch is swept with one wavefront per
// walker by default (larger batches with one lane per walker): cls the kernel
// class, l_max the side of its largest lattice, two_state an Ising model or
// q = 2 Potts throughout, n_wg the lane form's workgroups (of up to 64 walkers
// of one instance), n_cu the compute units.
//
// A wavefront makes an attempt in 110 to 200 ns while no SIMD holds two of them
// (1024 walkers), from there on the time grows with their number, and faster
// on small lattices, where more of 64 attempts touch each other's sites.  A
// lane takes as long however many there are, until the workgroups wait for
// one another.  ns per attempt below are lanes, wavefronts, of batches that
// have run for 30000 attempts per walker.
//
// Up to a workgroup per compute unit, each with its producer, lanes are at
// their best, and the better the smaller the lattice.  8 walkers per window:
//   Ising, walkers  4096      4608      5120      5632      6144      7168
//     L =  8     305, 302  304, 353  305, 351  304, 398  306, 405  306, 470
//     L = 16     325, 268  326, 312  325, 314  327, 356  326, 355  327, 410
//     L = 24     377, 242  375, 292  378, 293  377, 334  379, 334  377, 384
//     L = 32     377, 230  380, 270  374, 274  377, 310  377, 312  382, 357
//     L = 48     514, 223  516, 257  513, 259  515, 295  514, 292  519, 340
//   Potts
//     q = 10, L =  8  400, 354  390, 411  391, 416  393, 480
//     q = 10, L = 12  400, 333  400, 388  400, 390  400, 431
//     q =  3, L = 16  432, 302  432, 349  435, 352  434, 406
//     q = 10, L = 20  416, 284  415, 368  416, 371  416, 419
// (two-float: Ising L = 8 330, 338 at 4096; L = 32 409, 406 at 7168; q = 10
// Potts L = 20 423, 405 at 5120, 425, 458 at 5632).  With more workgroups than
// that there is no producer, and up to one workgroup per SIMD wavefronts win
// throughout: 16 walkers per instance, Ising L = 8 508, 475 at 7168, L = 24
// 621, 389; q = 10 Potts L = 8 632, 480 at 5632.
//
// Where the lane form's workgroups outnumber the SIMDs, their time grows with
// their number as well, and the limit becomes one of walkers per workgroup: 7
// (Potts 5.5).  16380 walkers, Ising of 7 per instance, L = 16 1222, 816; q =
// 10 Potts L = 20 of 5 2609, 891.  Beyond five workgroups per SIMD the lane
// form's turns on a compute unit are all full ones, and small lattices of two
// states, whose lanes are quick, are better off with fewer walkers per
// workgroup.  40960 (65536) walkers: Ising L = 8 of 4 2341, 2243 (3355, 3452),
// of 5 1965, 2183 (2805, 3338); L = 12 of 6 1939, 2008 (2769, 3093); L = 16 of
// 6 2077, 1930 (2921, 2932), of 7 1884, 1879 (2673, 2912); L = 20 of 7 2182,
// 1866 (3073, 2919); q = 2 Potts L = 8 of 5 2406, 2540 (3514, 3926); but L = 32
// of 7 2590, 1696 (3723, 2629), q = 10 Potts L = 6 of 5 3063, 2278 (4507,
// 3505).
inline int64_t wave_max_walkers(int cls, int l_max, bool two_state, int n_wg, int n_cu) {
  const int64_t most = cls == 2 ? 5632 : 7168;
  if (n_wg <= n_cu) {
    const int64_t alone = 3072 + 128 * (int64_t)l_max;
    return alone < most ? alone : most;
  }
  if (n_wg <= kSimds) return most;
  const int64_t crowded = 3328 + 192 * (int64_t)l_max;
  const int64_t per_simd = n_wg > 5 * kSimds && two_state && crowded < most ? crowded : most;
  return per_simd * n_wg / kSimds;
}
constexpr int kMaxTemps = 16384;  // rewl_thermo temperatures per call
// Allocation-free jackknife: doubles of the per-GPU device array that holds
// one instance's (m + 2) x nbins leave-one-out rows (4 MiB), and the device
// ordinals it serves.
constexpr size_t kScratchDoubles = (size_t)1 << 19;
constexpr int kMaxDevices = 64;

enum Model : int32_t { kIsing = 0, kPotts = 1 };
enum Prec : int32_t { kFP64 = 0, kFP32C = 1 };
enum Schedule : int32_t { kHalving = 0, kOneOverT = 1 };
enum Tag : uint32_t { kTagMC = 0, kTagPerm = 1, kTagAcc = 2, kTagWarm = 3, kTagInit = 4 };

struct InstDesc {
  int32_t model, L, N, q;
  int32_t binw, binw_shift, emin, nbins;
  int32_t h, m, W, inst;
  int32_t slot_base, win_base, flat_num, flat_den;
  int32_t npad;          // bytes per stored configuration (multiple of 16)
  int32_t nbmax;         // largest window of this instance, bins
  int32_t r_base;        // offset of this instance's joined ln g in the R / out arrays
  int32_t rep_base;      // window bins of the instances before (read by no kernel, part of saved states)
  int64_t spin_base;     // byte offset of configuration 0 of this instance
  double lnf_final;
  uint32_t key0, key1;
  int32_t schedule;      // kHalving or kOneOverT
};

struct WinDesc {
  int32_t lo, hi, nb, inst;
  int64_t lng_base;      // element offset of walker k = 0, bin lo of this window
  int32_t u_base;        // offset of the visited mask
  int32_t rep_off;       // window bins of the windows before, over the batch
};

struct WinState {
  double lnf;
  int32_t stage, frozen;
  int32_t phase;         // 1/t schedule: 0 = halving phase, 1 = ln f = 1/t
  int32_t pad;
};

struct InstState {
  int32_t done, error;
  int64_t done_merge;
  int64_t merges;
  uint64_t rounds;
};

// A sweep workgroup: up to 64 consecutive walker slots of one instance, and
// the kernel class of that instance (0 Ising L <= 32, 1 Ising L <= 64, 2 Potts).
struct WgDesc {
  int32_t inst, slot_first, count, cls;
};

struct DevPtrs {
  const InstDesc* inst;
  const WinDesc* win;
  const WgDesc* wg;
  InstState* ist;
  WinState* wst;
  int64_t* stage_merge;      // [windows][kMaxStages]
  uint64_t* xstats;          // [windows][3]: tries, in-range, accepts
  int32_t* cfg;              // [slots] configuration carried by each slot
  int32_t* E;                // [slots] energy of that configuration
  uint64_t* att;             // [slots] MC attempt counter
  uint64_t* watt;            // [slots] warm-up attempt counter
  int8_t* spins;             // configurations, npad bytes each
  double* lng;               // FP64 ln g, [sum over windows of m*nb]
  float* lhi;                // FP32C two-float ln g
  float* llo;
  uint32_t* H;               // histograms, same indexing as ln g
  double* pieces;            // ln g of every walker just before its window froze
  uint8_t* U;                // visited-union masks per window
  double* R;                 // joined ln g per instance
  double* thermo;            // 3 kMaxTemps: T, then from kMaxTemps on nT <E> and nT C_V
  int32_t* joins;            // [windows] join bin of (w-1, w)
  double* jk;                // jackknife scratch: (m + 2) x nbins of one instance
  int32_t n_inst, n_win, n_slots, n_wg;
  int32_t prec;
  int32_t cycle_end_threads;
};

// Threads of a block of the cycle end, from the most exchange proposals a
// round of one of the batch's instances has: enough that each takes about one,
// but no more than a batch of many small instances needs.
constexpr int kCycleEndThreads = 256, kCycleEndMaxThreads = 1024;
inline int cycle_end_threads(int64_t proposals) {
  int t = kCycleEndThreads;
  while (t < kCycleEndMaxThreads && t < proposals) t *= 2;
  return t;
}

// Launch shape of one sweep kernel class (Ising L <= 32, Ising L <= 64,
// Potts): lanes per LDS row (walkers per workgroup), 32-bit lattice words
// per lane, ln g / H page rows per lane, first workgroup in the table, for
// Potts whether spins are kept as 4-bit nibbles (else bytes), and whether
// the workgroup keeps a table of every site's neighbours in LDS (8 bytes
// per site after the page; nibble lattices).
struct SweepShape {
  int32_t stride, nw, page, wg_offset, nib, tab;
};

// f(first, n) launches workgroups first to first + n - 1 of `total`, each of
// `threads` threads.  A launch's threads have to stay below 2^32: beyond that
// their number wraps round and the rest is left out without an error, which a
// wavefront per walker reaches with 2^26 walkers.
template <typename F>
hipError_t in_slices(int32_t total, int32_t threads, F f) {
  const int32_t most = (int32_t)(((int64_t)1 << 31) / threads);
  hipError_t e = hipSuccess;
  for (int64_t first = 0; first < total && e == hipSuccess; first += most) {
    f((int32_t)first, total - first < most ? (int32_t)(total - first) : most);
    e = hipGetLastError();
  }
  return e;
}

// Launchers (kernels TU).  All enqueue on `s` and return the launch status.
// lat_bytes: spins of the batch's largest lattice, rounded up to 16.
hipError_t launch_init(const DevPtrs& P, int32_t lat_bytes, hipStream_t s);
// One sweep kernel class: 0 = Ising L <= 32, 1 = Ising 32 < L <= 64,
// 2 = Potts; n_wg workgroups starting at sh.wg_offset of the table;
// producer: a second wavefront per workgroup computes the random numbers;
// all_counts: h_in_page (else kRotationLoop for class 0, kNone for the others).
hipError_t launch_sweep_class(const DevPtrs& P, int cls, SweepShape sh, int32_t n_wg, int64_t flips,
                              size_t lds_bytes, bool producer, bool all_counts, hipStream_t s);
// Which lane loops keep whole counts of H in the page, loaded and stored with
// their ln g; the others keep increments, added to H by an atomic when a bin
// leaves.  The load is one more per entering bin; the atomic takes longer to
// leave and fetches its line.  ns per attempt, increments against counts
// (batches that have run for 30000 attempts per walker, FP64, two-float in
// brackets):
//   the rotation loop (Ising L = 32) gains at every size and page: 8192 walkers
//     384, 379 (410, 405), 24576 443, 431 (476, 470), 65536 531, 507 (555,
//     549), 131072 1321, 1227 (1430, 1368);
//   the other Ising loops gain where the traffic binds, with a workgroup per
//     SIMD and more ln g and H (12 bytes per bin) than stay in the 256 MB
//     last-level cache: L = 24, 331 MB 1053, 988 (1178, 1135); L = 31, 1135 MB
//     1215, 1118 (1326, 1229); L = 36, 431 MB 1992, 1939 (2082, 1981); L = 50,
//     415 MB 809, 802 (855, 820); L = 64, 679 MB 1493, 1454 (1533, 1478);
//     below that they lose or gain little: L = 16, 148 MB 717, 727 (767, 815);
//     L = 24, 248 MB 853, 854 (888, 901); L = 40, 266 MB 655, 667 (704, 683);
//     L = 31 with 768 workgroups, 567 MB 536, 539 (569, 577); L = 20, 8192
//     walkers 343, 340 (390, 363), 16384 348, 356 (393, 378);
//   Potts, whose pages shift most often, loses (L = 20, q = 10, 65536 walkers
//     684, 695; two-float, 131072 1508, 1540; L = 32, 340 MB 1604, 1619), and
//     so does the fused launch of 64 uneven instances (0.5 %).
enum class HCounts : int32_t { kNone, kRotationLoop, kAllLoops };
// kAllLoops for a class of n_wg workgroups in a batch of lng_elems bins.
inline bool h_in_page(int cls, int n_wg, int64_t lng_elems) {
  return cls != 2 && n_wg >= kSimds && 12 * lng_elems > (int64_t)288 << 20;
}
// Deals the wavefronts of the next launch evenly to the SIMDs of every
// compute unit; before a sweep of at least as many workgroups as there are.
hipError_t launch_even_out(int32_t n_cu, hipStream_t s);
// Shorter sweeps (attempts per walker) do without: they take less than 70 us.
constexpr int64_t kEvenOutFlips = 512;
// One wavefront per walker: n_wg entries of the table from wg_offset, each of
// one walker of class cls; lat_bytes: spins of the class's largest lattice,
// rounded up to 16; l_min: side of its smallest.
hipError_t launch_sweep_wave(const DevPtrs& P, int cls, int32_t wg_offset, int32_t n_wg,
                             int32_t lat_bytes, int32_t l_min, int64_t flips, hipStream_t s);
// Whether such a workgroup keeps a 64-bit lane mask per site (else a count in a
// byte), and its LDS.  The masks say which accepted moves concern a later
// attempt, the counts only which concern another; they are taken while all
// n_wg workgroups stay resident with them (17 per compute unit at 1024
// sites).  At L = 2 right and left neighbour are one site, which a mask
// cannot say for Ising.
inline bool wave_masks(int cls, int32_t lat_bytes, int32_t l_min, int32_t n_wg) {
  return (cls == 2 || l_min >= 3) && (lat_bytes <= 256 || (lat_bytes <= 1024 && n_wg <= 4096));
}
inline int32_t wave_lds_bytes(int cls, int32_t lat_bytes, int32_t l_min, int32_t n_wg) {
  return (wave_masks(cls, lat_bytes, l_min, n_wg) ? 9 : 2) * lat_bytes;
}
// Every class in one launch (k_sweep_fused): n_wg entries of the table from
// 0, class shapes sh[0..2], lds_bytes of the largest class.
hipError_t launch_sweep_fused(const DevPtrs& P, const SweepShape sh[3], int32_t n_wg, int64_t flips,
                              size_t lds_bytes, bool producer, hipStream_t s);
hipError_t launch_merge(const DevPtrs& P, hipStream_t s);
hipError_t launch_exchange(const DevPtrs& P, hipStream_t s);
// The end of a cycle: launch_merge and launch_exchange in one launch less.
hipError_t launch_merge_exchange(const DevPtrs& P, hipStream_t s);
// reps: sum of the instance's window sizes; packed: null, or room for the
// joined curve (nbins doubles) followed by the h - 1 join bins (int32).
hipError_t launch_join(const DevPtrs& P, const InstDesc& I, int32_t reps, int32_t normalise, double* packed,
                       hipStream_t s);
// Leave-one-out joins of an instance's frozen pieces, rows 0..m-1 of jk
// ((m + 2) x nbins); mean and error land in rows m and m + 1.
hipError_t launch_jackknife(const DevPtrs& P, const InstDesc& I, int32_t reps, double* jk, hipStream_t s);
hipError_t prepare_join_lds();
// Device address, on the current GPU, of the allocation-free jackknife's
// kScratchDoubles-double array (looked up once per device).
hipError_t scratch_address(double** out);
hipError_t launch_thermo(const DevPtrs& P, int32_t instance, int32_t nT, hipStream_t s);
hipError_t prepare_sweep_lds(size_t lds_bytes);

}  // namespace rewl
