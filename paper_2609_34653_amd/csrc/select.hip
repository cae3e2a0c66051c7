// Budgeted whole-unit selection, one workgroup per segment.  Up to 128 units (512 where there are
// many segments): a single wave (select_small_kernel); beyond: 1024 threads (select_kernel).
//
// Groups (paper: must-keep, recent-context, selected-history):
//   protected  units holding a system token (all kept; over budget -> OMNITIDE_E_BUDGET)
//   recent     newest live non-system units whose suffix total fits min(R, B - T_sys); because
//              lengths are positive the suffix total grows monotonically, so "walk newest to
//              oldest and stop at the first misfit" is the set {u : suffix(u) <= cap}
//   selected   remaining live units in descending order of the 64-bit key (score << 13 | id),
//              kept while the inclusive prefix of their lengths fits; the prefix sum grows
//              monotonically, so "stop at the first misfit" is a threshold on the key, found by
//              a radix select without sorting.
#include "common.h"
#include "kernels.h"

namespace omnitide {
namespace {

constexpr int kSelThreads = 1024;
constexpr int kMaxUnits = OMNITIDE_MAX_UNITS;
constexpr int kIdBits = 13;   // 2^13 = kMaxUnits
// Scores below 2^51 fit the 64-bit ranking key (score << kIdBits | id) with one bit to spare.
// omnitide_score_units never exceeds 2^43: a slot contributes at most 4,096 elements x 2^21 x
// a weight of 2^10.
constexpr int kScoreBits = 51;

// floor(n / d) for d >= 1.  Below 2^53 the dividend is exact in double: the correctly rounded
// quotient is at most one above the floor (when the true quotient lies just below an integer),
// which the remainder's sign corrects.  Larger dividends take the integer division.
__device__ inline uint64_t udiv64(uint64_t n, uint32_t d) {
  if (n < (1ull << 53)) {
    uint64_t q = static_cast<uint64_t>(static_cast<double>(n) / static_cast<double>(d));
    if (static_cast<int64_t>(n - q * d) < 0) --q;
    return q;
  }
  return n / d;
}

// Beyond 128 units: the budget cut by the same radix select as the single-wave variant below,
// over a workgroup.  Thread t owns units [t*per, (t+1)*per); its keys stay in registers.  Digits
// are 12 bits (4,096 buckets; thread t scans buckets 4095 - 4t .. 4092 - 4t, highest first) and
// start at the highest bit in which two candidates differ, so the first pass already spreads
// the candidates over most buckets and two or three passes end the search.  A bucket holds its
// candidates' token total (low 44 bits) and their number (high 20) in one 64-bit LDS atomic.
// Bound by latency (barriers and LDS round trips) and by the one CU's instruction issue, so the
// units per thread are a template argument (1, 2, 4 or 8).  A full bitonic sort of the keys in LDS
// (78 barrier-separated steps at 4,096) took 74.5 us at 3,880 units; this takes 11.8 us, 13.5 with
// eight units' code for every thread.
constexpr int kWideDigitBits = 12;
constexpr int kWideBuckets = 1 << kWideDigitBits;
constexpr int kWidePer = kWideBuckets / kSelThreads;
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kCountShift = 44;
static_assert(kSelWaves == 16, "wave totals are read by lanes 0..15");
static_assert(kMaxUnits < (1 << (64 - kCountShift)), "a bucket's count field");

// Bitwise OR over the wave, the same in every lane (the DPP steps of the wave scans).
__device__ inline uint32_t wave_or_u32(uint32_t v) {
  int x = static_cast<int>(v);
  x |= dpp_move<kDppRowShr1, 0xf>(0, x);
  x |= dpp_move<kDppRowShr2, 0xf>(0, x);
  x |= dpp_move<kDppRowShr4, 0xf>(0, x);
  x |= dpp_move<kDppRowShr8, 0xf>(0, x);
  x |= dpp_move<kDppRowBcast15, 0xa>(0, x);
  x |= dpp_move<kDppRowBcast31, 0xc>(0, x);
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(x, kWave - 1));
}
__device__ inline uint64_t wave_or_u64(uint64_t v) {
  return (static_cast<uint64_t>(wave_or_u32(static_cast<uint32_t>(v >> 32))) << 32) |
         wave_or_u32(static_cast<uint32_t>(v));
}

template <int PER>
__global__ __launch_bounds__(kSelThreads) void select_kernel(
    const uint64_t* __restrict__ wsum_g, const int32_t* __restrict__ len_g,
    const int32_t* __restrict__ first_g, const int32_t* __restrict__ last_g,
    const uint32_t* __restrict__ flags_g, int n_units, int budget, int recent,
    uint64_t* __restrict__ score_g, uint8_t* __restrict__ keep_g,
    int32_t* __restrict__ kept_tokens_g, int32_t* __restrict__ status) {
  __shared__ __attribute__((aligned(16))) unsigned long long hist[kWideBuckets];
  __shared__ int32_t w_max[kSelWaves], w_elig[kSelWaves], w_sys[kSelWaves], w_err[kSelWaves];
  __shared__ int32_t w_rec[kSelWaves], w_bad[kSelWaves], w_tot[kSelWaves];
  __shared__ uint64_t w_or[kSelWaves], w_zero[kSelWaves];
  __shared__ int32_t s_cut, s_taken, s_left, s_all;

  const int seg = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int U = n_units;
  const int per = (U + kSelThreads - 1) / kSelThreads;
  const int u0 = tid * per;
  const size_t base = static_cast<size_t>(seg) * U;

  int ln[PER], fs[PER], ls[PER];
  uint32_t fl[PER];
  uint64_t ws[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {           // all loads first: one memory round trip
    ln[i] = fs[i] = ls[i] = 0;
    fl[i] = 0;
    ws[i] = 0;
    if (i < per) {                           // uniform
      const int u = min(u0 + i, U - 1);
      ln[i] = len_g[base + u];
      fs[i] = first_g[base + u];
      ls[i] = last_g[base + u];
      fl[i] = flags_g[base + u];
      ws[i] = wsum_g[base + u];
    }
  }
#pragma unroll
  for (int j = 0; j < kWidePer; ++j) hist[kWidePer * tid + j] = 0;
  bool sys[PER];
  uint64_t key[PER];
  bool bad = false, big = false;
  int my_max_first = -1, my_sys = 0, my_elig = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int u = u0 + i;
    const bool mine = i < per && u < U;
    if (!mine || ln[i] <= 0) ln[i] = 0;
    const bool live = ln[i] > 0;
    sys[i] = live && (fl[i] & 1u) != 0;
    const uint64_t sc = live ? udiv64(ws[i], static_cast<uint32_t>(ln[i])) : 0;
    bad |= live && (ls[i] - fs[i] + 1) != ln[i];
    big |= (sc >> kScoreBits) != 0;          // the ranking key holds kScoreBits of score
    if (live) my_max_first = max(my_max_first, fs[i]);
    my_sys += sys[i] ? ln[i] : 0;
    my_elig += (live && !sys[i]) ? ln[i] : 0;
    if (mine) score_g[base + u] = sc;
    key[i] = (sc << kIdBits) | static_cast<uint64_t>(mine ? u : 0);
  }
  // wave totals, then every wave combines the 16 waves' (lane l < 16 holds wave l's)
  const int inc_max = wave_scan_max_i32(my_max_first, -1);
  const int inc_elig = wave_scan_add_i32(my_elig);
  const int sum_sys = static_cast<int>(wave_sum_u32(static_cast<uint32_t>(my_sys)));
  const int err = (__any(bad) ? 1 : 0) | (__any(big) ? 2 : 0);
  if (lane == kWave - 1) {
    w_max[wave] = inc_max;
    w_elig[wave] = inc_elig;
    w_sys[wave] = sum_sys;
    w_err[wave] = err;
  }
  __syncthreads();
  const bool has = lane < kSelWaves;
  const int all_max = has && lane < wave ? w_max[lane & 15] : -1;
  const int all_elig = has ? w_elig[lane & 15] : 0;
  const int all_err = has ? w_err[lane & 15] : 0;
  const int max_before = wave_max_i32(all_max);
  const int elig_before_wave =
      static_cast<int>(wave_sum_u32(static_cast<uint32_t>(lane < wave ? all_elig : 0)));
  const int elig_total = static_cast<int>(wave_sum_u32(static_cast<uint32_t>(all_elig)));
  const int t_sys =
      static_cast<int>(wave_sum_u32(static_cast<uint32_t>(has ? w_sys[lane & 15] : 0)));
  bool any_bad = __any((all_err & 1) != 0);
  const bool any_big = __any((all_err & 2) != 0);

  // live units must appear in unit order: each first slot exceeds every earlier live unit's
  int run = max(max_before, dpp_move<kDppWaveShr1, 0xf>(-1, inc_max));
  bad = false;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (ln[i] > 0) {
      bad |= fs[i] <= run;
      run = max(run, fs[i]);
    }
  }
  // recent window: suffix sums of eligible (live, non-system) lengths
  const int cap_rec = min(recent, budget - t_sys);
  int suffix = elig_total - elig_before_wave - inc_elig;   // eligible tokens in later threads
  bool rec[PER];
  int my_rec = 0;
#pragma unroll
  for (int i = PER - 1; i >= 0; --i) {
    rec[i] = false;
    if (ln[i] > 0 && !sys[i]) {
      suffix += ln[i];
      rec[i] = suffix <= cap_rec;
      my_rec += rec[i] ? ln[i] : 0;
    }
  }
  // candidates (state: 1 active, 2 kept, 0 dropped), and the bits in which their keys differ
  int state[PER];
  uint64_t k_or = 0, k_zero = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    state[i] = (ln[i] > 0 && !sys[i] && !rec[i]) ? 1 : 0;
    k_or |= state[i] ? key[i] : 0;
    k_zero |= state[i] ? ~key[i] : 0;
  }
  k_or = wave_or_u64(k_or);
  k_zero = wave_or_u64(k_zero);
  const int sum_rec = static_cast<int>(wave_sum_u32(static_cast<uint32_t>(my_rec)));
  const bool wave_bad = __any(bad);
  if (lane == 0) {
    w_or[wave] = k_or;
    w_zero[wave] = k_zero;
    w_rec[wave] = sum_rec;
    w_bad[wave] = wave_bad ? 1 : 0;
  }
  __syncthreads();
  any_bad |= __any(has && w_bad[lane & 15] != 0);
  if (any_bad || any_big || t_sys > budget) {
    for (int u = tid; u < U; u += kSelThreads) keep_g[base + u] = 0;
    if (tid == 0) {
      kept_tokens_g[seg] = 0;
      set_status(status, any_bad   ? OMNITIDE_E_TAGS
                         : any_big ? OMNITIDE_E_RANGE
                                   : OMNITIDE_E_BUDGET);
    }
    return;
  }
  const int t_rec =
      static_cast<int>(wave_sum_u32(static_cast<uint32_t>(has ? w_rec[lane & 15] : 0)));
  const uint64_t differ = wave_or_u64(has ? w_or[lane & 15] : 0) &
                          wave_or_u64(has ? w_zero[lane & 15] : 0);
  const int cap_sel = budget - t_sys - t_rec;

  // Radix select of the first misfit in (score desc, id desc) order.  All active keys agree above
  // bit hi.  With one candidate (or none) no bits differ and one digit of width 1 decides.
  int taken = 0;                                    // tokens kept by the search so far
  int hi = max(64 - __builtin_clzll(differ | 1), 1);
  while (true) {
    const int lo = max(hi - kWideDigitBits, 0);
    const uint64_t mask = (1ull << (hi - lo)) - 1;
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (state[i] == 1)
        atomicAdd(&hist[(key[i] >> lo) & mask],
                  (1ull << kCountShift) + static_cast<uint32_t>(ln[i]));
    __syncthreads();
    // buckets top + kWidePer - 1 .. top, read highest first and cleared for the next pass
    const int top = kWideBuckets - kWidePer * (tid + 1);
    uint64_t hv[kWidePer];
    int hsum = 0;
#pragma unroll
    for (int j = 0; j < kWidePer; ++j) {
      hv[j] = hist[top + kWidePer - 1 - j];
      hsum += static_cast<int>(hv[j] & ((1ull << kCountShift) - 1));
    }
#pragma unroll
    for (int j = 0; j < kWidePer; ++j) hist[top + j] = 0;
    const int inc = wave_scan_add_i32(hsum);
    if (lane == kWave - 1) w_tot[wave] = inc;
    if (tid == 0) s_cut = -1;
    __syncthreads();
    const int before_wave = static_cast<int>(
        wave_sum_u32(static_cast<uint32_t>(has && lane < wave ? w_tot[lane & 15] : 0)));
    int acc = taken + before_wave + inc - hsum;
    if (acc <= cap_sel && acc + hsum > cap_sel) {   // the first misfit is in this thread's range
      bool open = true;
#pragma unroll
      for (int j = 0; j < kWidePer; ++j) {
        const int h = static_cast<int>(hv[j] & ((1ull << kCountShift) - 1));
        if (open && acc + h > cap_sel) {
          s_cut = top + kWidePer - 1 - j;
          s_taken = acc;
          s_left = static_cast<int>(hv[j] >> kCountShift);
          open = false;
        }
        acc += open ? h : 0;
      }
    } else if (tid == kSelThreads - 1) {
      s_all = acc + hsum;
    }
    __syncthreads();
    const int cut = s_cut;
    if (cut < 0) {                                  // every active candidate fits
      taken = s_all;
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (state[i] == 1) state[i] = 2;
      break;
    }
    taken = s_taken;
    const bool last = s_left <= 1 || lo == 0;       // one key left in the bucket: the misfit
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (state[i] == 1) {
        const int dg = static_cast<int>((key[i] >> lo) & mask);
        state[i] = dg > cut ? 2 : (dg < cut || last) ? 0 : 1;
      }
    }
    if (last) break;
    hi = lo;
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int u = u0 + i;
    if (i < per && u < U) keep_g[base + u] = (sys[i] || rec[i] || state[i] == 2) ? 1 : 0;
  }
  if (tid == 0) kept_tokens_g[seg] = t_sys + t_rec + taken;
}

// Single-wave variant for U <= 512 (every lane owns PER consecutive units): the same plan with
// wave-level scans (no workgroup barriers) and, instead of a full sort, an MSD radix select of
// the cut.  The walk "rank order, stop at the first misfit" keeps exactly the candidates whose
// key exceeds the first misfit's key; the misfit is found digit by digit: a histogram of
// candidate lengths over the next key bits (LDS atomics) and a scan in descending digit order
// locate the bucket where the running total first exceeds the cap; higher buckets are kept,
// lower ones dropped, and the search continues inside that bucket until it holds one key.
// Digits are 10 bits wide (1,024 buckets), so a 50-bit key takes five passes.
constexpr int kDigitBits = 10;                       // radix-select digit
constexpr int kBuckets = 1 << kDigitBits;
constexpr int kBucketsPerLane = kBuckets / kWave;


__device__ inline int wave_exclusive_sum(int v, int* total) {
  const int inc = wave_inclusive_scan(v);
  *total = __shfl(inc, kWave - 1, kWave);
  return inc - v;
}

template <int PER>
__global__ __launch_bounds__(kWave) void select_small_kernel(
    const uint64_t* __restrict__ wsum_g, const int32_t* __restrict__ len_g,
    const int32_t* __restrict__ first_g, const int32_t* __restrict__ last_g,
    const uint32_t* __restrict__ flags_g, int n_units, int budget, int recent,
    uint64_t* __restrict__ score_g, uint8_t* __restrict__ keep_g,
    int32_t* __restrict__ kept_tokens_g, int32_t* __restrict__ status) {
  __shared__ __attribute__((aligned(16))) int32_t hist[kBuckets];
  const int seg = blockIdx.x;
  const int lane = threadIdx.x;
  const int U = n_units;
  const int u0 = lane * PER;
  const size_t base = static_cast<size_t>(seg) * U;

  int ln[PER], fs[PER], ls[PER];
  uint32_t fl[PER];
  uint64_t ws[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {      // all loads first: one memory round trip
    const int u = min(u0 + i, U - 1);
    ln[i] = len_g[base + u];
    fs[i] = first_g[base + u];
    ls[i] = last_g[base + u];
    fl[i] = flags_g[base + u];
    ws[i] = wsum_g[base + u];
  }
  bool sys[PER];
  uint64_t key[PER];
  bool bad = false, big = false;
  int my_max_first = -1;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int u = u0 + i;
    if (u >= U || ln[i] <= 0) ln[i] = 0;
    const bool live = ln[i] > 0;
    sys[i] = live && (fl[i] & 1u) != 0;
    const uint64_t sc = live ? udiv64(ws[i], static_cast<uint32_t>(ln[i])) : 0;
    bad |= live && (ls[i] - fs[i] + 1) != ln[i];
    big |= (sc >> kScoreBits) != 0;
    if (live) my_max_first = max(my_max_first, fs[i]);
    if (u < U) score_g[base + u] = sc;
    key[i] = (sc << kIdBits) | static_cast<uint64_t>(u);
  }
  // unit order: every live unit's first slot exceeds all earlier live units' first slots
  int run = wave_exclusive_max_i32(my_max_first, -1);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (ln[i] > 0) {
      bad |= fs[i] <= run;
      run = max(run, fs[i]);
    }
  }
  int my_sys = 0, my_elig = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    my_sys += sys[i] ? ln[i] : 0;
    my_elig += (ln[i] > 0 && !sys[i]) ? ln[i] : 0;
  }
  int t_sys, elig_total;
  wave_exclusive_sum(my_sys, &t_sys);
  const int elig_before = wave_exclusive_sum(my_elig, &elig_total);
  const bool any_bad = __any(bad);
  const bool any_big = __any(big);
  if (any_bad || any_big || t_sys > budget) {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (u0 + i < U) keep_g[base + u0 + i] = 0;
    if (lane == 0) {
      kept_tokens_g[seg] = 0;
      set_status(status, any_bad   ? OMNITIDE_E_TAGS
                         : any_big ? OMNITIDE_E_RANGE
                                   : OMNITIDE_E_BUDGET);
    }
    return;
  }
  // recent window: suffix sums of eligible lengths, newest unit first
  const int cap_rec = min(recent, budget - t_sys);
  int suffix = elig_total - elig_before - my_elig;
  bool rec[PER];
  int my_rec = 0;
#pragma unroll
  for (int i = PER - 1; i >= 0; --i) {
    rec[i] = false;
    if (ln[i] > 0 && !sys[i]) {
      suffix += ln[i];
      rec[i] = suffix <= cap_rec;
      my_rec += rec[i] ? ln[i] : 0;
    }
  }
  int t_rec;
  wave_exclusive_sum(my_rec, &t_rec);
  const int cap_sel = budget - t_sys - t_rec;

  // radix select of the first misfit among candidates (state: 1 active, 2 kept, 0 dropped)
  int state[PER];
  uint64_t kmax = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    state[i] = (ln[i] > 0 && !sys[i] && !rec[i]) ? 1 : 0;
    if (state[i]) kmax = max(kmax, key[i]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) kmax = max(kmax, __shfl_xor(kmax, off, kWave));
  int taken = 0;                                   // tokens already kept by the search
  int hi = 64 - __builtin_clzll(kmax | 1);         // key bits in use
  while (hi > 0) {
    const int lo = max(hi - kDigitBits, 0);
    const uint64_t mask = (1ull << (hi - lo)) - 1;
#pragma unroll
    for (int j = 0; j < kBucketsPerLane / 4; ++j)
      *reinterpret_cast<int4*>(&hist[kBucketsPerLane * lane + 4 * j]) = make_int4(0, 0, 0, 0);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (state[i] == 1) atomicAdd(&hist[(key[i] >> lo) & mask], ln[i]);
    __syncthreads();
    // descending digit order: lane owns digits kBuckets-1 - kBucketsPerLane*lane - j
    int hv[kBucketsPerLane], hsum = 0;
    {
      const int top = kBuckets - kBucketsPerLane * (lane + 1);   // lowest digit of the lane
#pragma unroll
      for (int j = 0; j < kBucketsPerLane / 4; ++j) {
        const int4 w = *reinterpret_cast<const int4*>(&hist[top + 4 * j]);
        hv[kBucketsPerLane - 1 - 4 * j] = w.x;
        hv[kBucketsPerLane - 2 - 4 * j] = w.y;
        hv[kBucketsPerLane - 3 - 4 * j] = w.z;
        hv[kBucketsPerLane - 4 - 4 * j] = w.w;
      }
#pragma unroll
      for (int j = 0; j < kBucketsPerLane; ++j) hsum += hv[j];
    }
    int tot;
    int acc = taken + wave_exclusive_sum(hsum, &tot);
    (void)tot;
    int cut = -1;                                  // first digit whose bucket overflows
#pragma unroll
    for (int j = 0; j < kBucketsPerLane; ++j) {
      if (cut < 0 && acc + hv[j] > cap_sel) cut = kBuckets - 1 - kBucketsPerLane * lane - j;
      acc += hv[j];
    }
    const uint64_t cut_lanes = __ballot(cut >= 0);
    if (cut_lanes == 0) {                          // every active candidate fits
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (state[i] == 1) state[i] = 2;
      break;
    }
    const int d_cut = __shfl(cut, __builtin_ctzll(cut_lanes), kWave);
    int my_above = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (state[i] == 1) {
        const int dg = static_cast<int>((key[i] >> lo) & mask);
        if (dg > d_cut) {
          state[i] = 2;
          my_above += ln[i];
        } else if (dg < d_cut) {
          state[i] = 0;
        }
      }
    }
    int above, my_left = 0, left;
#pragma unroll
    for (int i = 0; i < PER; ++i) my_left += state[i] == 1 ? 1 : 0;
    wave_exclusive_sum(my_above, &above);
    wave_exclusive_sum(my_left, &left);
    taken += above;
    hi = lo;
    __syncthreads();
    if (hi == 0 || left <= 1) {                    // one key left in the bucket: the misfit
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (state[i] == 1) state[i] = 0;
      break;
    }
  }
  int my_sel = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int u = u0 + i;
    if (u < U) {
      const bool kp = sys[i] || rec[i] || state[i] == 2;
      keep_g[base + u] = kp ? 1 : 0;
      my_sel += state[i] == 2 ? ln[i] : 0;
    }
  }
  int t_sel;
  wave_exclusive_sum(my_sel, &t_sel);
  if (lane == 0) kept_tokens_g[seg] = t_sys + t_rec + t_sel;
}

}  // namespace

hipError_t launch_select(const uint64_t* wsum, const int32_t* len, const int32_t* first,
                         const int32_t* last, const uint32_t* flags, int n_seg, int n_units,
                         int budget, int recent, uint64_t* score, uint8_t* keep,
                         int32_t* kept_tokens, int32_t* status, hipStream_t stream) {
  // One wave up to 128 units, a workgroup beyond: the plan of a wave is bound by its instructions,
  // which grow with the units per lane (by graph replay: 37 units 3.1 us with one per lane, 6.7 with
  // eight; 128 units 3.4 with two; 256 units 5.2 with four and 4.5 by the workgroup, 474 units 8.3
  // with eight and 4.6).  One workgroup's 16 waves have a CU to themselves up to 256 segments and two
  // share it up to 512; with more the segments' waves are what fills the chip, and one each is
  // enough (200 units, 384 segments: 8.1 us by the workgroup, 6.2 by a wave with four per lane; 358
  // units, 512 segments: 8.8 and 10.4, 768: 12.1 and 11.2, 2,048: 26.8 and 17.1).
#define OMNITIDE_SELECT_SMALL(PER)                                                              \
  if (n_units <= PER * kWave && (PER <= 2 || n_seg > (PER == 4 ? 256 : 512)))                   \
    hipLaunchKernelGGL(select_small_kernel<PER>, dim3(n_seg), dim3(kWave), 0, stream, wsum,     \
                       len, first, last, flags, n_units, budget, recent, score, keep,           \
                       kept_tokens, status);                                                    \
  else
  OMNITIDE_SELECT_SMALL(1)
  OMNITIDE_SELECT_SMALL(2)
  OMNITIDE_SELECT_SMALL(4)
  OMNITIDE_SELECT_SMALL(8)
#undef OMNITIDE_SELECT_SMALL
#define OMNITIDE_SELECT_CASE(PER)                                                               \
  if (n_units <= PER * kSelThreads)                                                             \
    hipLaunchKernelGGL(select_kernel<PER>, dim3(n_seg), dim3(kSelThreads), 0, stream, wsum,     \
                       len, first, last, flags, n_units, budget, recent, score, keep,           \
                       kept_tokens, status);                                                    \
  else
  OMNITIDE_SELECT_CASE(1)
  OMNITIDE_SELECT_CASE(2)
  OMNITIDE_SELECT_CASE(4)
  OMNITIDE_SELECT_CASE(8)
#undef OMNITIDE_SELECT_CASE
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace omnitide
