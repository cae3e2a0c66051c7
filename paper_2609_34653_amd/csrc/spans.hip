// OmniPick span plan: a census of the units, the plan, the slot mask.  Up to 512 units and not too
// many workgroups the plan is made by every workgroup of the mask kernel (two launches), beyond by
// a kernel of its own.
//
// 1. Census (one wave per unit).  The wave walks its unit's slots 1024 at a time (one aligned
//    16-byte block of tags per lane) and
//    finds where each span starts: at the unit's first slot and wherever the tag changes.  A
//    running maximum of the start slots (wave scan plus a carry across chunks) gives every
//    token its place in its span.  Each slot gets a code in the workspace: marker tokens and
//    the first sink_video / sink_audio tokens of each video / audio span are sinks (kept while
//    the unit is retained at all), text tokens get their rank among the unit's text tokens,
//    everything else is dropped from a partially kept unit.  Per unit: sinks, text tokens.
// 2. Plan (one wave up to 512 units, a workgroup of 1024 threads per segment beyond).  Each
//    thread owns up to 8 consecutive units.  Every step of the plan is a scan over units in id
//    (temporal) order, so the sequential walks of the planner become thresholds on prefix sums:
//      recent    newest live non-system units whose suffix total (own tokens included) is at
//                most R: lengths are positive, so the suffix grows monotonically and "stop at
//                the first misfit" is the set {u : suffix(u) <= R}
//      older     unit u keeps its sinks plus clamp(text_budget - T_u, 0, text_u) of its text
//                tokens, T_u = text tokens of older units before u
//      trimming  drop order = partially retained units by id, then complete non-system units
//                by id.  The i-th candidate is dropped iff, before it, the plan still exceeds
//                the low watermark and more than one unit is retained.  Both quantities only
//                decrease along the order, so each candidate decides from its exclusive prefix
//                (tokens and count of earlier candidates) alone.
// 3. Mark (one thread per slot): the slot stays if its unit is kept whole, or its unit is kept
//    in part and the slot is a sink or one of the unit's first text_keep text tokens.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace omnitide {

size_t span_plan_workspace_bytes(int n_seg, int n_slots, int n_units) {
  return span_ws_seg_bytes(n_slots, n_units) * static_cast<size_t>(n_seg);
}

namespace {

constexpr int kMaxPer = 8;
constexpr int kCensusWaves = 4;
constexpr int32_t kInfoSink = -1;   // marker, or inside the sink prefix of its span
constexpr int32_t kInfoDrop = -2;   // any other non-text token

struct SpanWs {
  int32_t* info;        // [n_slots] per-slot code: kInfoSink, kInfoDrop or text rank in unit
  int32_t* sinks;       // [U] sink tokens of the unit (-1: bad tag or slots outside the pool)
  int32_t* text;        // [U] text tokens of the unit
  int32_t* text_keep;   // [U] text tokens an older unit keeps
};

__device__ inline SpanWs span_ws(uint8_t* ws, int seg, int n_slots, int n_units) {
  uint8_t* b = ws + span_ws_seg_bytes(n_slots, n_units) * static_cast<size_t>(seg);
  const size_t info_bytes = span_ws_info_bytes(n_slots);
  const size_t ub = static_cast<size_t>(n_units) * 4;
  return SpanWs{reinterpret_cast<int32_t*>(b), reinterpret_cast<int32_t*>(b + info_bytes),
                reinterpret_cast<int32_t*>(b + info_bytes + ub),
                reinterpret_cast<int32_t*>(b + info_bytes + 2 * ub)};
}

constexpr int kCensusPer = 16;          // consecutive slots per lane in one census step
// Buffer resource word 3 for raw (unformatted) 32-bit data on this chip, and a byte offset past
// any buffer (accesses there read zero and write nothing).
constexpr int kBufferFlags = 0x00020000;
constexpr int kOutOfBuffer = 0x7fffffff;

__global__ __launch_bounds__(kCensusWaves * kWave) void span_census_kernel(
    const uint8_t* __restrict__ mod_g, const int32_t* __restrict__ len_g,
    const int32_t* __restrict__ first_g, int n_slots, int n_units, int sink_video,
    int sink_audio, uint8_t* __restrict__ ws, int32_t* __restrict__ status) {
  constexpr int P = kCensusPer;
  const int seg = blockIdx.y;
  const int lane = threadIdx.x & (kWave - 1);
  const int u = blockIdx.x * kCensusWaves + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (u >= n_units) return;
  const SpanWs W = span_ws(ws, seg, n_slots, n_units);
  const size_t ub = static_cast<size_t>(seg) * n_units;
  const int n = len_g[ub + u];
  const int f = first_g[ub + u];
  if (n <= 0 || f < 0 || f > n_slots - n) {     // no slots, or not inside the pool (the plan
    if (lane == 0) {                            // reports the latter as a tag error)
      W.sinks[u] = n <= 0 ? 0 : -1;
      W.text[u] = 0;
    }
    return;
  }
  // aligned 16-slot blocks of the segment's tag bytes (slot s at seg_tags + s)
  const uint8_t* seg_tags = mod_g + static_cast<size_t>(seg) * n_slots;
  const uintptr_t blk0 = block16_floor(seg_tags + f);
  const uintptr_t end = reinterpret_cast<uintptr_t>(seg_tags + f + n);
  const __amdgpu_buffer_rsrc_t info_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(W.info, 0, 4 * n_slots, kBufferFlags);
  int carry_tag = -1;      // tag of the slot before the step (-1 at the unit's start)
  int carry_start = f;     // first slot of the span that slot belongs to
  int carry_text = 0;      // the unit's text tokens before the step
  int sinks = 0;
  bool bad = false;
  for (uintptr_t c = blk0; c < end; c += P * kWave) {
    const uintptr_t b = c + P * static_cast<uintptr_t>(lane);   // this lane's block
    const int s0 = static_cast<int>(static_cast<intptr_t>(b) -
                                    reinterpret_cast<intptr_t>(seg_tags));
    int m[P];
    {
      uint8_t raw[16] = {};
      if (b < end) load_block16(b, raw);
#pragma unroll
      for (int j = 0; j < P; ++j) m[j] = ((s0 + j >= f) & (s0 + j < f + n)) ? raw[j] : -1;
    }
    int prev = __shfl_up(m[P - 1], 1, kWave);
    if (lane == 0) prev = carry_tag;
    int run = -1, nt = 0;
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const int pm = j == 0 ? prev : m[j - 1];
      if (m[j] >= 0 && m[j] != pm) run = s0 + j;   // a span starts here
      nt += m[j] == OMNITIDE_MOD_TEXT ? 1 : 0;
    }
    // running maximum of span starts, and over the lanes before this one
    const int inc = wave_scan_max_i32(run, -1);
    const int exc = dpp_move<kDppWaveShr1, 0xf>(-1, inc);
    int start = max(exc, carry_start);             // span start of the slot before s0
    const int incl = wave_inclusive_scan(nt);
    const int text_tot = __shfl(incl, kWave - 1, kWave);
    int text_rank = carry_text + incl - nt;        // the unit's text tokens before s0
    // Branch-free per slot (selects instead of divergent branches); the code of a slot outside
    // the unit goes to an offset past the buffer, which the hardware drops.
    int pm = prev;
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const int s = s0 + j;
      // (bitwise & and | on the conditions: no short-circuit branches)
      const bool live = m[j] >= 0;
      start = (live & (m[j] != pm)) ? s : start;
      const int place = s - start + 1;             // 1-based place in its span
      const bool text = m[j] == OMNITIDE_MOD_TEXT;
      const bool sink = (m[j] == OMNITIDE_MOD_MARK) |
                        ((m[j] == OMNITIDE_MOD_VIDEO) & (place <= sink_video)) |
                        ((m[j] == OMNITIDE_MOD_AUDIO) & (place <= sink_audio));
      const int32_t code = text ? text_rank : (sink ? kInfoSink : kInfoDrop);
      text_rank += (live & text) ? 1 : 0;
      sinks += (live & !text & sink) ? 1 : 0;
      bad |= live & (m[j] > OMNITIDE_MOD_MARK);
      __builtin_amdgcn_raw_buffer_store_b32(code, info_rsrc, live ? 4 * s : kOutOfBuffer, 0, 0);
      pm = m[j];
    }
    carry_tag = __shfl(m[P - 1], kWave - 1, kWave);
    carry_start = max(carry_start, __shfl(inc, kWave - 1, kWave));
    carry_text += text_tot;
  }
  const uint32_t tot = wave_sum_u32(static_cast<uint32_t>(sinks));
  const bool any_bad = __any(bad);
  if (lane == 0) {
    W.sinks[u] = any_bad ? -1 : static_cast<int32_t>(tot);
    W.text[u] = carry_text;
    if (any_bad) set_status(status, OMNITIDE_E_TAGS);
  }
}

// Scans of the plan over units: by one wave (registers only, no barrier) or by the workgroup.
template <bool WAVE>
struct PlanScan {
  int32_t* scr;                              // workgroup scratch (unused by one wave)
  __device__ int exclusive_sum(int v, int* total) const {
    if constexpr (WAVE) {
      const int inc = wave_inclusive_scan(v);
      *total = __builtin_amdgcn_readlane(inc, kWave - 1);
      return inc - v;
    } else {
      return block_exclusive_scan(v, scr, total);
    }
  }
  __device__ int sum(int v) const {
    if constexpr (WAVE) return static_cast<int>(wave_sum_u32(static_cast<uint32_t>(v)));
    else return block_sum(v, scr);
  }
  __device__ int exclusive_max(int v, int lo) const {
    if constexpr (WAVE) {
      return wave_exclusive_max_i32(v, lo);
    } else {
      int ignored;
      return block_exclusive_max(v, lo, scr, &ignored);
    }
  }
};

struct SpanPlanIn {
  const int32_t* len;
  const int32_t* first;
  const int32_t* last;
  const uint32_t* flags;
  int n_slots, n_units, low, high, recent, text_budget;
};

// The plan of one segment: thread t owns units [t*per, (t+1)*per).  Leaves the unit lengths (0 past
// U and for units without slots), kept lengths and kept text tokens of its units in ln, kl and tk,
// and returns the segment's total, or -1 for malformed units (kl is then 0).
template <bool WAVE>
__device__ inline int plan_units(const SpanPlanIn& in, size_t base, const SpanWs& W, int tid,
                                 int per, const PlanScan<WAVE>& sc, int (&ln)[kMaxPer],
                                 int (&kl)[kMaxPer], int (&tk)[kMaxPer]) {
  const int U = in.n_units;
  const int u0 = tid * per;
  int fs[kMaxPer], ls[kMaxPer], sk[kMaxPer], tx[kMaxPer];
  uint32_t fl[kMaxPer];
#pragma unroll
  for (int i = 0; i < kMaxPer; ++i) {        // all loads first: one memory round trip
    const int u = min(u0 + i, U - 1);
    ln[i] = in.len[base + u];
    fs[i] = in.first[base + u];
    ls[i] = in.last[base + u];
    fl[i] = in.flags[base + u];
    sk[i] = W.sinks[u];
    tx[i] = W.text[u];
    kl[i] = tk[i] = 0;
  }
  bool bad = false;
  int my_max_first = -1;
#pragma unroll
  for (int i = 0; i < kMaxPer; ++i) {
    if (!(i < per && u0 + i < U) || ln[i] <= 0) ln[i] = 0;
    const bool live = ln[i] > 0;
    const bool in_range = live && fs[i] >= 0 && fs[i] <= in.n_slots - ln[i];
    bad |= live && (!in_range || ls[i] - fs[i] + 1 != ln[i] || sk[i] < 0);
    if (live) my_max_first = max(my_max_first, fs[i]);
  }
  // live units must appear in unit order
  int run = sc.exclusive_max(my_max_first, -1);
#pragma unroll
  for (int i = 0; i < kMaxPer; ++i) {
    if (ln[i] > 0) {
      bad |= fs[i] <= run;
      run = max(run, fs[i]);
    }
  }
  if (sc.sum(bad ? 1 : 0) > 0) return -1;

  int my_len = 0;
#pragma unroll
  for (int i = 0; i < kMaxPer; ++i) my_len += ln[i];
  const int total = sc.sum(my_len);
  if (total <= in.high) {                      // at or below the high watermark: keep all
#pragma unroll
    for (int i = 0; i < kMaxPer; ++i) kl[i] = ln[i];
    return total;
  }

  bool sys[kMaxPer];
  int my_elig = 0;
#pragma unroll
  for (int i = 0; i < kMaxPer; ++i) {
    sys[i] = ln[i] > 0 && (fl[i] & 1u) != 0;
    my_elig += (ln[i] > 0 && !sys[i]) ? ln[i] : 0;
  }
  // recent window: suffix sums of eligible lengths
  int elig_total;
  const int elig_before = sc.exclusive_sum(my_elig, &elig_total);
  int suffix = elig_total - elig_before - my_elig;
  bool rec[kMaxPer];
#pragma unroll
  for (int i = kMaxPer - 1; i >= 0; --i) {
    rec[i] = false;
    if (ln[i] > 0 && !sys[i]) {
      suffix += ln[i];
      rec[i] = suffix <= in.recent;
    }
  }
  // older units: their sinks, and text tokens under the shared budget (oldest first)
  int my_text = 0;
#pragma unroll
  for (int i = 0; i < kMaxPer; ++i) my_text += (ln[i] > 0 && !sys[i] && !rec[i]) ? tx[i] : 0;
  int text_total;
  int text_before = sc.exclusive_sum(my_text, &text_total);
  int my_kept = 0, my_part = 0, my_part_n = 0, my_comp = 0, my_comp_n = 0, my_ret = 0;
#pragma unroll
  for (int i = 0; i < kMaxPer; ++i) {
    int k = 0;
    if (ln[i] > 0) {
      if (sys[i] || rec[i]) {
        k = ln[i];
      } else {
        tk[i] = min(tx[i], max(in.text_budget - text_before, 0));
        k = sk[i] + tk[i];
        text_before += tx[i];
      }
    }
    kl[i] = k;
    my_kept += k;
    my_ret += k > 0 ? 1 : 0;
    if (k > 0 && k < ln[i]) {
      my_part += k;
      ++my_part_n;
    } else if (k > 0 && !sys[i]) {
      my_comp += k;
      ++my_comp_n;
    }
  }
  const int kept0 = sc.sum(my_kept);
  const int retained0 = sc.sum(my_ret);
  int part_tok, part_n, comp_tok, comp_n;
  int part_before = sc.exclusive_sum(my_part, &part_tok);
  int part_rank = sc.exclusive_sum(my_part_n, &part_n);
  int comp_before = sc.exclusive_sum(my_comp, &comp_tok);
  int comp_rank = sc.exclusive_sum(my_comp_n, &comp_n);
  (void)comp_tok;
  (void)comp_n;
  int my_final = 0;
#pragma unroll
  for (int i = 0; i < kMaxPer; ++i) {
    const int k = kl[i];
    if (k > 0 && k < ln[i]) {
      // candidate number part_rank (0-based) of the drop order
      if (kept0 - part_before > in.low && retained0 - part_rank > 1) kl[i] = 0;
      part_before += k;
      ++part_rank;
    } else if (k > 0 && !sys[i]) {
      if (kept0 - part_tok - comp_before > in.low && retained0 - part_n - comp_rank > 1) kl[i] = 0;
      comp_before += k;
      ++comp_rank;
    }
    my_final += kl[i];
  }
  return sc.sum(my_final);
}

// The plan as a kernel of its own, one workgroup per segment: one wave up to kMarkUnits units
// (WAVE), kPlanThreads beyond.
constexpr int kPlanThreads = 1024;

template <bool WAVE>
__global__ __launch_bounds__(WAVE ? kWave : kPlanThreads) void plan_spans_kernel(
    SpanPlanIn in, int32_t* __restrict__ keep_len_g, int32_t* __restrict__ kept_g,
    uint8_t* __restrict__ ws, int32_t* __restrict__ status) {
  constexpr int T = WAVE ? kWave : kPlanThreads;
  __shared__ int32_t scr[T / kWave + 1];
  const int seg = blockIdx.x;
  const int tid = threadIdx.x;
  const int per = (in.n_units + T - 1) / T;
  const size_t base = static_cast<size_t>(seg) * in.n_units;
  const SpanWs W = span_ws(ws, seg, in.n_slots, in.n_units);
  int ln[kMaxPer], kl[kMaxPer], tk[kMaxPer];
  const int kept = plan_units<WAVE>(in, base, W, tid, per, PlanScan<WAVE>{scr}, ln, kl, tk);
#pragma unroll
  for (int i = 0; i < kMaxPer; ++i) {
    const int u = tid * per + i;
    if (i < per && u < in.n_units) {
      keep_len_g[base + u] = kl[i];
      W.text_keep[u] = tk[i];
    }
  }
  if (tid == 0) {
    kept_g[seg] = max(kept, 0);
    if (kept < 0) set_status(status, OMNITIDE_E_TAGS);
  }
}

// The slot's keep flag, given its unit's length, kept length and kept text tokens.
__device__ inline uint8_t slot_kept(int ln, int kl, int tk, int32_t code) {
  return kl > 0 && (kl >= ln || code == kInfoSink || (code >= 0 && code < tk)) ? 1 : 0;
}

constexpr int kMarkThreads = 256;

__global__ __launch_bounds__(kMarkThreads) void span_mark_kernel(
    const int32_t* __restrict__ uid_g, const int32_t* __restrict__ len_g,
    const int32_t* __restrict__ keep_len_g, int n_slots, int n_units, uint8_t* __restrict__ ws,
    uint8_t* __restrict__ keep_slot_g) {
  const int seg = blockIdx.y;
  const int s = blockIdx.x * kMarkThreads + threadIdx.x;
  if (s >= n_slots) return;
  const size_t sb = static_cast<size_t>(seg) * n_slots;
  const size_t ub = static_cast<size_t>(seg) * n_units;
  const int u = uid_g[sb + s];
  uint8_t out = 0;
  if (u >= 0 && u < n_units) {
    const int kl = keep_len_g[ub + u];
    if (kl > 0) {
      const SpanWs W = span_ws(ws, seg, n_slots, n_units);
      out = slot_kept(len_g[ub + u], kl, W.text_keep[u], W.info[s]);
    }
  }
  keep_slot_g[sb + s] = out;
}

// Plan and mask in one launch for up to kMarkUnits units: wave 0 of every workgroup plans the
// segment into LDS (about 2 us, in all workgroups at once) while the other waves' tags and codes
// are on their way, then the workgroup marks its kMarkSlots slots; workgroup 0 writes the plan
// out.  Latency-bound: one launch less where the host launches, and by graph replay 8-10% less for
// the whole call where many segments have few units (36 x 32,768 slots in 38 units: 16.3 us
// against 17.7 with a plan launch), the same for one segment (358 units and 81,920 slots: 10.4).
constexpr int kMarkUnits = kWave * kMaxPer;
constexpr int kMarkPer = 4;
constexpr int kMarkSlots = kMarkThreads * kMarkPer;
// Every workgroup repeats the plan, so its launch is saved only while all of them run at once (five
// per CU: 1,280 of 8 x 1,024 slots in 39 units 17.6 us against 19.6 in two launches, 1,600 of them
// 24.3 and 22.7) and the units they read between them are few (8 x 81,920 slots in 358 units,
// 640 workgroups: 15.2 and 14.9; 36 x 81,920: 40.4 and 32.1).
constexpr long kFusedMarks = 1280;
constexpr long kFusedUnits = 65536;

__global__ __launch_bounds__(kMarkThreads) void span_plan_mark_kernel(
    SpanPlanIn in, const int32_t* __restrict__ uid_g, int32_t* __restrict__ keep_len_g,
    int32_t* __restrict__ kept_g, uint8_t* __restrict__ ws, uint8_t* __restrict__ keep_slot_g,
    int32_t* __restrict__ status) {
  __shared__ int32_t s_len[kMarkUnits], s_keep[kMarkUnits], s_text[kMarkUnits];
  const int seg = blockIdx.y;
  const int tid = threadIdx.x;
  const int U = in.n_units;
  const size_t base = static_cast<size_t>(seg) * U;
  const size_t sb = static_cast<size_t>(seg) * in.n_slots;
  const SpanWs W = span_ws(ws, seg, in.n_slots, U);
  int uid[kMarkPer], code[kMarkPer];
#pragma unroll
  for (int i = 0; i < kMarkPer; ++i) {
    const int s = blockIdx.x * kMarkSlots + i * kMarkThreads + tid;
    uid[i] = s < in.n_slots ? uid_g[sb + s] : -1;
    code[i] = s < in.n_slots ? W.info[s] : 0;      // garbage for slots of no unit, unused
  }
  if (tid < kWave) {
    int ln[kMaxPer], kl[kMaxPer], tk[kMaxPer];
    const int kept = plan_units<true>(in, base, W, tid, kMaxPer, PlanScan<true>{nullptr}, ln, kl,
                                      tk);
#pragma unroll
    for (int i = 0; i < kMaxPer; ++i) {
      const int u = kMaxPer * tid + i;
      s_len[u] = ln[i];
      s_keep[u] = kl[i];
      s_text[u] = tk[i];
      if (blockIdx.x == 0 && u < U) keep_len_g[base + u] = kl[i];
    }
    if (blockIdx.x == 0 && tid == 0) {
      kept_g[seg] = max(kept, 0);
      if (kept < 0) set_status(status, OMNITIDE_E_TAGS);
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kMarkPer; ++i) {
    const int s = blockIdx.x * kMarkSlots + i * kMarkThreads + tid;
    if (s >= in.n_slots) continue;
    const int u = uid[i];
    keep_slot_g[sb + s] =
        u >= 0 && u < U ? slot_kept(s_len[u], s_keep[u], s_text[u], code[i]) : 0;
  }
}

}  // namespace

hipError_t launch_plan_spans(const SpanPlanArgs& a, hipStream_t stream) {
  uint8_t* ws = static_cast<uint8_t*>(a.workspace);
  const dim3 cgrid((a.n_units + kCensusWaves - 1) / kCensusWaves, a.n_seg);
  hipLaunchKernelGGL(span_census_kernel, cgrid, dim3(kCensusWaves * kWave), 0, stream,
                     a.modality, a.unit_len, a.unit_first, a.n_slots, a.n_units, a.sink_video,
                     a.sink_audio, ws, a.d_status);
  const SpanPlanIn in{a.unit_len, a.unit_first, a.unit_last, a.unit_flags, a.n_slots,
                      a.n_units,  a.low,        a.high,      a.recent,     a.text_budget};
  const long marks = a.n_seg * ((static_cast<long>(a.n_slots) + kMarkSlots - 1) / kMarkSlots);
  if (a.n_units <= kMarkUnits && marks <= kFusedMarks && marks * a.n_units <= kFusedUnits) {
    // one workgroup at least: it writes the plan also for a pool without slots
    const dim3 grid(std::max(1, (a.n_slots + kMarkSlots - 1) / kMarkSlots), a.n_seg);
    hipLaunchKernelGGL(span_plan_mark_kernel, grid, dim3(kMarkThreads), 0, stream, in, a.unit_id,
                       a.keep_len, a.kept_tokens, ws, a.keep_slot, a.d_status);
    return hipGetLastError();
  }
  if (a.n_units <= kMarkUnits)
    hipLaunchKernelGGL(plan_spans_kernel<true>, dim3(a.n_seg), dim3(kWave), 0, stream, in,
                       a.keep_len, a.kept_tokens, ws, a.d_status);
  else
    hipLaunchKernelGGL(plan_spans_kernel<false>, dim3(a.n_seg), dim3(kPlanThreads), 0, stream, in,
                       a.keep_len, a.kept_tokens, ws, a.d_status);
  if (a.n_slots > 0) {
    const dim3 mgrid((a.n_slots + kMarkThreads - 1) / kMarkThreads, a.n_seg);
    hipLaunchKernelGGL(span_mark_kernel, mgrid, dim3(kMarkThreads), 0, stream, a.unit_id,
                       a.unit_len, a.keep_len, a.n_slots, a.n_units, ws, a.keep_slot);
  }
  return hipGetLastError();
}

}  // namespace omnitide
