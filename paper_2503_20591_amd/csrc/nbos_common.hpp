// nbos_common.hpp — shared device helpers of the replay kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include "../../include/nbos.h"

namespace {

// ---- path profile (diagnostic build only: -DNBOS_PATH_PROFILE) -----------------------------------------
// Where does a replay spend its time? The wave that runs the replay reads the cycle counter at the marks
// below and adds the clocks since the previous mark to the category of the path just left (and a count);
// the sums of every replay go to a device array that nbos_path_profile_read copies out. The marks cost
// time of their own (two counter reads and two LDS atomics each), so a profiled launch runs a fifth to
// two fifths longer; the shares are what it is for. In the product build every mark is empty.
#ifdef NBOS_PATH_PROFILE
enum { PC_TILE, PC_ROUND, PC_ELECT, PC_MIGR, PC_FAIL, PC_START, PC_END, PC_TIMER_OTHER, PC_TICK, PC_RETRY_ELECT,
       PC_RETRY_MIGR, PC_RETRY_FAIL, PC_QUIET_RETRIES, PC_DROP, PC_LOOP_HORIZON, PC_LOOP_ROUND, PC_LOOP_TIMER,
       PC_LOOP_STARTEND, PC_LOOP_ATTEMPT, PC_HORIZON, PC_A_ELECT, PC_A_TARGET, PC_A_VICTIM, PC_A_BIND, PC_N };
constexpr int PATH_PROFILE_REPLAYS = 16384;      // replays beyond this many are not recorded
static __device__ unsigned long long g_path_profile[PATH_PROFILE_REPLAYS * 2 * PC_N];
__shared__ unsigned long long prof_t[PC_N];
__shared__ unsigned long long prof_n[PC_N];
#define PROF_BEGIN() if (threadIdx.x < PC_N) { prof_t[threadIdx.x] = 0; prof_n[threadIdx.x] = 0; } unsigned long long pt0 = __builtin_readcyclecounter()
#define PROF(cat, cnt) do { const unsigned long long now_ = __builtin_readcyclecounter(); if (threadIdx.x == 0) { atomicAdd(&prof_t[cat], now_ - pt0); atomicAdd(&prof_n[cat], (unsigned long long)(cnt)); } pt0 = __builtin_readcyclecounter(); } while (0)
// marks inside attempt(): clocks since the attempt began or since the mark before (these overlap PROF's)
#define PROF_SUB_BEGIN() unsigned long long pa0 = __builtin_readcyclecounter()
#define PROF_SUB(cat) do { const unsigned long long now_ = __builtin_readcyclecounter(); if (threadIdx.x == 0) { atomicAdd(&prof_t[cat], now_ - pa0); atomicAdd(&prof_n[cat], 1ull); } pa0 = __builtin_readcyclecounter(); } while (0)
#define PROF_OUT(rep) do { __syncthreads(); if (threadIdx.x < PC_N && (rep) < PATH_PROFILE_REPLAYS) { g_path_profile[((rep) * 2) * PC_N + threadIdx.x] = prof_t[threadIdx.x]; g_path_profile[((rep) * 2 + 1) * PC_N + threadIdx.x] = prof_n[threadIdx.x]; } } while (0)
// an attempt is booked by what came of it: the cell started by election, after a migration, or not at all
#define PROF_ATTEMPT_BEGIN(m, r) const uint32_t prof_st0 = (r).c_started; wave_sync(); const uint32_t prof_mg0 = uni((m).c32[CS_MIGR])
#define PROF_ATTEMPT_END(m, r, is_retry) do { wave_sync(); const uint32_t mg1_ = uni((m).c32[CS_MIGR]); \
    const int cat_ = (r).c_started == prof_st0 ? ((is_retry) ? PC_RETRY_FAIL : PC_FAIL) : mg1_ != prof_mg0 ? ((is_retry) ? PC_RETRY_MIGR : PC_MIGR) : ((is_retry) ? PC_RETRY_ELECT : PC_ELECT); \
    PROF(cat_, 1); } while (0)
#else
#define PROF_BEGIN() do { } while (0)
#define PROF(cat, cnt) do { } while (0)
#define PROF_SUB_BEGIN() do { } while (0)
#define PROF_SUB(cat) do { } while (0)
#define PROF_OUT(rep) do { } while (0)
#define PROF_ATTEMPT_BEGIN(m, r) do { } while (0)
#define PROF_ATTEMPT_END(m, r, is_retry) do { } while (0)
#endif

constexpr int WAVE = 64;
constexpr int32_t NEVER = 0x7FFFFFFF;
constexpr int NGPU = NBOS_MAX_GPUS;

// session states
constexpr uint32_t SS_UNPLACED = 0, SS_PLACED = 1, SS_QUEUED = 2, SS_REJECTED = 3, SS_ENDED = 4;
// session flag word: state[0..2] g-1[3..5] ending[6] queued_once[7] retries[8..11]
constexpr uint32_t SF_ENDING = 1u << 6, SF_QONCE = 1u << 7;
// queue entry kinds, in the order they run when due at the same time
constexpr uint32_t QK_END = 0, QK_RETRY = 2, QK_NEXT = 3;   // QK_NEXT: closed loop, the session's next event is due

struct KParams {
  const int64_t *ev_offset;
  const int32_t *ev_time, *ev_dur, *ev_sk;
  const int32_t *sess_offset;
  const uint8_t *sess_gpus;
  const int32_t *trace_of_replay, *cap_milli;
  nbos_stats *stats;
  uint64_t *dlog;          // null unless the decision log is on
  int32_t *ovf_dur;        // open loop: [n_replays][n_cap] (any-size kernel: n_cap + 1, the last one for lanes that have
                           // nothing to store) durations of queued cells whose timer is outside the sorted registers
  int64_t dlog_stride;     // codes per replay
  int32_t n_replays, H0, Hmax, HP, G;
  uint32_t flags;
  int32_t migr, boot, retry_iv, max_retries, scale_iv, idle_pct, min_hosts;
  int32_t f_milli, buffer; // auto-scaler: f * 1000 of the expected capacity, extra hosts
  int32_t batch_delay;     // Batch baseline: container start per job
  int32_t warm_n, warm_migr, prewarm;   // pre-warmed containers per host, warm migration delay, pre-warm time
  int32_t n_cap;           // LDS capacity: sessions
  int32_t batch;           // event-parallel rounds on (LDS kernel)
  // closed loop only. cl_chain: per event of the traces {the next event of its session (index within
  // the trace, -1: none), the think time before that event}; the second word is -1 for an event no
  // chain holds. cl_cursor: per replay and session the event that is due next or under way.
  const int2 *cl_chain;
  int32_t *cl_cursor;
  // null, or a word a validation kernel of the same stream has left: when it is not 0 the traces are
  // invalid and every replay ends at once with status NBOS_E_RANGE (calls that cannot wait for the
  // validation on the host)
  const uint32_t *trace_err;
  // null, or the replay each workgroup runs (a permutation of 0..n_replays-1): the order of the launch
  const int32_t *order;
};

// Workgroups start in the order of their index, and consecutive ones go to different XCDs of the chip. The
// library therefore hands the replays out longest first (see order_replays in nbos_replay.hip): the heavy
// replays are spread over the XCDs and the short ones fill the tail of the launch.
__device__ __forceinline__ int launch_slot_replay(const KParams &p) {
  if ((int)blockIdx.x >= p.n_replays) return p.n_replays;       // (the callers return at once)
  return p.order ? p.order[blockIdx.x] : (int)blockIdx.x;
}

// A replay that cannot run (invalid traces, more sessions than the launch has LDS for): its record
// holds the status and zeros.
__device__ __forceinline__ void refuse_replay(const KParams &p, int rep, int lane, int32_t status) {
  int32_t *out = (int32_t *)(p.stats + rep);
  for (int i = lane; i < (int)(sizeof(nbos_stats) / 4); i += WAVE) out[i] = i == 0 ? status : 0;
}

__device__ __forceinline__ int32_t uni(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ int32_t lane_get(int32_t v, int l) { return __builtin_amdgcn_readlane(v, l); }
// v with lane l mod 64 holding x (v_writelane_b32; clang has no builtin for it, so the intrinsic is declared under its own
// name: with a compiler that does not know it by that name the device link ends with an undefined symbol)
extern "C" __device__ __attribute__((const)) int nbos_writelane(int x, int l, int v) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ uint32_t lane_set(uint32_t v, uint32_t l, uint32_t x) {
  return (uint32_t)nbos_writelane((int)x, (int)l, (int)v);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }

// Minimum of v over the 64 lanes, returned wave-uniform. Needs all lanes active. Six DPP steps, each one
// v_min_u32 that reads its other operand from the lane next door: the lanes that a step leaves out take
// the identity of the minimum, which is what lets the compiler fold the move into the minimum. Four steps
// make each row of 16 lanes uniform (quad swaps, half-row mirror, row mirror), two broadcasts hand row 0's
// result to row 1, row 2's to row 3 and then row 1's to row 3. Bound by latency (a lone wave waits for every
// step); measured 84 clocks against 140 with separate moves and the four rows combined on the scalar unit.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_ones(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  v = umin(v, dpp_or_ones<0xB1, 0xF>(v));    // quad_perm [1,0,3,2]
  v = umin(v, dpp_or_ones<0x4E, 0xF>(v));    // quad_perm [2,3,0,1]
  v = umin(v, dpp_or_ones<0x141, 0xF>(v));   // row_half_mirror
  v = umin(v, dpp_or_ones<0x140, 0xF>(v));   // row_mirror
  v = umin(v, dpp_or_ones<0x142, 0xA>(v));   // row_bcast:15 into rows 1 and 3
  v = umin(v, dpp_or_ones<0x143, 0xC>(v));   // row_bcast:31 into rows 2 and 3
  return (uint32_t)lane_get((int)v, 63);
}

// Lanes of the one wave talk through LDS (one lane writes, others read later). The hardware runs a
// wave's LDS operations in order; this only stops the compiler from keeping LDS values in registers
// or moving LDS accesses across the point. It emits no instruction.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Times that every lane works out although only some lanes' are looked at: a lane without a timer or a cell of its
// own holds NEVER, or what belongs to others, and its sum may leave the type's range. They wrap: of a signed sum that
// leaves its range nothing that is computed from it is defined, and neither & nor pick shields the lanes that count.
__host__ __device__ __forceinline__ int32_t wrap_add(int32_t a, int32_t b) { return (int32_t)((uint32_t)a + (uint32_t)b); }
// a closed loop's next event: think time after the finish of the cell that started at t
__host__ __device__ __forceinline__ int32_t next_event_time(int32_t t, int32_t dur, int32_t think) { return wrap_add(wrap_add(t, dur), think); }
// a job of the Batch baseline that holds its GPUs from start on (a lane without one: an earlier job's start, and of a START
// or END event a duration that nobody has checked)
__host__ __device__ __forceinline__ int32_t job_finish(int32_t start, int32_t held) { return wrap_add(start, held); }
// the n-th retry of a cell
__host__ __device__ __forceinline__ int32_t retry_time(int32_t t_submit, int32_t n, int32_t interval) {
  return wrap_add(t_submit, (int32_t)((uint32_t)n * (uint32_t)interval));
}

// t + by (neither below 0), at most the end of the range
__host__ __device__ __forceinline__ int32_t add_in_range(int32_t t, int32_t by) {
  const uint32_t sum = (uint32_t)t + (uint32_t)by;
  return (int32_t)(sum < (uint32_t)NEVER ? sum : (uint32_t)NEVER);
}

// `by` after t. An open loop's times are checked against the range when the replay is created; the lag of a closed
// loop is not bounded in advance, and a time beyond the range stays at its end (a cell's start there ends the replay,
// a pre-warmed container is never available again).
template <class C>
__host__ __device__ __forceinline__ int32_t after(const C &, int32_t t, int32_t by) {
  if constexpr (!C::closed) return t + by;
  return add_in_range(t, by);
}

// c ? a : b without a branch, whatever a and b take to work out (the compiler likes to move that into an arm)
__device__ __forceinline__ int32_t pick(bool c, int32_t a, int32_t b) {
  const int32_t m = c ? -1 : 0;
  return (a & m) | (b & ~m);
}

// The value again, in a way that keeps the compiler from working out what depends on it before the loop: a
// comparison with a lane's number is one instruction, its result kept over the whole kernel is a pair of
// scalar registers, and those are spilled to vector lanes (two reads for each use).
__device__ __forceinline__ int fresh_lane(int lane) { asm volatile("" : "+v"(lane)); return lane; }
__device__ __forceinline__ int fresh(int v) { asm volatile("" : "+s"(v)); return v; }

// the lanes of a mask, as the per-lane condition it is (a select reads the scalar pair)
__device__ __forceinline__ bool in_mask(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// the median of three (one v_med3_i32)
__device__ __forceinline__ int32_t med3(int32_t a, int32_t b, int32_t c) { return max(min(a, b), min(max(a, b), c)); }

// wave-wide ballot straight from the predicate (no int round trip)
__device__ __forceinline__ uint64_t wballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

__device__ __forceinline__ int lane_rank(uint64_t mask) {   // set bits of mask below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// ---- what the replay kernels share ---------------------------------------------------------------------
// Each kernel has its own context type C (the replay's parameters p, its LDS arrays m, the lane, the
// per-lane registers) and its own wave-uniform register block R; the helpers below work on either.

// Kernel instances: F is the set of policy flags when it is known at compile time (the common sets get
// an instance of their own, which drops the code of everything that is switched off), or one of the two
// values that leave the flags to run time.
constexpr uint32_t kRuntimeFlags = 0xFFFFFFFFu;
constexpr uint32_t kRuntimeClosed = 0xFFFFFFFEu;     // policy flags at run time, closed-loop reading of the trace
constexpr uint32_t kPolicyFlags = NBOS_F_MIGRATE | NBOS_F_SCALE_OUT | NBOS_F_SCALE_IN | NBOS_F_AUTOSCALE | NBOS_F_DYNAMIC_SR |
                                  NBOS_F_STICKY_EXECUTOR | NBOS_F_WARM_POOL;
constexpr bool closed_loop_instance(uint32_t F) {
  return F == kRuntimeClosed || (F != kRuntimeFlags && (F & NBOS_F_CLOSED_LOOP) != 0);
}
template <uint32_t F>
__device__ __forceinline__ uint32_t instance_flags(const KParams &p) {
  return F == kRuntimeFlags ? (p.flags & ~NBOS_F_CLOSED_LOOP) : F == kRuntimeClosed ? (p.flags | NBOS_F_CLOSED_LOOP) : F;
}

// closed loop: a sorted timer's event has been loaded (bit 31 of qx); the widest refill window
constexpr int32_t CLX_LOADED = (int32_t)0x80000000;
constexpr int32_t CL_WIN_MAX = 1 << 24;

// Control flow of the replay kernels is wave-uniform, and no branch in their loops is divergent: a region that
// only some lanes execute costs about 40 clocks of its own (exec saved, a branch, exec restored) and, worse,
// makes the compiler rebuild the uniform branches around it with flags in scalar registers. So per-lane
// conditions are joined by & and | (&& and || on lanes are branches), a store that
// one lane would do is done by all lanes, same value and same address, loads clamp their index, and an LDS
// atomic that is one lane's business is done by all lanes too, the others adding 0 to words of their own
// somewhere in the first 512 bytes.
//
// Cold counters kept in LDS (ds_add, no return value). CS_BLAZY and the CL_B* sums are only fed by the
// event-parallel rounds of the any-size kernel. The head of a replay's LDS: c64[8], c32[16], hist[32].
enum { CS_PLACED, CS_REJECTED, CS_QUEUED, CS_ABORTED, CS_MIGR, CS_SO, CS_SI, CS_PEAK, CS_MAXDELAY,
       CS_NON, CS_SUMS, CS_OPENG, CS_BLAZY, CS_NREP, CS_MIGRWARM, CS_N32 };
enum { CL_SUMDELAY, CL_GWAIT, CL_PROV, CL_RESV, CL_SUB, CL_BDUR, CL_BGEXEC, CL_REPL, CL_N64 };

constexpr size_t LDS_HEAD = 8 * 8 + 16 * 4 + 32 * 4;
constexpr size_t LDS_LEAST = 512;              // what the adds below may touch (with zeros)

template <class L>
__device__ __forceinline__ void c32_add(L &m, int lane, int idx, uint32_t v) {
  lane = fresh_lane(lane);
  atomicAdd(&m.c32[(idx + lane) & (WAVE - 1)], lane == 0 ? v : 0u);
}
template <class L>
__device__ __forceinline__ void c32_max(L &m, int lane, int idx, uint32_t v) {
  lane = fresh_lane(lane);
  atomicMax(&m.c32[(idx + lane) & (WAVE - 1)], lane == 0 ? v : 0u);
}
template <class L>
__device__ __forceinline__ void c64_add(L &m, int lane, int idx, int64_t v) {
  lane = fresh_lane(lane);
  atomicAdd(&m.c64[(idx + lane) & (WAVE - 1)], lane == 0 ? (unsigned long long)v : 0ull);
}
template <class L>
__device__ __forceinline__ void hist_add(L &m, int lane, int32_t delay) {        // delay > 0
  const int b = 32 - __builtin_clz((uint32_t)delay);
  lane = fresh_lane(lane);
  atomicAdd(&m.hist[((b > 31 ? 31 : b) + lane) & (WAVE - 1)], lane == 0 ? 1u : 0u);
}

// Lanes with `hit` put v side by side into `staged`, from lane `at` on, in lane order; lanes below `at` keep what
// they have. One push through the LDS crossbar: the lanes without a hit fill the remaining places.
__device__ __forceinline__ int32_t stage_hits(int32_t staged, int lane, int at, bool hit, uint64_t hits, int32_t v) {
  const int n = __builtin_popcountll(hits);
  const int rank = lane_rank(hits);
  const int dst = (at + (hit ? rank : n + lane - rank)) & (WAVE - 1);
  const int32_t got = __builtin_amdgcn_ds_permute(dst << 2, v);
  return lane < at ? staged : got;
}

// Lane i < cnt holds a timer (t, key): how many of the cnt timers come before it. The other lanes hold NEVER and all
// ones, and get what they get. Times alone decide unless two are equal - then the ranks do not add up to
// 0 + 1 + ... + (cnt - 1) - so a timer costs one lane read, one comparison and one addition per other timer; timers
// of one instant are told apart by a second count over times and keys. Bound by the chain of lane reads: 40 timers
// took 440 instructions with times and keys compared from the start.
__device__ __forceinline__ int timer_ranks(int lane, int cnt, int32_t t, uint32_t key) {
  int rank = 0;
  for (int j0 = 0; j0 < cnt; j0 += 8) {
#pragma unroll
    for (int j = 0; j < 8; j++) rank += lane_get(t, j0 + j) < t ? 1 : 0;      // (NEVER is before nothing)
  }
  int sum = lane < cnt ? rank : 0;                 // at most 63 each, 2,016 in all
  sum += (int)dpp<0xB1>((uint32_t)sum);
  sum += (int)dpp<0x4E>((uint32_t)sum);
  sum += (int)dpp<0x141>((uint32_t)sum);
  sum += (int)dpp<0x140>((uint32_t)sum);
  const int total = lane_get(sum, 0) + lane_get(sum, 16) + lane_get(sum, 32) + lane_get(sum, 48);
  if (total != cnt * (cnt - 1) / 2) {
    rank = 0;
    for (int j = 0; j < cnt; j++) {
      const int32_t tj = lane_get(t, j);
      const uint32_t kj = (uint32_t)lane_get((int)key, j);
      rank += (tj < t) | ((tj == t) & (kj < key)) ? 1 : 0;
    }
  }
  return rank;
}

// Can the dynamic limit of Section 3.4.1 ever admit a host that the replay's own cap turns away? Not while
// every host that is on holds at most slim subscribed GPUs and more hosts are on than a request has GPUs:
// (S + g) n <= sum S + g <= n slim + g gives S + g <= slim + g / n, i.e. S + g <= slim for g < n. A host's
// S only grows through a placement or a migration that passed the limit (so S + g <= slim as long as the
// claim held so far) or starts at g on a host that was booted for the request (g <= G), so with slim >= G
// the claim holds for the whole replay, provided the cluster never has G hosts or fewer: it starts with
// H0 and the periodic release stops at min_hosts. Then the limit in force is the replay's cap, and the
// kernels keep the bounds that rest on a fixed cap. Otherwise (small clusters, caps below one request
// per empty host) the limit is worked out at every test.
__device__ __forceinline__ bool dynamic_limit_matters(const KParams &p, uint32_t flags, int32_t slim) {
  if (!(flags & NBOS_F_DYNAMIC_SR)) return false;
  const int32_t fewest = (flags & NBOS_F_SCALE_IN) ? (p.H0 < p.min_hosts ? p.H0 : p.min_hosts) : p.H0;
  return !(slim >= p.G && fewest > p.G);
}

// Largest S a host may hold and still take one more replica with request g (Section 3.4.1): the
// replay's cap, or with the dynamic limit the cluster-wide ratio after placing when that is larger:
// (S + g) / (G R) <= (sum S + g) / (n G R)  <=>  S + g <= floor((sum S + g) / n), n = hosts not off.
template <class C>
__device__ __forceinline__ int32_t cap_room(const C &c, int g) {
  int32_t lim = c.slim;
  if ((c.flags() & NBOS_F_DYNAMIC_SR) && c.dyn) {
    wave_sync();
    const uint32_t n_on = uni(c.m.c32[CS_NON]), tot = uni(c.m.c32[CS_SUMS]);
    if (n_on > 0) {
      const int32_t mean = (int32_t)((tot + (uint32_t)g) / n_on);
      lim = lim > mean ? lim : mean;
    }
  }
  return lim - g;
}

// One decision of the policy as a 64-bit code: host (10 bits), replica slot (2), outcome (4), session
// (16), time (32). The replay's digest is the FNV-style fold of its codes in order.
constexpr uint64_t DIGEST_PRIME = 0x100000001B3ULL;
__device__ __forceinline__ uint64_t decision_code(int32_t now, uint32_t outcome, uint32_t s, uint32_t slot,
                                                  uint32_t host) {
  return (uint64_t)(host | (slot << 10) | (outcome << 12) | (s << 16)) | ((uint64_t)(uint32_t)now << 32);
}
// Sum of a 64-bit value over the wave, wave-uniform (four DPP steps make the sum of every row of 16 lanes, the four
// rows are added on the scalar unit)
template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t v) {
  return ((uint64_t)dpp<CTRL>((uint32_t)(v >> 32)) << 32) | dpp<CTRL>((uint32_t)v);
}
__device__ __forceinline__ uint64_t lane_get64(uint64_t v, int l) {
  return ((uint64_t)(uint32_t)lane_get((int)(uint32_t)(v >> 32), l) << 32) | (uint32_t)lane_get((int)(uint32_t)v, l);
}
__device__ __forceinline__ uint64_t wave_sum64(uint64_t v) {
  v += dpp64<0xB1>(v);
  v += dpp64<0x4E>(v);
  v += dpp64<0x141>(v);
  v += dpp64<0x140>(v);
  return lane_get64(v, 0) + lane_get64(v, 16) + lane_get64(v, 32) + lane_get64(v, 48);
}

// The digest of many decisions at once: the codes of the lanes of `mask`, in the order of the lanes, are
// digest * P^n + sum over i of code_i * P^(n-1-i), every lane its own term. (On the scalar unit a decision is a 64-bit
// multiplication and an addition, a dozen instructions of the serial chain; here the multiplications of up to 64 are one.)
// power: per lane P^(63 - lane), see digest_powers.
__device__ __forceinline__ uint64_t digest_powers(int lane) {
  uint64_t power = 1, square = DIGEST_PRIME;
#pragma unroll
  for (int b = 0; b < 6; b++, square *= square) power *= ((63 - lane) >> b) & 1 ? square : 1ull;
  return power;
}
__device__ __forceinline__ uint64_t fold_decisions(uint64_t digest, uint64_t power, uint64_t mask, uint32_t code_lo, uint32_t code_hi) {
  const int n = __builtin_popcountll(mask);
  if (n == 0) return digest;
  // the factor P^(n-1-i) is held by lane i + 64 - n
  const int at = ((lane_rank(mask) + WAVE - n) & (WAVE - 1)) << 2;
  const uint32_t pl = (uint32_t)__builtin_amdgcn_ds_bpermute(at, (int)(uint32_t)power);
  const uint32_t ph = (uint32_t)__builtin_amdgcn_ds_bpermute(at, (int)(uint32_t)(power >> 32));
  const uint32_t lo = in_mask(mask) ? code_lo : 0u, hi = in_mask(mask) ? code_hi : 0u;
  const uint64_t sum = wave_sum64((((uint64_t)hi << 32) | lo) * (((uint64_t)ph << 32) | pl));
  return digest * (lane_get64(power, WAVE - n) * DIGEST_PRIME) + sum;
}

template <class C, class R>
__device__ __forceinline__ void decide(C &c, R &r, int32_t now, uint32_t outcome, uint32_t s, uint32_t slot,
                                       uint32_t host) {
  const uint64_t code = decision_code(now, outcome, s, slot, host);
  r.digest = r.digest * DIGEST_PRIME + code;
  if (__builtin_expect(c.dlog != nullptr, 0)) {
    if ((int64_t)r.n_dec < c.p.dlog_stride) c.dlog[r.n_dec] = code;
  }
  r.n_dec++;
}

// ---- timers: the 64 earliest, sorted ascending by (time, kind << 16 | id), entry i in lane i -----
// Invariant: every entry in the registers is earlier than every timer that waits in the session
// records, and the registers are empty only if none waits there. Each kernel brings its own
// ovf_push (a timer goes to wait in its session's record) and refill (the earliest waiting timers come
// into the registers).
template <class C, class R>
__device__ __forceinline__ void timer_push(C &c, R &r, int32_t t, uint32_t kind, uint32_t id, int32_t d,
                                           int32_t x = 0, int32_t nx = -1, int32_t nth = 0) {
  uint32_t k = (kind << 16) | id;
  if (__builtin_expect(r.q_n == WAVE, 0)) {
    int32_t mt = lane_get(c.qt, WAVE - 1);
    uint32_t mk = (uint32_t)lane_get((int)c.qk, WAVE - 1);
    if (t < mt || (t == mt && k < mk)) {
      ovf_push(c, r, mt, mk, lane_get(c.qd, WAVE - 1));   // the latest register entry moves out
      r.q_n = WAVE - 1;
    } else {
      ovf_push(c, r, t, k, d);
      return;
    }
  } else if (r.o_n > 0 && !(t < r.o_min_t || (t == r.o_min_t && k < r.o_min_k))) {
    ovf_push(c, r, t, k, d);
    return;
  }
  const bool before = (c.lane < r.q_n) & ((c.qt < t) | ((c.qt == t) & (c.qk < k)));
  int pos = __builtin_popcountll(wballot(before));
  int32_t st = __builtin_amdgcn_update_dpp(c.qt, c.qt, 0x138, 0xF, 0xF, false);          // wave_shr:1
  int32_t sd = __builtin_amdgcn_update_dpp(c.qd, c.qd, 0x138, 0xF, 0xF, false);
  uint32_t sk = (uint32_t)__builtin_amdgcn_update_dpp((int)c.qk, (int)c.qk, 0x138, 0xF, 0xF, false);
  const bool up = c.lane > pos, here = c.lane == pos;
  c.qt = here ? t : up ? st : c.qt;   c.qd = here ? d : up ? sd : c.qd;   c.qk = here ? k : up ? sk : c.qk;
  if constexpr (C::closed) {
    const int32_t sx = __builtin_amdgcn_update_dpp(c.qx, c.qx, 0x138, 0xF, 0xF, false);
    const int32_t sn = __builtin_amdgcn_update_dpp(c.qnx, c.qnx, 0x138, 0xF, 0xF, false);
    const int32_t sh = __builtin_amdgcn_update_dpp(c.qnth, c.qnth, 0x138, 0xF, 0xF, false);
    c.qx = here ? x : up ? sx : c.qx;   c.qnx = here ? nx : up ? sn : c.qnx;   c.qnth = here ? nth : up ? sh : c.qnth;
  }
  r.q_n++;
  if (pos == 0) r.q_head_t = t;
}

// remove the earliest timer (lane 0); refill from the session records when the registers run empty
template <class C, class R>
__device__ __forceinline__ void timer_pop(C &c, R &r) {
  c.qt = __builtin_amdgcn_update_dpp(c.qt, c.qt, 0x130, 0xF, 0xF, false);                // wave_shl:1
  c.qd = __builtin_amdgcn_update_dpp(c.qd, c.qd, 0x130, 0xF, 0xF, false);
  c.qk = (uint32_t)__builtin_amdgcn_update_dpp((int)c.qk, (int)c.qk, 0x130, 0xF, 0xF, false);
  r.q_n--;
  if constexpr (C::closed) {
    c.qx = __builtin_amdgcn_update_dpp(c.qx, c.qx, 0x130, 0xF, 0xF, false);
    c.qnx = __builtin_amdgcn_update_dpp(c.qnx, c.qnx, 0x130, 0xF, 0xF, false);
    c.qnth = __builtin_amdgcn_update_dpp(c.qnth, c.qnth, 0x130, 0xF, 0xF, false);
  }
  if (__builtin_expect(r.q_n == 0 && r.o_n > 0, 0)) refill(c, r);
  r.q_head_t = r.q_n > 0 ? lane_get(c.qt, 0) : NEVER;
}

}  // namespace
