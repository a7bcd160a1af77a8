// nbos_kernel_reg.hpp — replay kernel for clusters of at most 64 hosts: host state in registers.
//
// One workgroup (one wave64) per replay.
//
// GPUs:   fin[j], j < NJ = ceil(hosts_max / 8). Lane L = (hl = L >> 3, k = L & 7) holds in fin[j] the
//         "busy until" time of GPU k of host 8 j + hl. A GPU is committed at time t iff fin > t, so
//         the ballot of (fin[j] > now) is a 64-bit word with one byte of busy-GPU bits per host. GPUs beyond
//         G are held for ever: counts are of 8, the same number too high on every host.
//         Binding g GPUs for a cell (paper Section 3.3) = writing its finish time into the g lowest
//         free GPUs of the host byte (ballot + lane rank). Completions need no timer: every timer
//         due at or before an item runs before that item and a completion only lowers C, so
//         "released once the clock has passed fin" is exact.
// Hosts:  lane h = host h holds ready_at (0 initial, NEVER while off: provisioning needs no timer
//         either, Section 3.4.2) and S | replicas << 16 (Section 3.4.1). The committed count C of
//         every host in lane = host layout comes from the NJ ballots by a byte extract + popcount.
// Choice: feasibility by ballot; executor election (Section 3.2.2) tests 3 bits of that ballot;
//         placement / migration target = wave minimum of the packed key (C, S, host), so ties go
//         to the lowest host index.
// Events: coalesced dword loads, one event per lane, next tile in flight while the current tile
//         is consumed from registers (v_readlane). At tile start every lane prefetches the record of
//         its event's session from LDS; events of sessions in a final state (rejected / ended) are
//         counted in bulk and skipped. A cell that starts at once brings the lanes of its session up to date, any
//         other change of a record marks them stale, and only those are read again from LDS.
// Timers: RETRY of a queued cell (Section 3.2.3) and the END of a session that was busy when its END
//         arrived are the only timers that change decisions. The 64 earliest live sorted in
//         registers (insert = ballot + DPP wave shift, pop = DPP wave shift); later ones stay with
//         their session (a flag in its record, their time implied by it) until the registers run empty.
// Closed loop (the paper's section "Interactive Deep Learning Training"; nbos_replay_reg_closed_kernel at the end of this file): only the
//         first STARTs come from the stream, every other event of a session is a timer that is due a
//         think time after the session's previous cell is over. See nbos_kernel_closed.hpp for the
//         chain records this reads and for the same scheme on the any-size kernel.
// Sessions in LDS, 8 bytes each: one word with the state, g, the retry count, the three replica hosts
//         (6 bits each) and the last executor slot; one time word (busy-until, or the submit time while
//         queued). The duration of a queued cell travels with its timer.
#pragma once
#include "nbos_common.hpp"

namespace {
namespace regk {

// Session record: x = state (bits 0-2) | g - 1 (3-5) | ENDING (6) | RK_OVF (7) | retries (8-11) |
// host of slot 0, 1, 2 (6 bits each from bit 12) | last executor slot + 1 (30-31); y = time word.
// The code below calls the word `hw` where it looks at the hosts and `fl` where it looks at the low
// bits; both names hold the whole word.
constexpr uint32_t RK_OVF = 1u << 7;
constexpr uint32_t RK_FLAGS = 0xFFFu;        // the bits below the hosts
__device__ __forceinline__ uint32_t slot_host(uint32_t hw, uint32_t slot) { return (hw >> (12u + 6u * slot)) & 63u; }

struct Lds {
  int32_t *warm;     // [64][4] when each pre-warmed container of a host is available (only with the pool)
  int2 *sess;
  uint32_t *hist;
  uint32_t *c32;
  unsigned long long *c64;
};

// hot uniform registers
struct Regs {
  uint32_t n_dec, c_total, c_imm, c_started, c_busy, c_unplaced, reused, h0;
  int64_t sum_dur, g_exec;
  int32_t lazy_max, t_end;
  int32_t q_n, q_head_t;                 // sorted register queue: size, time of lane 0
  int32_t o_n, o_min_t;                  // timers outside the registers: how many, the earliest
  uint32_t o_min_k;
  int32_t status;
  uint64_t at_once;                      // lanes of the current tile whose cells started at once, not in the sums yet
  // closed loop: the event being handled, its duration and kind (packed as in Ctx::qx), its session's next
  // event and the think time before that; the time window the next refill takes
  int32_t cl_e, cl_x, cl_nx, cl_nth, cl_win;
};

template <int NJ, uint32_t F>
struct Ctx {
  const KParams &p;
  Lds m;
  int lane;
  int n_sess;
  int32_t slim;              // floor(cap_milli * G * 3 / 1000): S + g <= slim is the cap test
  uint64_t *dlog;
  int32_t *ovf_dur;          // [n_sess] durations of queued cells whose timer is outside the registers
  // per-lane state
  int32_t fin[NJ];
  int32_t hr;                // ready_at of host = lane
  uint32_t hs;               // S | nrep << 16 of host = lane
  int32_t qt, qd;            // sorted timers, entry i in lane i
  uint32_t qk;
  // this lane's event in the current tile, if it is a cell of a placed session that is not ending and whose record nobody
  // has changed since but by starting cells at once: the session and its busy-until time (else ~0 and NEVER)
  uint32_t vsid;
  int32_t vtm;
  uint64_t digest;           // the same in all lanes, see decide_code
  int32_t fu;                // lane g-1 (g = 1..8): no host can have g idle GPUs before this time
  // closed loop: the replay's cursors, the events of the trace; and with every sorted timer what firing
  // it needs: qd = the event's index, qx = its duration | kind << 28 | CLX_LOADED (0: not loaded yet),
  // qnx / qnth = its chain record
  int32_t *cl_cur;
  const int32_t *cl_dur, *cl_sk;
  const int2 *cl_chain;
  int32_t qx, qnx, qnth;
  bool dyn;                  // the dynamic limit can differ from the replay's cap (see dynamic_limit_matters)
  int32_t latest;            // open loop: the latest finish among this lane's cells that started at once
  static constexpr bool closed = closed_loop_instance(F);
  __device__ __forceinline__ uint32_t flags() const { return instance_flags<F>(p); }
};

// A decision's code goes into the digest (and into the log). The digest is kept in vector registers, the same in all lanes:
// the scalar unit, which is what many small replays are bound by (with the scalar product 0.86 instructions a clock with 64
// of them on a compute unit), would take nine instructions for the 64-bit product, the vector side takes four. 24 hosts,
// 16,384 replays: 45.0 ms with the scalar product, 42.5 with this; 300 short replays 0.766 -> 0.744. (Codes kept in lanes and folded 64 at a
// time: 43.5, but 30 hosts 27.2 -> 31.3 and 64 hosts 64.6 -> 71.7, as every path then carries two more registers.)
template <int NJ, uint32_t F>
__device__ __forceinline__ void decide_code(Ctx<NJ, F> &c, Regs &r, int32_t now, uint32_t code_lo) {
  const uint64_t code = ((uint64_t)(uint32_t)now << 32) | code_lo, d = c.digest;
  static_assert(DIGEST_PRIME == (1ull << 40) + 0x1B3u, "the product below");
  uint64_t low = (uint64_t)(uint32_t)d * 0x1B3u + code;
  uint32_t high = (uint32_t)(low >> 32) + (uint32_t)(d >> 32) * 0x1B3u + ((uint32_t)d << 8);
  uint32_t keep = (uint32_t)low;
  asm volatile("" : "+v"(keep), "+v"(high));             // (uniform, but kept off the scalar unit)
  c.digest = ((uint64_t)high << 32) | keep;
  if (__builtin_expect(c.dlog != nullptr, 0)) {
    if ((int64_t)r.n_dec < c.p.dlog_stride) c.dlog[r.n_dec] = code;
  }
  r.n_dec++;
}
template <int NJ, uint32_t F>
__device__ __forceinline__ void decide(Ctx<NJ, F> &c, Regs &r, int32_t now, uint32_t outcome, uint32_t s, uint32_t slot, uint32_t host) {
  decide_code(c, r, now, host | (slot << 10) | (outcome << 12) | (s << 16));
}

// a session record has been written: lanes of the current tile that hold it go stale
template <int NJ, uint32_t F>
__device__ __forceinline__ void mark_stale(Ctx<NJ, F> &c, uint32_t s) {
  if constexpr (!Ctx<NJ, F>::closed) {
    const bool stale = c.vsid == s;
    c.vtm = stale ? NEVER : c.vtm;
    c.vsid = stale ? 0xFFFFFFFFu : c.vsid;
  }
}
template <int NJ, uint32_t F>
__device__ __forceinline__ void sess_write(Ctx<NJ, F> &c, uint32_t s, uint32_t hw, int32_t tm, uint32_t fl) {
  c.m.sess[s] = make_int2((int)((hw & ~RK_FLAGS) | (fl & RK_FLAGS)), tm);
  mark_stale(c, s);
}
template <int NJ, uint32_t F>
__device__ __forceinline__ void sess_write_flag(Ctx<NJ, F> &c, uint32_t s, uint32_t fl) {
  c.m.sess[s].x = (int)fl;
  mark_stale(c, s);
}

// ---- timers beyond the 64 sorted ones stay with their session -------------------------------------
// Such a session carries RK_OVF. Its timer is implied by its record: a queued session retries at
// submit time + retries * interval (the duration of its cell waits in a per-replay array in device
// memory), a placed session that is ending ends at its busy-until time. A lower bound of the earliest of them
// is tracked; when the registers run empty, refill() moves up to 64 of them in at once.
template <int NJ, uint32_t F>
__device__ __forceinline__ void ovf_push(Ctx<NJ, F> &c, Regs &r, int32_t t, uint32_t k, int32_t d) {
  const uint32_t s = k & 0xFFFFu;
  if constexpr (Ctx<NJ, F>::closed) {
    // the session's one timer waits in its record: a retry is implied by it as ever, the time of a
    // next event replaces the busy-until time (a closed loop never asks for it)
    wave_sync();
    const int2 rec = c.m.sess[s];
    c.m.sess[s] = make_int2(rec.x | (int)RK_OVF, (k >> 16) != QK_RETRY ? t : rec.y);
  } else {
    wave_sync();
    c.m.sess[s].x |= (int)RK_OVF;
    c.ovf_dur[s] = d;
  }
  mark_stale(c, s);
  if (r.o_n == 0 || t < r.o_min_t || (t == r.o_min_t && k < r.o_min_k)) { r.o_min_t = t; r.o_min_k = k; }
  r.o_n++;
}

// the time of the timer that waits in a session's record (a retry's is implied by it)
template <int NJ, uint32_t F>
__device__ __forceinline__ int32_t waiting_time(const Ctx<NJ, F> &c, const int2 rec) {
  const uint32_t fl = (uint32_t)rec.x;
  const int32_t at = retry_time(rec.y, (int32_t)((fl >> 8) & 15u), c.p.retry_iv);
  return (fl & 7u) == SS_QUEUED ? at : rec.y;
}

// Registers empty: all timers that are due within a window after the earliest one move
// from the session records into the registers at once, at most 64 (whole instants, so everything
// taken is earlier than everything left behind whatever the kinds; the window adapts to fill 32 to
// 56 registers; more than 64 timers at one instant: the single earliest), and what firing them will
// need is gathered one lane per timer. The same scheme as in the any-size kernel. The kind of a timer
// that is no retry: the deferred end of a busy session (open loop), the session's next event (closed loop).
template <int NJ, uint32_t F>
__device__ __forceinline__ void refill(Ctx<NJ, F> &c, Regs &r) {
  constexpr uint32_t kOther = Ctx<NJ, F>::closed ? QK_NEXT : QK_END;
  wave_sync();
  int cnt;
  int32_t staged = 0;                            // the sessions whose timers come in, one per lane
  int32_t left;                                  // earliest time left behind
  uint32_t left_k = 0;                           // ... and a lower bound of the keys left behind at that time
  int32_t win = r.cl_win;
  for (;;) {
    const int64_t lim = (int64_t)r.o_min_t + win;
    const int32_t T = lim < NEVER - 1 ? (int32_t)lim : NEVER - 1;
    cnt = 0;
    int32_t mn = NEVER;
    for (int s0 = 0; s0 < c.n_sess; s0 += WAVE) {
      const int s = s0 + c.lane;
      const int2 rec = c.m.sess[min(s, c.n_sess - 1)];
      const int32_t due = waiting_time(c, rec);
      const int32_t d = (s < c.n_sess) & (((uint32_t)rec.x & RK_OVF) != 0) ? due : NEVER;
      const bool hit = d <= T;
      const uint64_t b = wballot(hit);
      if (b != 0) {
        staged = cnt < WAVE ? stage_hits(staged, c.lane, cnt, hit, b, s) : staged;
        cnt += __builtin_popcountll(b);
      }
      mn = hit ? mn : (d < mn ? d : mn);
    }
    left = (int32_t)wave_min((uint32_t)mn);
    if (cnt == 0) {                              // the stored bound was below the earliest time: use that
      if (left == NEVER) { r.o_n = 0; r.o_min_t = NEVER; return; }      // nothing waits (not reached: o_n counts them)
      r.o_min_t = left;
      continue;
    }
    if (cnt <= WAVE) break;
    if (win == 0) {
      // more than 64 timers at the instant o_min_t: the earliest by kind and session alone
      wave_sync();
      uint32_t best = 0xFFFFFFFFu;
      for (int s0 = 0; s0 < c.n_sess; s0 += WAVE) {
        const int s = s0 + c.lane;
        const int2 rec = c.m.sess[min(s, c.n_sess - 1)];
        const uint32_t fl = (uint32_t)rec.x;
        const uint32_t k = (((fl & 7u) == SS_QUEUED ? QK_RETRY : kOther) << 16) | (uint32_t)s;
        const int32_t due = waiting_time(c, rec);
        best = umin(best, (s < c.n_sess) & ((fl & RK_OVF) != 0) & (due == T) ? k : 0xFFFFFFFFu);
      }
      best = wave_min(best);
      staged = (int32_t)(best & 0xFFFFu);
      cnt = 1;
      left = T;
      left_k = best;                             // (all that stay are later; a timer pushed before it belongs into the registers)
      break;
    }
    win = (int32_t)((int64_t)win * 40 / cnt);    // aim at 40 of the 64 registers
    wave_sync();
  }
  if (cnt < WAVE / 2 && win < CL_WIN_MAX) r.cl_win = win == 0 ? 1 : win + (win + 1) / 2;
  else if (cnt > 7 * WAVE / 8) r.cl_win = win - win / 4;
  else r.cl_win = win;
  wave_sync();
  // lane i < cnt takes the timer of the session staged there
  const bool take = c.lane < cnt;
  const int last_staged = lane_get(staged, cnt - 1);
  const int s = take ? staged : last_staged;                   // (the lanes beyond do what the last one does)
  const int2 rec = c.m.sess[s];
  const uint32_t fl = (uint32_t)rec.x;
  const int32_t due = waiting_time(c, rec);
  const int32_t t = take ? due : NEVER;
  const uint32_t own_key = (((fl & 7u) == SS_QUEUED ? QK_RETRY : kOther) << 16) | (uint32_t)s;
  const uint32_t key = take ? own_key : 0xFFFFFFFFu;
  int32_t e = 0;
  c.m.sess[s].x = (int)(fl & ~RK_OVF);
  // the cursors / durations were stored when the timers were scheduled, by whichever lane of this wave: the fence
  // orders those stores before the loads of the lanes that look at them now
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  int32_t x = 0, nx = -1, nth = 0;
  if constexpr (Ctx<NJ, F>::closed) {
    e = c.cl_cur[s];
    const int2 ch = c.cl_chain[e];
    x = c.cl_dur[e] | (int32_t)(((uint32_t)c.cl_sk[e] >> 24) << 28) | CLX_LOADED;
    nx = ch.x; nth = ch.y;
  } else {
    e = c.ovf_dur[s];                            // qd carries the queued cell's duration (of a deferred end: not looked at)
    // (the records taken have lost their mark: lanes of the tile with one of those sessions are stale, as it was queued or
    // ending when the tile was loaded or has become so since)
  }
  const int rank = timer_ranks(c.lane, cnt, t, key);
  const int dst = take ? rank : c.lane;          // a permutation: the timers taken in order, the rest where they are
  c.qt = __builtin_amdgcn_ds_permute(dst << 2, t);
  c.qk = (uint32_t)__builtin_amdgcn_ds_permute(dst << 2, (int)key);
  c.qd = __builtin_amdgcn_ds_permute(dst << 2, e);
  if constexpr (Ctx<NJ, F>::closed) {
    c.qx = __builtin_amdgcn_ds_permute(dst << 2, x);
    c.qnx = __builtin_amdgcn_ds_permute(dst << 2, nx);
    c.qnth = __builtin_amdgcn_ds_permute(dst << 2, nth);
  }
  r.q_n = cnt;
  r.o_n -= cnt;
  r.o_min_t = r.o_n > 0 ? left : NEVER;
  r.o_min_k = left_k;                            // a lower bound: pushes for that very instant wait in the records
}

// ---- hosts ----------------------------------------------------------------------------------------
// committed GPUs of host = lane at time `now` (those beyond G included): byte (lane & 7) of the ballot of register (lane >> 3)
template <int NJ, uint32_t F>
__device__ __forceinline__ int committed(const Ctx<NJ, F> &c, int32_t now) {
  const int sh = 8 * (c.lane & 7), grp = c.lane >> 3;
  uint32_t bits = 0;
#pragma unroll
  for (int j = 0; j < NJ; j++) {
    const uint64_t busy = wballot(c.fin[j] > now);
    const uint32_t mine = (uint32_t)(busy >> sh);
    bits = grp == j ? mine : bits;
  }
  return __builtin_popcount(bits & 0xFFu);
}

// The same on top of `more`, with the words of the busy GPUs kept for binding.
template <int NJ, uint32_t F>
__device__ __forceinline__ uint32_t committed_words(const Ctx<NJ, F> &c, int32_t now, uint32_t more, uint64_t (&busy)[NJ]) {
  const int sh = 8 * (c.lane & 7), grp = c.lane >> 3;
  uint32_t bits = 0;
#pragma unroll
  for (int j = 0; j < NJ; j++) {
    busy[j] = wballot(c.fin[j] > now);
    const uint32_t mine = (uint32_t)(busy[j] >> sh);
    bits = grp == j ? mine : bits;
  }
  return (uint32_t)__builtin_popcount(bits & 0xFFu) + more;
}
// bind g free GPUs of host h until `finish`
template <int NJ, uint32_t F>
__device__ __forceinline__ void bind_words(Ctx<NJ, F> &c, int h, int g, int32_t finish, const uint64_t (&busy)[NJ]) {
  const int j = h >> 3, hl = h & 7;
  const uint64_t mine = 0xFFull << (8 * hl);
#pragma unroll
  for (int jj = 0; jj < NJ; jj++) {
    if (jj == j) {
      const uint64_t fr = mine & ~busy[jj];
      const int rank = lane_rank(fr) | (in_mask(fr) ? 0 : WAVE);
      c.fin[jj] = rank < g ? finish : c.fin[jj];
      // (keeps the arms apart: merged into one store through a chosen pointer they put the rows into memory)
      asm volatile("; group %1" : "+v"(c.fin[jj]) : "n"(jj));
    }
  }
}

// The same for migrations and new hosts. On more than 40 hosts the one word that counts is made again (one comparison): two
// scalar registers per group of hosts, kept over the choice of a target, the pool and a new host for the sake of a few
// bindings, are spilled there. Lane reads of the closed loop's instances for 48 and 64 hosts 225 and 424 with the words,
// 158 and 206 with this; 4,096 replays of 48 hosts 6.16 -> 5.99 ms, of 64 hosts 6.15 -> 6.03, open loops the same. On 12
// hosts with scale-in, 2,048 replays, 3.05 ms with the words and 3.14 with this, on 40 hosts with closed loops 21.47 and 21.60.
template <int NJ, uint32_t F>
__device__ __forceinline__ void bind_late(Ctx<NJ, F> &c, int h, int g, int32_t finish, int32_t now, const uint64_t (&busy)[NJ]) {
  if constexpr (NJ <= 5) return bind_words(c, h, g, finish, busy);
  const int j = h >> 3, hl = h & 7;
  const uint64_t mine = 0xFFull << (8 * hl);
#pragma unroll
  for (int jj = 0; jj < NJ; jj++) {
    if (jj == j) {
      const uint64_t fr = mine & ~wballot(c.fin[jj] > now);
      const int rank = lane_rank(fr) | (in_mask(fr) ? 0 : WAVE);
      c.fin[jj] = rank < g ? finish : c.fin[jj];
      asm volatile("; group %1" : "+v"(c.fin[jj]) : "n"(jj));
    }
  }
}

// the ready hosts with g idle GPUs, one bit each (a host that is not ready counts as full; with two comparisons joined the
// scalar unit has to wait for both before the vector side can go on)
template <int NJ, uint32_t F>
__device__ __forceinline__ uint64_t hosts_with_idle(const Ctx<NJ, F> &c, int32_t now, int g) {
  uint64_t busy[NJ];
  return wballot((int)committed_words(c, now, c.hr <= now ? 0u : 16u, busy) <= NGPU - g);
}
// a session's three hosts, likewise
__device__ __forceinline__ uint64_t own_hosts(uint32_t hw) {
  return (1ull << slot_host(hw, 0)) | (1ull << slot_host(hw, 1)) | (1ull << slot_host(hw, 2));
}

template <int NJ, uint32_t F>
__device__ __forceinline__ int boot_host(Ctx<NJ, F> &c, Regs &r, int32_t now, uint32_t hs_new) {
  const uint64_t off = wballot((c.lane < c.p.Hmax) & (c.hr == NEVER));
  int h = (int)__builtin_ctzll(off);                 // the caller has checked that one exists
  int32_t ra = after(c, now, c.p.boot);
  if (c.lane == h) { c.hr = ra; c.hs = hs_new; }
  if (c.flags() & NBOS_F_WARM_POOL) {         // its pre-warmed containers are there once it is up
    c.m.warm[4 * h + (c.lane & 3)] = after(c, ra, c.p.prewarm);
  }
  c.fu = c.fu < ra ? c.fu : ra;               // a new host may have idle GPUs from then on
  c32_add(c.m, c.lane, CS_NON, 1u);
  c64_add(c.m, c.lane, CL_PROV, -(int64_t)c.p.G * now);
  c32_add(c.m, c.lane, CS_SO, 1u);
  r.lazy_max = r.lazy_max > ra ? r.lazy_max : ra;
  return h;
}

// Earliest time at which some host that is on could have g idle GPUs if nothing new were committed:
// min over hosts of max(ready_at, g-th smallest busy-until time of the host's GPUs). Later commits
// only push it back, so no election or migration for a request of g GPUs can succeed before it
// (as long as no host is added). Each lane counts, inside its host's group of 8 lanes, the GPUs that
// are free no later than its own GPU (DPP quad rotations of the value and of its half-row mirror
// reach all 8 lanes of the group). hosts: the hosts that are looked at, one bit each.
template <int NJ, uint32_t F>
__device__ __forceinline__ int32_t earliest_idle(const Ctx<NJ, F> &c, int g, uint64_t hosts = ~0ull) {
  int32_t best = NEVER;
#pragma unroll
  for (int j = 0; j < NJ; j++) {
    const int32_t f = c.fin[j];
    const int32_t mir = __builtin_amdgcn_update_dpp(f, f, 0x141, 0xF, 0xF, false);   // row_half_mirror
    int cnt = 1;
    cnt += __builtin_amdgcn_update_dpp(f, f, 0x39, 0xF, 0xF, false) <= f ? 1 : 0;      // quad_perm [1,2,3,0]
    cnt += __builtin_amdgcn_update_dpp(f, f, 0x4E, 0xF, 0xF, false) <= f ? 1 : 0;      // quad_perm [2,3,0,1]
    cnt += __builtin_amdgcn_update_dpp(f, f, 0x93, 0xF, 0xF, false) <= f ? 1 : 0;      // quad_perm [3,0,1,2]
    cnt += mir <= f ? 1 : 0;
    cnt += __builtin_amdgcn_update_dpp(mir, mir, 0x39, 0xF, 0xF, false) <= f ? 1 : 0;
    cnt += __builtin_amdgcn_update_dpp(mir, mir, 0x4E, 0xF, 0xF, false) <= f ? 1 : 0;
    cnt += __builtin_amdgcn_update_dpp(mir, mir, 0x93, 0xF, 0xF, false) <= f ? 1 : 0;
    const int32_t ra = __builtin_amdgcn_ds_bpermute((8 * j + (c.lane >> 3)) << 2, c.hr);  // ready_at of host 8j+hl
    const bool in = (((uint32_t)(hosts >> (8 * j)) >> (c.lane >> 3)) & 1u) != 0;
    int32_t y = (cnt >= g) & in ? f : NEVER;
    y = y > ra ? y : ra;
    best = best < y ? best : y;
  }
  return (int32_t)wave_min((uint32_t)best);
}

// No retry of a queued cell before this time can succeed, whatever happens until then (if no host can be added). Where
// cells do not migrate either, only the session's own three hosts can take it, and they have the GPUs idle no earlier
// than their busy-until times as they stand. Working that out takes about 20 instructions per group of 8 hosts, a retry
// that fails 120. One small cluster (8 hosts, 2,000 cells), create to destroy: 1.206 -> 1.148 ms.
template <int NJ, uint32_t F>
__device__ __forceinline__ int32_t retry_bound(const Ctx<NJ, F> &c, uint32_t hw, int g) {
  int32_t bound = lane_get(c.fu, g - 1);
  if (!(c.flags() & (NBOS_F_MIGRATE | NBOS_F_SCALE_OUT))) {
    bound = max(bound, earliest_idle(c, g, own_hosts(hw)));
  }
  return bound;
}

// ---- closed loop: the session's next event is due one think time after `base` --------------------
// r.cl_nx / r.cl_nth: the event after the one being handled and the think time before it. The timer
// carries the event's index; the cursor keeps it for the time the timer waits outside the registers.
template <int NJ, uint32_t F>
__device__ __forceinline__ void cl_schedule(Ctx<NJ, F> &c, Regs &r, uint32_t s, int32_t base) {
  const int32_t e = r.cl_nx;
  if (e < 0) return;
  const int64_t t = (int64_t)base + r.cl_nth;
  if (t >= 0x7FFFFFFFLL) { r.status = NBOS_E_RANGE; return; }
  c.cl_cur[s] = e;
  timer_push(c, r, (int32_t)t, QK_NEXT, s, e);
}

// ---- SESSION_START: Sections 3.2.1, 3.4.1, 3.4.2 -----------------------------------------------
template <int NJ, uint32_t F>
__device__ __forceinline__ void session_start(Ctx<NJ, F> &c, Regs &r, uint32_t s, uint32_t fl, int32_t now) {
  if ((fl & 7u) != SS_UNPLACED) return;
  const int g = (int)((fl >> 3) & 7u) + 1;
  const int C = committed(c, now);
  const int S = (int)(c.hs & 0xFFFFu);
  const int32_t room = cap_room(c, g);
  uint32_t key = (c.hr <= now) & (S <= room) ? (((uint32_t)C << 22) | ((uint32_t)S << 10) | (uint32_t)c.lane)
                                            : 0xFFFFFFFFu;
  int pick0 = -1, pick1 = -1, pick2 = -1, k = 0;
  uint32_t m0 = wave_min(key);
  if (m0 != 0xFFFFFFFFu) {
    pick0 = (int)(m0 & 1023u); k = 1;
    key = c.lane == pick0 ? 0xFFFFFFFFu : key;
    uint32_t m1 = wave_min(key);
    if (m1 != 0xFFFFFFFFu) {
      pick1 = (int)(m1 & 1023u); k = 2;
      key = c.lane == pick1 ? 0xFFFFFFFFu : key;
      uint32_t m2 = wave_min(key);
      if (m2 != 0xFFFFFFFFu) { pick2 = (int)(m2 & 1023u); k = 3; }
    }
  }
  const int missing = 3 - k;
  if (missing > 0) {
    wave_sync();
    int n_on = (int)uni(c.m.c32[CS_NON]);
    if (!((c.flags() & NBOS_F_SCALE_OUT) && n_on + missing <= c.p.Hmax)) {
      sess_write_flag(c, s, (fl & ~7u) | SS_REJECTED);
      c32_add(c.m, c.lane, CS_REJECTED, 1u);
      decide(c, r, now, NBOS_D_REJECT, s, 0, 0);
      return;
    }
  }
  const uint32_t add = (uint32_t)g | (1u << 16);
  uint32_t hw = 0;
#pragma unroll
  for (int i = 0; i < 3; i++) {
    int h = i == 0 ? pick0 : (i == 1 ? pick1 : pick2);
    if (i < k) {
      if (c.lane == h) c.hs += add;
      decide(c, r, now, NBOS_D_PLACE, s, (uint32_t)i, (uint32_t)h);
    } else {
      h = boot_host(c, r, now, add);
      decide(c, r, now, NBOS_D_PLACE_NEW, s, (uint32_t)i, (uint32_t)h);
    }
    hw |= (uint32_t)h << (12 + 6 * i);
  }
  if (missing > 0) {
    wave_sync();
    c32_max(c.m, c.lane, CS_PEAK, uni(c.m.c32[CS_NON]));
  }
  sess_write(c, s, hw, 0, (fl & ~7u) | SS_PLACED);
  c32_add(c.m, c.lane, CS_PLACED, 1u);
  c32_add(c.m, c.lane, CS_SUMS, (uint32_t)(3 * g));
  c32_add(c.m, c.lane, CS_OPENG, (uint32_t)g);
  c64_add(c.m, c.lane, CL_SUB, -(int64_t)(3 * g) * now);
  c64_add(c.m, c.lane, CL_RESV, -(int64_t)g * now);
  c32_add(c.m, c.lane, CS_NREP, 3u);
  c64_add(c.m, c.lane, CL_REPL, -(int64_t)3 * now);
  if constexpr (Ctx<NJ, F>::closed) cl_schedule(c, r, s, now);
}

// the replicas of session s give their subscriptions back at time `now`
template <int NJ, uint32_t F>
__device__ __forceinline__ void end_session(Ctx<NJ, F> &c, Regs &r, uint32_t s, uint32_t hw, uint32_t fl, int32_t now) {
  const int g = (int)((fl >> 3) & 7u) + 1;
  const uint32_t sub = (uint32_t)g | (1u << 16);
  const int h0 = (int)slot_host(hw, 0), h1 = (int)slot_host(hw, 1), h2 = (int)slot_host(hw, 2);
  c.hs -= (c.lane == h0) | (c.lane == h1) | (c.lane == h2) ? sub : 0u;
  sess_write_flag(c, s, (fl & ~(7u | SF_ENDING)) | SS_ENDED);
  c32_add(c.m, c.lane, CS_SUMS, (uint32_t)(-3 * g));
  c64_add(c.m, c.lane, CL_SUB, (int64_t)(3 * g) * now);
  c32_add(c.m, c.lane, CS_NREP, (uint32_t)-3);
  c64_add(c.m, c.lane, CL_REPL, (int64_t)3 * now);
}

// ---- a cell starts on (slot, host): Section 3.3 and the metrics of sections "Resource Usage & Efficiency", "Interactivity" and "Task Completion Time" ---------
template <int NJ, uint32_t F>
__device__ __forceinline__ void start_cell(Ctx<NJ, F> &c, Regs &r, uint32_t s, uint32_t hw, uint32_t fl, int slot, int host,
                                           int32_t now, int32_t start, int32_t t_submit, int32_t dur,
                                           uint32_t outcome) {
  const int g = (int)((fl >> 3) & 7u) + 1;
  if constexpr (Ctx<NJ, F>::closed) {         // the lag of a closed loop is not bounded in advance
    if ((int64_t)start + dur >= 0x7FFFFFFFLL) { r.status = NBOS_E_RANGE; return; }
  }
  const int32_t finish = start + dur;
  const int32_t delay = start - t_submit;
  r.c_started++;
  r.sum_dur += dur;
  r.g_exec += (int64_t)g * dur;
  const uint32_t last = hw >> 30;               // 0 none, else slot + 1
  if (last == (uint32_t)slot + 1u) r.reused++;
  hw = (hw & 0x3FFFFFFFu) | ((uint32_t)(slot + 1) << 30);
  hw = (hw & ~(63u << (12 + 6 * slot))) | ((uint32_t)host << (12 + 6 * slot));
  // the record's word: hosts and last executor from hw, state back to "placed", retry count cleared
  const uint32_t nw = (hw & ~RK_FLAGS) | (((fl & ~(7u | (15u << 8))) | SS_PLACED) & RK_FLAGS);
  if (__builtin_expect(delay == 0, 1)) {
    r.h0++;                                     // histogram bin 0 lives in a register
  } else {
    hist_add(c.m, c.lane, delay);
    c64_add(c.m, c.lane, CL_SUMDELAY, delay);
    c32_max(c.m, c.lane, CS_MAXDELAY, (uint32_t)delay);
    c64_add(c.m, c.lane, CL_GWAIT, (int64_t)g * (start - now));
  }
  c.m.sess[s] = make_int2((int)nw, finish);
  mark_stale(c, s);
  r.lazy_max = r.lazy_max > finish ? r.lazy_max : finish;
  decide(c, r, now, outcome, s, (uint32_t)slot, (uint32_t)host);
  if (__builtin_expect((fl & SF_ENDING) != 0, 0)) timer_push(c, r, finish, QK_END, s, 0);
  if constexpr (Ctx<NJ, F>::closed) cl_schedule(c, r, s, finish);
}

// ---- executor election, Section 3.2.2 ----------------------------------------------------------------
// key: per lane = host, (committed GPUs, and 16 more where the host is not ready) << 8 | host << 2. Among the session's three
// hosts: fewest committed GPUs, then lowest host index, i.e. the smallest of their keys; where that one has too few GPUs
// idle, all have. Returns it with the replica's slot in its low two bits; (key >> 8) + g <= 8 if it can bind.
// (Used by attempts and retries as well as by the loop of starts, with the busy words kept for binding, in place of keys
// masked by two joined comparisons: 30 hosts 27.3 -> 26.4 ms, closed loops on 30 hosts 55.2 -> 54.1.)
template <int NJ, uint32_t F>
__device__ __forceinline__ uint32_t elect_slot(const Ctx<NJ, F> &c, uint32_t hw, uint32_t key, int g) {
  const uint32_t k0 = (uint32_t)lane_get((int)key, (int)slot_host(hw, 0)), k1 = (uint32_t)lane_get((int)key, (int)slot_host(hw, 1)) | 1u,
                 k2 = (uint32_t)lane_get((int)key, (int)slot_host(hw, 2)) | 2u;
  // (two scalar minima: left alone, the compiler makes one three-way minimum on the vector side, with the way there and back)
  uint32_t kb = umin(k0, (uint32_t)fresh((int)umin(k1, k2)));
  if (c.flags() & NBOS_F_STICKY_EXECUTOR) {
    const uint32_t last = hw >> 30;
    const uint32_t kp = last == 1u ? k0 : (last == 2u ? k1 : (last == 3u ? k2 : 0xFFFFFFFFu));
    if ((int)(kp >> 8) + g <= NGPU) kb = kp;
  }
  return kb;
}

// A cell of an idle placed session starts by election at the instant it is submitted (open loop): what
// start_cell does for a delay of 0, with nothing of the other cases in it. The cell's lane is marked in r.at_once:
// the sums that nobody reads during the replay are made from those marks once per tile (see fold_starts). code: the
// session and the outcome in their places of the decision code.
template <int NJ, uint32_t F>
__device__ __forceinline__ void start_at_once(Ctx<NJ, F> &c, Regs &r, int32_t &vhw, uint32_t code, uint32_t hw, uint32_t slot, uint32_t host,
                                              int32_t now, int32_t finish) {
  const uint32_t s = code >> 16;
  r.reused += (hw >> 30) == slot + 1u ? 1u : 0u;
  // the record's word: hosts as they are, this slot the last executor; state "placed", retry count 0 already
  const uint32_t nw = (hw & 0x3FFFFFFFu) | ((slot + 1u) << 30);
  c.m.sess[s] = make_int2((int)nw, finish);
  const bool same = c.vsid == s;
  vhw = same ? (int32_t)nw : vhw;
  c.vtm = same ? finish : c.vtm;
  decide_code(c, r, now, host | (slot << 10) | code);
}

// The tile's cells that started at once (lanes of r.at_once), all at a time: counts on the scalar unit, durations,
// GPU time added up by the LDS unit, the latest finish per lane. fl: the word of the prefetched record (a session's g never changes). In the
// loop of starts, bound by the number of its instructions (a lone wave takes 7 clocks for each), these sums were
// fourteen of 165. Taken out of it, together with other cuts of the same kind: 24 hosts 50.2 -> 47.2 ms (16,384 replays of
// 20,000 cells), 300 short replays 0.90 -> 0.85, 64 hosts 71.7 -> 69.9.
template <int NJ, uint32_t F>
__device__ __forceinline__ void fold_starts(Ctx<NJ, F> &c, Regs &r, int32_t vt, int32_t vd, uint32_t fl) {
  const uint32_t n = (uint32_t)__builtin_popcountll(r.at_once);
  r.c_started += n; r.c_imm += n; r.h0 += n;
  const uint32_t d = in_mask(r.at_once) ? (uint32_t)vd : 0u;       // (8 * NBOS_MAX_DUR_MS is below 2^32)
  atomicAdd(&c.m.c64[CL_BDUR], (unsigned long long)d);
  atomicAdd(&c.m.c64[CL_BGEXEC], (unsigned long long)((((fl >> 3) & 7u) + 1u) * d));
  c.latest = max(c.latest, in_mask(r.at_once) ? vt + vd : 0);
  r.at_once = 0;
}

// ---- one attempt to run the pending cell of session s at time `now` -----------------------------
template <int NJ, uint32_t F>
__device__ __forceinline__ void attempt(Ctx<NJ, F> &c, Regs &r, uint32_t s, uint32_t hw, uint32_t fl, int32_t now,
                                        int32_t t_submit, int32_t dur) {
  const int g = (int)((fl >> 3) & 7u) + 1;
  const uint32_t h0 = slot_host(hw, 0), h1 = slot_host(hw, 1), h2 = slot_host(hw, 2);
  // Known in advance that no host has g idle GPUs yet? Then neither election nor migration can work.
  const bool hopeless = now < lane_get(c.fu, g - 1);
  uint32_t Cx = 0;                                  // committed GPUs, and 16 more where the host is not ready
  uint64_t busy[NJ] = {}, idle_ok = 0;
  uint32_t kb = 0xFFFFFFFFu;
  if (!hopeless) {
    Cx = committed_words(c, now, c.hr <= now ? 0u : 16u, busy);
    idle_ok = wballot((int)Cx <= NGPU - g);          // ready hosts with g idle GPUs
    // (a) election, Section 3.2.2: among the session's hosts that can bind, fewest committed GPUs, then
    // lowest host index: the smallest of the three hosts' keys
    kb = elect_slot(c, hw, (Cx << 8) | ((uint32_t)c.lane << 2), g);
  }
  if ((int)(kb >> 8) <= NGPU - g) {
    const int hl = (int)((kb >> 2) & 63u), lead = (int)(kb & 3u);
    bind_words(c, hl, g, wrap_add(now, dur), busy);       // (out of range: start_cell ends the replay)
    if (now == t_submit) r.c_imm++;
    start_cell(c, r, s, hw, fl, lead, hl, now, now, t_submit, dur, NBOS_D_START);
    return;
  }
  // No host at all with g idle GPUs: work out when the first one could have them, once, for every
  // later attempt with a request of g or more (commits only push that time back; a booted host
  // lowers it again, see boot_host).
  if (!hopeless && idle_ok == 0) {
    const int32_t bound = earliest_idle(c, g);
    c.fu = (c.lane >= g - 1) & (c.fu < bound) ? bound : c.fu;
  }
  // (b), (c): a target exists? Only then is the replica to move worked out: the one on the fullest
  // ready host (ties: lowest host); replicas on booting hosts only if all three are.
  const int S = (int)(c.hs & 0xFFFFu);
  uint64_t target = 0;
  if ((c.flags() & NBOS_F_MIGRATE) && idle_ok != 0) target = idle_ok & wballot(S <= cap_room(c, g));
  bool grow = false;
  if (target == 0 && (c.flags() & NBOS_F_SCALE_OUT)) {
    wave_sync();
    grow = (int)uni(c.m.c32[CS_NON]) < c.p.Hmax;
  }
  if (target != 0 || grow) {
    if (hopeless) Cx = committed_words(c, now, c.hr <= now ? 0u : 16u, busy);
    const int x0 = lane_get((int)Cx, (int)h0), x1 = lane_get((int)Cx, (int)h1), x2 = lane_get((int)Cx, (int)h2);
    const int C0 = x0 & 15, C1 = x1 & 15, C2 = x2 & 15;
    const int ok0 = x0 < 16 ? 1 : 0, ok1 = x1 < 16 ? 1 : 0, ok2 = x2 < 16 ? 1 : 0;
    const int any_ready = ok0 | ok1 | ok2;
    const uint32_t v0 = (!any_ready || ok0) ? (((uint32_t)(8 - C0) << 12) | (h0 << 2) | 0u) : 0xFFFFFFFFu;
    const uint32_t v1 = (!any_ready || ok1) ? (((uint32_t)(8 - C1) << 12) | (h1 << 2) | 1u) : 0xFFFFFFFFu;
    const uint32_t v2 = (!any_ready || ok2) ? (((uint32_t)(8 - C2) << 12) | (h2 << 2) | 2u) : 0xFFFFFFFFu;
    const uint32_t vb = umin(v0, umin(v1, v2));
    const int victim = (int)(vb & 3u), hv = (int)((vb >> 2) & 1023u);
    const uint32_t moved = (uint32_t)g | (1u << 16);
    if (target != 0) {
      // (b) migration, Section 3.2.3: the target binds the GPUs at once. A ready host of this session
      // with g idle GPUs would have won the election, so none of its hosts can show up as a target.
      const uint32_t key = in_mask(target) ? ((Cx << 22) | ((uint32_t)S << 10) | (uint32_t)c.lane)
                                                      : 0xFFFFFFFFu;
      const int dst = (int)(wave_min(key) & 1023u);
      bool warm = false;
      if (c.flags() & NBOS_F_WARM_POOL) {
        // Section 3.2.3: the target's pre-warmed container that has been available longest, if any
        // is available now, shortens the start; its replacement is there one pre-warm time later
        wave_sync();
        const uint32_t av_own = (uint32_t)c.m.warm[4 * dst + (c.lane & 3)];
        const uint32_t av = c.lane < c.p.warm_n ? av_own : 0xFFFFFFFFu;
        const uint32_t first = wave_min(av);
        if ((int32_t)first <= now) {
          const int w = (int)__builtin_ctzll(wballot(av == first));
          c.m.warm[4 * dst + w] = after(c, now, c.p.prewarm);
          c32_add(c.m, c.lane, CS_MIGRWARM, 1u);
          warm = true;
        }
      }
      if (c.lane == hv) c.hs -= moved;
      if (c.lane == dst) c.hs += moved;
      c32_add(c.m, c.lane, CS_MIGR, 1u);
      if (warm) {
        const int32_t start = after(c, now, c.p.warm_migr);
        bind_late(c, dst, g, wrap_add(start, dur), now, busy);
        start_cell(c, r, s, hw, fl, victim, dst, now, start, t_submit, dur, NBOS_D_MIGRATE_WARM);
      } else {
        const int32_t start = after(c, now, c.p.migr);
        bind_late(c, dst, g, wrap_add(start, dur), now, busy);
        start_cell(c, r, s, hw, fl, victim, dst, now, start, t_submit, dur, NBOS_D_MIGRATE);
      }
    } else {
      // (c) a new host for the cell, Section 3.4.2: reserved and bound before it is up
      const int32_t start = after(c, after(c, now, c.p.boot), c.p.migr);
      if (c.lane == hv) c.hs -= moved;
      const int h = boot_host(c, r, now, moved);
      wave_sync();
      c32_max(c.m, c.lane, CS_PEAK, uni(c.m.c32[CS_NON]));
      bind_late(c, h, g, wrap_add(start, dur), now, busy);       // (a host that was off has all its GPUs idle)
      c32_add(c.m, c.lane, CS_MIGR, 1u);
      start_cell(c, r, s, hw, fl, victim, h, now, start, t_submit, dur, NBOS_D_SCALE_CELL);
    }
    return;
  }
  // (d) queue and retry periodically, then give up, Section 3.2.3
  int retries = (int)((fl >> 8) & 15u);
  if (retries < c.p.max_retries) {
    const bool first = retries == 0;             // an arrival comes in with the count at 0, a retry never
    retries++;
    // A retry that is bound to fail only bumps the retry count: skip straight to the first retry
    // that could succeed (or to the last one, which aborts). Valid while no host can be added:
    // not with the periodic auto-scaler, and not when hosts can be both released and provisioned.
    if (!(c.flags() & NBOS_F_AUTOSCALE) &&
        (c.flags() & (NBOS_F_SCALE_IN | NBOS_F_SCALE_OUT)) != (NBOS_F_SCALE_IN | NBOS_F_SCALE_OUT)) {
      const int32_t bound = retry_bound(c, hw, g);
      while (retries < c.p.max_retries && t_submit + retries * c.p.retry_iv < bound) retries++;
    }
    const uint32_t nfl = (fl & ~(7u | (15u << 8))) | SS_QUEUED | ((uint32_t)retries << 8);
    if (first) {                                 // first time in the queue: the submit time goes in
      c32_add(c.m, c.lane, CS_QUEUED, 1u);
      c.m.sess[s] = make_int2((int)nfl, t_submit);
    } else {
      c.m.sess[s].x = (int)nfl;
    }
    mark_stale(c, s);
    if constexpr (Ctx<NJ, F>::closed) {
      // every timer carries its event (the cursor still points at the cell under way)
      if ((int64_t)t_submit + (int64_t)retries * c.p.retry_iv >= 0x7FFFFFFFLL) { r.status = NBOS_E_RANGE; return; }
      timer_push(c, r, t_submit + retries * c.p.retry_iv, QK_RETRY, s, r.cl_e, r.cl_x, r.cl_nx, r.cl_nth);
    } else {
      timer_push(c, r, t_submit + retries * c.p.retry_iv, QK_RETRY, s, dur);
    }
    return;
  }
  c32_add(c.m, c.lane, CS_ABORTED, 1u);
  decide(c, r, now, NBOS_D_ABORT, s, 0, 0);
  const uint32_t nfl = (fl & ~(7u | (15u << 8))) | SS_PLACED;
  sess_write(c, s, hw, 0, nfl);
  if (fl & SF_ENDING) end_session(c, r, s, hw, nfl, now);
  if constexpr (Ctx<NJ, F>::closed) cl_schedule(c, r, s, now);
}

// ---- runs of retries that fail again ---------------------------------------------------------------
// On a saturated cluster most timers are retries of queued cells (Section 3.2.3) that fail once more:
// no replica's host can bind the GPUs, no migration target, no host to add. Such an attempt changes
// nothing but the session's retry count and its place in the timer queue. This loop takes due
// retries off the head of the sorted registers for as long as they are of that kind (same tests as
// attempt(), same order), re-inserting each with one pass over the registers; the first timer that
// needs anything else is left for the general path. A retry that fails with no retries left gives its
// cell up right here. t_limit = time of the next arrival (timers due
// at or before it run first), tick_t = next auto-scaler period (a timer due at the same time runs
// before it). Returns the time of the last retry handled, or -1. CROWDED: timers are waiting in the session
// records as well (more than 64 pending); a retry that is then no longer earlier than all of those goes to
// wait there too, and the registers are refilled when they run empty. Two instances, so that the common
// case keeps its shorter loop.
template <bool CROWDED, int NJ, uint32_t F>
__device__ __forceinline__ int32_t failing_retries(Ctx<NJ, F> &c, Regs &r, int32_t t_limit, int32_t tick_t) {
  int32_t last = -1;
  const int32_t due = t_limit < tick_t ? t_limit : tick_t;
  const bool may_skip = !(c.flags() & NBOS_F_AUTOSCALE) &&
                        (c.flags() & (NBOS_F_SCALE_IN | NBOS_F_SCALE_OUT)) != (NBOS_F_SCALE_IN | NBOS_F_SCALE_OUT);
  while (r.q_n > 0 && (CROWDED || r.o_n == 0) && r.q_head_t <= due) {
    const int32_t now = r.q_head_t;
    const uint32_t key = (uint32_t)lane_get((int)c.qk, 0);
    if ((key >> 16) != QK_RETRY) break;
    const uint32_t s = key & 0xFFFFu;
    wave_sync();
    const int2 rec = c.m.sess[s];
    const uint32_t hw = uni((uint32_t)rec.x), fl = hw;
    const int32_t t_submit = uni(rec.y);
    int retries = (int)((fl >> 8) & 15u);
    const bool give_up = retries >= c.p.max_retries;           // no retry left: the cell is aborted
    if (give_up && (fl & SF_ENDING)) break;                    // ... and the session ends: general path
    const int g = (int)((fl >> 3) & 7u) + 1;
    if (now >= lane_get(c.fu, g - 1)) {
      const uint64_t idle_ok = hosts_with_idle(c, now, g);
      if (idle_ok & own_hosts(hw)) break;                                           // the election succeeds
      if (idle_ok == 0) {
        const int32_t bound = earliest_idle(c, g);
        c.fu = (c.lane >= g - 1) & (c.fu < bound) ? bound : c.fu;
      } else if (c.flags() & NBOS_F_MIGRATE) {
        const int S = (int)(c.hs & 0xFFFFu);
        if (idle_ok & wballot(S <= cap_room(c, g))) break;                        // a migration target
      }
    }
    if (c.flags() & NBOS_F_SCALE_OUT) {
      wave_sync();
      if ((int)uni(c.m.c32[CS_NON]) < c.p.Hmax) break;                            // a host can be added
    }
    last = now;
    if (__builtin_expect(give_up, 0)) {
      // it fails for the last time: the cell is given up, the session is idle again, the timer goes
      c32_add(c.m, c.lane, CS_ABORTED, 1u);
      decide(c, r, now, NBOS_D_ABORT, s, 0, 0);
      c.m.sess[s] = make_int2((int)((fl & ~(7u | (15u << 8))) | SS_PLACED), 0);
      mark_stale(c, s);
      c.qt = __builtin_amdgcn_update_dpp(c.qt, c.qt, 0x130, 0xF, 0xF, false);                      // wave_shl:1
      c.qd = __builtin_amdgcn_update_dpp(c.qd, c.qd, 0x130, 0xF, 0xF, false);
      c.qk = (uint32_t)__builtin_amdgcn_update_dpp((int)c.qk, (int)c.qk, 0x130, 0xF, 0xF, false);
      r.q_n--;
      if constexpr (CROWDED) { if (r.q_n == 0 && r.o_n > 0) refill(c, r); }
      r.q_head_t = r.q_n > 0 ? lane_get(c.qt, 0) : NEVER;
      continue;
    }
    // it fails again: bump the retry count (skipping retries that are bound to fail as well) ...
    retries++;
    if (may_skip) {
      const int32_t bound = retry_bound(c, hw, g);
      while (retries < c.p.max_retries && t_submit + retries * c.p.retry_iv < bound) retries++;
    }
    const uint32_t nfl = (fl & ~(15u << 8)) | ((uint32_t)retries << 8);
    c.m.sess[s].x = (int)nfl;
    mark_stale(c, s);
    // ... and move the entry from lane 0 to its new place: entries before it shift down one lane
    const int32_t t_new = t_submit + retries * c.p.retry_iv;
    const int32_t st = __builtin_amdgcn_update_dpp(c.qt, c.qt, 0x130, 0xF, 0xF, false);          // wave_shl:1
    const int32_t sd = __builtin_amdgcn_update_dpp(c.qd, c.qd, 0x130, 0xF, 0xF, false);
    const uint32_t sk = (uint32_t)__builtin_amdgcn_update_dpp((int)c.qk, (int)c.qk, 0x130, 0xF, 0xF, false);
    const int32_t d_own = lane_get(c.qd, 0);
    if constexpr (CROWDED) {
      if (r.o_n > 0 && !(t_new < r.o_min_t || (t_new == r.o_min_t && key < r.o_min_k))) {
        // no longer earlier than all that waits in the records: the timer goes there, off the registers
        ovf_push(c, r, t_new, key, d_own);
        c.qt = st; c.qd = sd; c.qk = sk;
        r.q_n--;
        if (r.q_n == 0 && r.o_n > 0) refill(c, r);
        r.q_head_t = r.q_n > 0 ? lane_get(c.qt, 0) : NEVER;
        continue;
      }
    }
    const bool before = (c.lane >= 1) & (c.lane < r.q_n) & ((c.qt < t_new) | ((c.qt == t_new) & (c.qk < key)));
    const int pos = __builtin_popcountll(wballot(before));
    const bool down = c.lane < pos, here = c.lane == pos;
    c.qt = here ? t_new : down ? st : c.qt;   c.qd = here ? d_own : down ? sd : c.qd;   c.qk = here ? key : down ? sk : c.qk;
    r.q_head_t = lane_get(c.qt, 0);
  }
  return last;
}

// ---- auto-scaler period (Section 3.4.2) -----------------------------------------------------------
// release the highest-numbered ready host without replicas
template <int NJ, uint32_t F>
__device__ __forceinline__ void release_host(Ctx<NJ, F> &c, Regs &r, int32_t now) {
  const uint64_t e = wballot((c.hr <= now) & ((c.hs >> 16) == 0));
  const int victim = 63 - (int)__builtin_clzll(e);
  if (c.lane == victim) c.hr = NEVER;
  c32_add(c.m, c.lane, CS_NON, (uint32_t)-1);
  c64_add(c.m, c.lane, CL_PROV, (int64_t)c.p.G * now);
  c32_add(c.m, c.lane, CS_SI, 1u);
  decide(c, r, now, NBOS_D_SCALE_IN, 0, 0, (uint32_t)victim);
}

template <int NJ, uint32_t F>
__device__ __forceinline__ void tick(Ctx<NJ, F> &c, Regs &r, int32_t now) {
  int A = __builtin_popcountll(wballot(c.hr <= now));
  int Z = __builtin_popcountll(wballot((c.hr <= now) & ((c.hs >> 16) == 0)));
  int released = 0;
  if (c.flags() & NBOS_F_AUTOSCALE) {
    // expected capacity f * sum C in whole hosts plus the scaling buffer; hosts being provisioned
    // count as capacity
    uint32_t sum_c = 0;
#pragma unroll
    for (int j = 0; j < NJ; j++) sum_c += (uint32_t)__builtin_popcountll(wballot(c.fin[j] > now));
    sum_c -= (uint32_t)(8 * NJ * (NGPU - c.p.G));            // (GPUs that are not there)
    const uint32_t per_host = 1000u * (uint32_t)c.p.G;
    const int want = (int)(((uint32_t)c.p.f_milli * sum_c + per_host - 1u) / per_host) + c.p.buffer;
    wave_sync();
    int n_on = (int)uni(c.m.c32[CS_NON]);
    const int before = n_on;
    while (n_on < want && n_on < c.p.Hmax) {
      const int h = boot_host(c, r, now, 0u);
      n_on++;
      decide(c, r, now, NBOS_D_SCALE_AUTO, 0, 0, (uint32_t)h);
    }
    if (n_on != before) c32_max(c.m, c.lane, CS_PEAK, (uint32_t)n_on);
    if (c.flags() & NBOS_F_SCALE_IN) {
      while (n_on > want && Z > 0 && A > c.p.min_hosts && released < 2) {
        release_host(c, r, now);
        n_on--; A--; Z--; released++;
      }
    }
    return;
  }
  // without the capacity test: release at most two hosts while too large a share of them is empty
  while ((int64_t)Z * 100 > (int64_t)A * c.p.idle_pct && A > c.p.min_hosts && released < 2) {
    release_host(c, r, now);
    A--; Z--; released++;
  }
}

template <int NJ, uint32_t F>
__device__ __forceinline__ void on_session_end(Ctx<NJ, F> &c, Regs &r, uint32_t s, uint32_t hw, int32_t tm, uint32_t fl,
                                               int32_t now) {
  const uint32_t st = fl & 7u;
  if ((st != SS_PLACED && st != SS_QUEUED) || (fl & SF_ENDING)) return;
  const int g = (int)((fl >> 3) & 7u) + 1;
  c32_add(c.m, c.lane, CS_OPENG, (uint32_t)-g);         // the Reservation lifetime closes at the END event
  c64_add(c.m, c.lane, CL_RESV, (int64_t)g * now);
  if (st == SS_PLACED && tm <= now) {
    end_session(c, r, s, hw, fl, now);
  } else {
    sess_write_flag(c, s, fl | SF_ENDING);
    if (st == SS_PLACED) timer_push(c, r, tm, QK_END, s, 0);
  }
}

// ---- closed-loop kernel: LDS layout of one replay and its initial state (S0) ---------------------------
// (the open-loop kernel below has both written out in its prologue: sharing them cost it 0.7 %)
__device__ __forceinline__ Lds lds_carve_closed(const KParams &p, unsigned char *q) {
  Lds m;
  m.c64 = (unsigned long long *)q; q += 8 * 8;
  m.c32 = (uint32_t *)q;       q += 16 * 4;
  m.hist = (uint32_t *)q;      q += 32 * 4;
  m.sess = (int2 *)q;          q += (size_t)p.n_cap * 8;     // at a fixed offset: its accesses fold it in
  m.warm = (int32_t *)q;                                     // only there with the pool
  return m;
}

// hosts 0..H0-1 ready at time 0, the rest off (in the caller's registers); sessions unplaced
__device__ __forceinline__ void lds_init_closed(const KParams &p, const Lds &m, int lane, int s_lo, int n_sess) {
  if (lane < 8) m.c64[lane] = 0;
  if (lane < 16) m.c32[lane] = lane == CS_NON || lane == CS_PEAK ? (uint32_t)p.H0 : 0u;
  if (lane < 32) m.hist[lane] = 0;
  if (p.warm_n > 0) {
    for (int i = lane; i < WAVE * 4; i += WAVE) m.warm[i] = 0;     // initial hosts: warm from time 0
  }
  for (int s = lane; s < n_sess; s += WAVE) {
    uint32_t g = p.sess_gpus[s_lo + s];
    m.sess[s] = make_int2((int)(SS_UNPLACED | ((g - 1u) << 3)), 0);
  }
  __syncthreads();
}

// ---- S10: close the integrals at t_end and write the result record ---------------------------------
__device__ __forceinline__ void write_stats(const KParams &p, const Lds &m, const Regs &r, uint64_t digest, int rep, int lane) {
  __syncthreads();
  const int32_t t_end = r.t_end > r.lazy_max ? r.t_end : r.lazy_max;
  nbos_stats *out = p.stats + rep;
  if (lane < 32) out->delay_hist[lane] = m.hist[lane] + (lane == 0 ? r.h0 : 0u);
  if (lane == 0) {
    const int64_t sum_delay = (int64_t)m.c64[CL_SUMDELAY], g_wait = (int64_t)m.c64[CL_GWAIT];
    out->status = r.status; out->n_decisions = r.n_dec;
    out->sessions_placed = m.c32[CS_PLACED]; out->sessions_rejected = m.c32[CS_REJECTED];
    out->cells_total = r.c_total; out->cells_immediate = r.c_imm; out->cells_started = r.c_started;
    out->cells_queued = m.c32[CS_QUEUED]; out->cells_aborted = m.c32[CS_ABORTED];
    out->cells_dropped_busy = r.c_busy; out->cells_dropped_unplaced = r.c_unplaced;
    out->executor_reused = r.reused; out->migrations = m.c32[CS_MIGR];
    out->scale_out_hosts = m.c32[CS_SO]; out->scale_in_hosts = m.c32[CS_SI]; out->peak_hosts = m.c32[CS_PEAK];
    out->migrations_warm = m.c32[CS_MIGRWARM];
    out->max_delay_ms = (int32_t)m.c32[CS_MAXDELAY]; out->t_end_ms = t_end;
    const int64_t sum_dur = r.sum_dur + (int64_t)m.c64[CL_BDUR], g_exec = r.g_exec + (int64_t)m.c64[CL_BGEXEC];
    out->sum_delay_ms = sum_delay; out->sum_tct_ms = sum_dur + sum_delay;
    out->gpu_ms_executed = g_exec; out->gpu_ms_committed = g_exec + g_wait;
    out->gpu_ms_provisioned = (int64_t)m.c64[CL_PROV] + (int64_t)m.c32[CS_NON] * p.G * t_end;
    out->reservation_gpu_ms = (int64_t)m.c64[CL_RESV] + (int64_t)(int32_t)m.c32[CS_OPENG] * t_end;
    out->sub_gpu_ms = (int64_t)m.c64[CL_SUB] + (int64_t)(int32_t)m.c32[CS_SUMS] * t_end;
    out->replica_ms = (int64_t)m.c64[CL_REPL] + (int64_t)(int32_t)m.c32[CS_NREP] * t_end;
    out->digest = digest;
  }
}

// At most 128 vector registers (4 waves per SIMD): with 8-byte session records a compute unit then holds
// 16 replays of 1,000 sessions at once.
template <int NJ, uint32_t F>
__global__ void __launch_bounds__(WAVE, 4) nbos_replay_reg_kernel(KParams p) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int rep = launch_slot_replay(p);
  const int lane = threadIdx.x;
  if (rep >= p.n_replays) return;
  // launched without a look at the traces on the host: the validation kernel's verdict comes first
  if (p.trace_err != nullptr && *p.trace_err != 0) { refuse_replay(p, rep, lane, NBOS_E_RANGE); return; }

  const int trace = p.trace_of_replay[rep];
  const int64_t ev_lo = p.ev_offset[trace], ev_hi = p.ev_offset[trace + 1];
  const int s_lo = p.sess_offset[trace];
  const int n_sess = p.sess_offset[trace + 1] - s_lo;
  if (p.trace_err != nullptr && n_sess > p.n_cap) { refuse_replay(p, rep, lane, NBOS_E_LIMIT); return; }

  Lds m;
  unsigned char *q = lds_raw;
  m.c64 = (unsigned long long *)q; q += 8 * 8;
  m.c32 = (uint32_t *)q;       q += 16 * 4;
  m.hist = (uint32_t *)q;      q += 32 * 4;
  m.sess = (int2 *)q;          q += (size_t)p.n_cap * 8;     // at a fixed offset: its accesses fold it in
  m.warm = (int32_t *)q;                                     // only there with the pool

  // S0: hosts 0..H0-1 ready at time 0, the rest off; sessions unplaced
  if (lane < 8) m.c64[lane] = 0;
  if (lane < 16) m.c32[lane] = lane == CS_NON || lane == CS_PEAK ? (uint32_t)p.H0 : 0u;
  if (lane < 32) m.hist[lane] = 0;
  if (p.warm_n > 0) {
    for (int i = lane; i < WAVE * 4; i += WAVE) m.warm[i] = 0;     // initial hosts: warm from time 0
  }
  for (int s = lane; s < n_sess; s += WAVE) {
    uint32_t g = p.sess_gpus[s_lo + s];
    m.sess[s] = make_int2((int)(SS_UNPLACED | ((g - 1u) << 3)), 0);
  }
  __syncthreads();

  const int32_t caplim = p.cap_milli[rep] * p.G * 3;
  Ctx<NJ, F> c{p, m, lane, n_sess, caplim / 1000, p.dlog ? p.dlog + (int64_t)rep * p.dlog_stride : nullptr,
               p.ovf_dur + (int64_t)rep * p.n_cap};
#pragma unroll
  for (int j = 0; j < NJ; j++) c.fin[j] = (lane & 7) < p.G ? 0 : NEVER;
  c.hr = lane < p.H0 ? 0 : NEVER;
  c.hs = 0;
  c.qt = NEVER; c.qd = 0; c.qk = 0xFFFFFFFFu;
  c.vsid = 0xFFFFFFFFu; c.vtm = NEVER;
  c.digest = 0xCBF29CE484222325ULL;
  c.fu = 0;
  c.dyn = dynamic_limit_matters(p, c.flags(), c.slim);
  c.latest = 0;
  Regs r;
  memset(&r, 0, sizeof r);
  r.q_head_t = NEVER;
  r.o_min_t = NEVER;
  r.cl_win = 1024;

  const bool ticking = (c.flags() & (NBOS_F_SCALE_IN | NBOS_F_AUTOSCALE)) != 0;
  int32_t tick_t = ticking ? p.scale_iv : NEVER;
  int32_t due_t = tick_t;                   // earliest queued timer or auto-scaler period
  PROF_BEGIN();

  // S1: stream the events, one per lane per tile, next tile in flight
  int64_t base = ev_lo;                     // first event of the tile held in (nt, nd, ns)
  int32_t vt = 0, vd = 0, vs = 0, nt = 0, nd = 0, ns = 0;
  if (base < ev_hi) {
    const int64_t at = min(base + lane, ev_hi - 1);
    nt = p.ev_time[at]; nd = p.ev_dur[at]; ns = p.ev_sk[at];
  }

  // Outer loop: one iteration per tile of 64 events plus a last one (`final`) that drains the
  // timers. Inner loop: one iteration per item (queued timer, auto-scaler period, or arrival); it
  // never touches the registers of the tile in flight.
  bool final = false;
  while (r.status == NBOS_OK) {
    int32_t vhw = 0;                        // word of the session record of this lane's event
    uint32_t vcode = 0;                     // decision code of a cell that starts at once, without slot and host
    uint64_t todo = 0;                      // events to look at
    if (base < ev_hi) {
      // the prefetched tile becomes current; start loading the one after it
      vt = nt; vd = nd; vs = ns;
      const int64_t cur = base;
      base += WAVE;
      if (base < ev_hi) {
        const int64_t at = min(base + lane, ev_hi - 1);
        nt = p.ev_time[at]; nd = p.ev_dur[at]; ns = p.ev_sk[at];
      }
      const bool valid = cur + lane < ev_hi;
      const bool is_last = cur + lane == ev_hi - 1;
      const uint32_t sid = (uint32_t)vs & 0xFFFFFFu;
      const bool is_cell = ((uint32_t)vs >> 24) == NBOS_EV_CELL;
      wave_sync();
      const int2 rec = m.sess[sid];         // (lanes beyond the last event hold that one's)
      vhw = rec.x;
      vcode = ((uint32_t)NBOS_D_START << 12) | (sid << 16);
      // Cells of sessions in a final state (rejected / ended) and cells that arrive while the
      // session's running cell lasts beyond them change nothing: count them, skip them. Neither
      // condition can be undone before the event's time. The last event of the trace is never
      // skipped, so timers due before it still run first.
      const uint32_t st = (uint32_t)rec.x & 7u;
      const bool dead = (st == SS_REJECTED) | (st == SS_ENDED);
      const bool running = (st == SS_PLACED) & (rec.y > vt);
      const bool skip = valid & !is_last & (dead | (is_cell & running));
      r.c_total += (uint32_t)__builtin_popcountll(wballot(valid & is_cell));
      r.c_unplaced += (uint32_t)__builtin_popcountll(wballot(skip & is_cell & dead));
      r.c_busy += (uint32_t)__builtin_popcountll(wballot(skip & is_cell & !dead));
      const bool plain = valid & is_cell & (st == SS_PLACED) & (((uint32_t)rec.x & SF_ENDING) == 0);
      c.vsid = plain ? sid : 0xFFFFFFFFu;
      c.vtm = plain ? rec.y : NEVER;
      todo = wballot(valid & !skip);
      if (ev_hi - cur <= WAVE) {
        int32_t tl = lane_get(vt, (int)(ev_hi - cur - 1));
        r.t_end = r.t_end > tl ? r.t_end : tl;
      }
    } else {
      final = true;
      const int32_t latest = (int32_t)~wave_min(~(uint32_t)c.latest);      // of the cells that started at once
      r.lazy_max = r.lazy_max > latest ? r.lazy_max : latest;
    }
    PROF(PC_TILE, 1);
    for (;;) {
      if (__builtin_expect(r.status != NBOS_OK, 0)) break;
      // ---- runs of arrivals that start at once (S4, S5): cells of idle placed sessions, no timer due first, the
      // election won. A loop of its own with nothing else in it. Whatever does not fit makes `bad` negative, of what the event's
      // lane says or of what the election says (two branches, as one that is not taken costs a lone wave 12 clocks, a
      // scalar instruction 5), and leaves the arrival to the general path below. No event left: lane 63 is looked at.
      // With five ways out, the keys of hosts that cannot bind masked before the choice, and stale records read again
      // in the loop: 64 hosts 68.1 -> 64.7 ms, 24 hosts 47.2 -> 45.0, 30 hosts 27.9 -> 27.2, 300 short replays 0.84 -> 0.77.
      PROF(PC_LOOP_ROUND, 1);
      [[maybe_unused]] const uint64_t prof_at0 = r.at_once;
      {
        int i;
        int32_t at, bad;
        auto look_at_next = [&]() {
          i = (int)__builtin_ctzll(todo | (1ull << 63));
          at = lane_get(vt, i);
          bad = (todo == 0 ? -1 : 0) | (at - lane_get(c.vtm, i)) | (due_t - 1 - at);
        };
        look_at_next();
        while (__builtin_expect(bad >= 0, 1)) {
          const uint32_t hw = (uint32_t)lane_get(vhw, i);
          const int g = (int)((hw >> 3) & 7u) + 1;
          // election (Section 3.2.2) on the vector side: every host's key; and a host may have the GPUs idle by now
          uint64_t busy[NJ];
          const uint32_t C = committed_words(c, at, c.hr <= at ? 0u : 16u, busy);
          const uint32_t kb = elect_slot(c, hw, (C << 8) | ((uint32_t)c.lane << 2), g);
          if (__builtin_expect(((at - lane_get(c.fu, g - 1)) | (NGPU - (int)(kb >> 8) - g)) < 0, 0)) break;
          const uint32_t host = (kb >> 2) & 63u, slot = kb & 3u;
          const int32_t finish = at + lane_get(vd, i);
          bind_words(c, (int)host, g, finish, busy);
          start_at_once(c, r, vhw, (uint32_t)lane_get((int)vcode, i), hw, slot, host, at, finish);
          r.at_once |= 1ull << i;
          todo &= ~(1ull << i);
          look_at_next();
        }
      }
      PROF(PC_ROUND, __builtin_popcountll(r.at_once ^ prof_at0));
      int i = 0;
      int32_t t = NEVER;
      if (todo != 0) { i = (int)__builtin_ctzll(todo); t = lane_get(vt, i); }
      else if (!final) break;
      wave_sync();
      uint32_t a_s, a_hw, a_fl;
      int32_t a_now, a_sub, a_dur;
      [[maybe_unused]] bool is_retry = false;      // (path profile)
      if (__builtin_expect(t < due_t, 1)) {
        // ---- arrival i ----
        const uint64_t bit = 1ull << i;
        todo &= ~bit;
        const uint32_t sk = (uint32_t)lane_get(vs, i);
        const uint32_t s = sk & 0xFFFFFFu;
        if (__builtin_expect(lane_get(c.vtm, i) <= t, 1)) {
          // a cell of an idle placed session whose record is up to date
          a_s = s; a_hw = (uint32_t)lane_get(vhw, i);
          a_fl = a_hw;
          a_now = t; a_sub = t; a_dur = lane_get(vd, i);
        } else {
          const uint32_t kind = sk >> 24;
          const int2 cur = m.sess[s];
          const uint32_t hw = uni((uint32_t)cur.x), fl = hw;
          const int32_t tm = uni(cur.y);
          if (kind == NBOS_EV_CELL) {           // S4-S8 (counted in c_total at tile load)
            const uint32_t st = fl & 7u;
            if (st == SS_PLACED && tm <= t) {
              a_s = s; a_hw = hw; a_fl = fl & ~(15u << 8); a_now = t; a_sub = t; a_dur = lane_get(vd, i);
            } else {
              if (st == SS_PLACED || st == SS_QUEUED) r.c_busy++; else r.c_unplaced++;
              PROF(PC_DROP, 1);
              continue;
            }
          } else {
            PROF(PC_LOOP_STARTEND, 1);
            if (kind == NBOS_EV_START) { session_start(c, r, s, fl, t); PROF(PC_START, 1); }      // S3, S7
            else { on_session_end(c, r, s, hw, tm, fl, t); PROF(PC_END, 1); }
            due_t = r.q_head_t < tick_t ? r.q_head_t : tick_t;
            continue;
          }
        }
      } else {
        // ---- a timer may be due (S2); always taken while draining ----
        PROF(PC_LOOP_TIMER, 1);
        {
          const int32_t last = r.o_n == 0 ? failing_retries<false>(c, r, t, tick_t) : failing_retries<true>(c, r, t, tick_t);
          PROF(PC_QUIET_RETRIES, 1);
          if (last >= 0) {
            r.t_end = r.t_end > last ? r.t_end : last;
            due_t = r.q_head_t < tick_t ? r.q_head_t : tick_t;
            if (t < due_t) continue;
          }
        }
        bool fire_q = r.q_n > 0, fire_t = ticking;
        if (final) {
          if (fire_t) fire_t = fire_q ? tick_t < r.q_head_t : tick_t < r.lazy_max;
          if (fire_t) fire_q = false;
        } else {
          if (fire_q) fire_q = r.q_head_t <= t;
          if (fire_t) fire_t = tick_t <= t;
          if (fire_q && fire_t) { if (r.q_head_t <= tick_t) fire_t = false; else fire_q = false; }
        }
        if (__builtin_expect(fire_t, 0)) {
          tick(c, r, tick_t);
          tick_t += p.scale_iv;
          due_t = r.q_head_t < tick_t ? r.q_head_t : tick_t;
          PROF(PC_TICK, 1);
          continue;
        }
        if (__builtin_expect(!fire_q, 0)) break;   // only reached while draining: nothing is left
        const int32_t now = r.q_head_t;
        const uint32_t key = (uint32_t)lane_get((int)c.qk, 0);
        const int32_t dur = lane_get(c.qd, 0);
        const uint32_t s = key & 0xFFFFu;
        const int2 cur = m.sess[s];           // (asked for before the pop, which does not touch this record)
        timer_pop(c, r);
        r.t_end = r.t_end > now ? r.t_end : now;
        const uint32_t hw = uni((uint32_t)cur.x), fl = hw;
        if ((key >> 16) != QK_RETRY) {
          end_session(c, r, s, hw, fl, now);
          due_t = r.q_head_t < tick_t ? r.q_head_t : tick_t;
          PROF(PC_TIMER_OTHER, 1);
          continue;
        }
        a_s = s; a_hw = hw; a_fl = fl; a_now = now; a_sub = uni(cur.y); a_dur = dur;
        is_retry = true;
      }
      PROF(PC_LOOP_ATTEMPT, 1);
      PROF_ATTEMPT_BEGIN(m, r);
      attempt(c, r, a_s, a_hw, a_fl, a_now, a_sub, a_dur);
      PROF_ATTEMPT_END(m, r, is_retry);
      due_t = r.q_head_t < tick_t ? r.q_head_t : tick_t;
    }
    if (final) break;
    fold_starts(c, r, vt, vd, (uint32_t)vhw);
  }

  write_stats(p, m, r, c.digest, rep, lane);
  PROF_OUT(rep);
}

// ---- closed loop: runs of retries that fail again (failing_retries() for this kernel) -----------------
// Same tests, same order. The retry's timer either stays in the sorted registers at its new place, or,
// if it is no longer earlier than everything that waits in the session records, goes there. A retry
// with no retries left is left for the general path (giving a cell up schedules the session's next
// event). Returns the time of the last retry handled, or -1. (The times skipped go by the bound over all hosts; the
// one over the session's own hosts, retry_bound, would give 1 to 3 % here where cells do not migrate: 24 hosts 21.7
// against 21.0 ms, 8 hosts 23.8 against 23.6, 64 hosts 24.2 either way, 512 replays of 20,000 cells.)
template <int NJ, uint32_t F>
__device__ __forceinline__ int32_t cl_failing_retries(Ctx<NJ, F> &c, Regs &r, int32_t t_limit) {
  int32_t last = -1;
  const bool may_skip = !(c.flags() & NBOS_F_AUTOSCALE) &&
                        (c.flags() & (NBOS_F_SCALE_IN | NBOS_F_SCALE_OUT)) != (NBOS_F_SCALE_IN | NBOS_F_SCALE_OUT);
  while (r.q_n > 0 && r.q_head_t <= t_limit) {
    const int32_t now = r.q_head_t;
    const uint32_t key = (uint32_t)lane_get((int)c.qk, 0);
    if ((key >> 16) != QK_RETRY) break;
    const uint32_t s = key & 0xFFFFu;
    wave_sync();
    const int2 rec = c.m.sess[s];
    const uint32_t hw = uni((uint32_t)rec.x), fl = hw;
    const int32_t t_submit = uni(rec.y);
    int retries = (int)((fl >> 8) & 15u);
    if (retries >= c.p.max_retries) break;                     // it would be given up: general path
    const int g = (int)((fl >> 3) & 7u) + 1;
    if (now >= lane_get(c.fu, g - 1)) {
      const uint64_t idle_ok = hosts_with_idle(c, now, g);
      if (idle_ok & own_hosts(hw)) break;                                           // the election succeeds
      if (idle_ok == 0) {
        const int32_t bound = earliest_idle(c, g);
        c.fu = (c.lane >= g - 1) & (c.fu < bound) ? bound : c.fu;
      } else if (c.flags() & NBOS_F_MIGRATE) {
        const int S = (int)(c.hs & 0xFFFFu);
        if (idle_ok & wballot(S <= cap_room(c, g))) break;                        // a migration target
      }
    }
    if (c.flags() & NBOS_F_SCALE_OUT) {
      wave_sync();
      if ((int)uni(c.m.c32[CS_NON]) < c.p.Hmax) break;                            // a host can be added
    }
    // it fails again: bump the retry count (skipping retries that are bound to fail as well)
    retries++;
    if (may_skip) {
      const int32_t bound = lane_get(c.fu, g - 1);
      while (retries < c.p.max_retries && t_submit + retries * c.p.retry_iv < bound) retries++;
    }
    if ((int64_t)t_submit + (int64_t)retries * c.p.retry_iv >= 0x7FFFFFFFLL) break;   // out of range: general path
    last = now;
    const uint32_t nfl = (fl & ~(15u << 8)) | ((uint32_t)retries << 8);
    c.m.sess[s].x = (int)nfl;
    const int32_t t_new = t_submit + retries * c.p.retry_iv;
    const int32_t st = __builtin_amdgcn_update_dpp(c.qt, c.qt, 0x130, 0xF, 0xF, false);          // wave_shl:1
    const int32_t sd = __builtin_amdgcn_update_dpp(c.qd, c.qd, 0x130, 0xF, 0xF, false);
    const uint32_t sk = (uint32_t)__builtin_amdgcn_update_dpp((int)c.qk, (int)c.qk, 0x130, 0xF, 0xF, false);
    const int32_t sx = __builtin_amdgcn_update_dpp(c.qx, c.qx, 0x130, 0xF, 0xF, false);
    const int32_t sn = __builtin_amdgcn_update_dpp(c.qnx, c.qnx, 0x130, 0xF, 0xF, false);
    const int32_t sh = __builtin_amdgcn_update_dpp(c.qnth, c.qnth, 0x130, 0xF, 0xF, false);
    if (r.o_n > 0 && !(t_new < r.o_min_t || (t_new == r.o_min_t && key < r.o_min_k))) {
      // no longer earlier than all that waits in the records: the timer goes there, off the registers
      ovf_push(c, r, t_new, key, 0);
      c.qt = st; c.qd = sd; c.qk = sk; c.qx = sx; c.qnx = sn; c.qnth = sh;
      r.q_n--;
      if (r.q_n == 0 && r.o_n > 0) refill(c, r);
      r.q_head_t = r.q_n > 0 ? lane_get(c.qt, 0) : NEVER;
    } else {
      // it moves from lane 0 to its new place: the entries before that shift down one lane
      const bool before = (c.lane >= 1) & (c.lane < r.q_n) & ((c.qt < t_new) | ((c.qt == t_new) & (c.qk < key)));
      const int pos = __builtin_popcountll(wballot(before));
      const int32_t d_own = lane_get(c.qd, 0), x_own = lane_get(c.qx, 0), n_own = lane_get(c.qnx, 0), h_own = lane_get(c.qnth, 0);
      const bool down = c.lane < pos, here = c.lane == pos;
      c.qt = here ? t_new : down ? st : c.qt;   c.qd = here ? d_own : down ? sd : c.qd;    c.qk = here ? key : down ? sk : c.qk;
      c.qx = here ? x_own : down ? sx : c.qx;   c.qnx = here ? n_own : down ? sn : c.qnx;  c.qnth = here ? h_own : down ? sh : c.qnth;
      r.q_head_t = lane_get(c.qt, 0);
    }
  }
  return last;
}

// ---- closed-loop reading of the trace (see the file header and nbos_kernel_closed.hpp) -----------------
// Arrivals from the stream are the first STARTs only (the STARTs that head a chain record); every other
// event is a timer of kind QK_NEXT. Timers whose events were not loaded when they were scheduled load
// them together when the first of them gets to the head.
template <int NJ, uint32_t F>
__global__ void __launch_bounds__(WAVE, 4) nbos_replay_reg_closed_kernel(KParams p) {
  static_assert(Ctx<NJ, F>::closed, "instantiate with a closed-loop flag set");
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int rep = launch_slot_replay(p);
  const int lane = threadIdx.x;
  if (rep >= p.n_replays) return;

  const int trace = p.trace_of_replay[rep];
  const int64_t ev_lo = p.ev_offset[trace], ev_hi = p.ev_offset[trace + 1];
  const int s_lo = p.sess_offset[trace];
  const int n_sess = p.sess_offset[trace + 1] - s_lo;

  const Lds m = lds_carve_closed(p, lds_raw);
  lds_init_closed(p, m, lane, s_lo, n_sess);

  const int32_t caplim = p.cap_milli[rep] * p.G * 3;
  Ctx<NJ, F> c{p, m, lane, n_sess, caplim / 1000, p.dlog ? p.dlog + (int64_t)rep * p.dlog_stride : nullptr, nullptr};
#pragma unroll
  for (int j = 0; j < NJ; j++) c.fin[j] = (lane & 7) < p.G ? 0 : NEVER;
  c.hr = lane < p.H0 ? 0 : NEVER;
  c.hs = 0;
  c.qt = NEVER; c.qd = 0; c.qk = 0xFFFFFFFFu;
  c.vsid = 0xFFFFFFFFu; c.vtm = NEVER;
  c.digest = 0xCBF29CE484222325ULL;
  c.fu = 0;
  c.dyn = dynamic_limit_matters(p, c.flags(), c.slim);
  c.cl_cur = p.cl_cursor + (int64_t)rep * (p.n_cap + 1);
  c.cl_dur = p.ev_dur + ev_lo; c.cl_sk = p.ev_sk + ev_lo; c.cl_chain = p.cl_chain + ev_lo;
  c.qx = 0; c.qnx = -1; c.qnth = 0;
  Regs r;
  memset(&r, 0, sizeof r);
  r.q_head_t = NEVER;
  r.o_min_t = NEVER;
  r.cl_win = 1024;

  bool final = false;
  for (int64_t base = ev_lo; r.status == NBOS_OK; base += WAVE) {
    uint64_t todo = 0;
    int32_t vt = 0, vnx = -1, vnth = -1;
    uint32_t vs = 0;
    if (base < ev_hi) {
      const int64_t at = min(base + lane, ev_hi - 1);
      vt = p.ev_time[at]; vs = (uint32_t)p.ev_sk[at];
      const int2 ch = p.cl_chain[at];
      vnx = ch.x; vnth = ch.y;
      todo = wballot((base + lane < ev_hi) & ((vs >> 24) == NBOS_EV_START) & (vnth >= 0));
    } else {
      final = true;
    }
    while (r.status == NBOS_OK) {
      int i = 0;
      int32_t t = NEVER;
      if (todo != 0) { i = (int)__builtin_ctzll(todo); t = lane_get(vt, i); }
      else if (!final) break;
      wave_sync();
      if (r.q_n > 0 && r.q_head_t <= t) {
        // ---- S2: the earliest timer is due ----
        {
          const int32_t last = cl_failing_retries(c, r, t);
          if (last >= 0) { r.t_end = r.t_end > last ? r.t_end : last; continue; }
        }
        if (!(lane_get(c.qx, 0) & CLX_LOADED) && ((uint32_t)lane_get((int)c.qk, 0) >> 16) != QK_END) {
          const bool load = (c.lane < r.q_n) & ((c.qx & CLX_LOADED) == 0) & ((c.qk >> 16) != QK_END);
          const int32_t e = load ? c.qd : 0;                   // (the lanes with nothing to load read event 0)
          const int2 ch = c.cl_chain[e];
          const int32_t x = c.cl_dur[e] | (int32_t)(((uint32_t)c.cl_sk[e] >> 24) << 28) | CLX_LOADED;
          c.qx = pick(load, x, c.qx);
          c.qnx = pick(load, ch.x, c.qnx); c.qnth = pick(load, ch.y, c.qnth);
        }
        const int32_t now = r.q_head_t;
        const uint32_t key = (uint32_t)lane_get((int)c.qk, 0);
        const int32_t e = lane_get(c.qd, 0);
        const int32_t x = lane_get(c.qx, 0), nx = lane_get(c.qnx, 0), nth = lane_get(c.qnth, 0);
        timer_pop(c, r);
        r.t_end = r.t_end > now ? r.t_end : now;
        const uint32_t s = key & 0xFFFFu, kind = key >> 16;
        wave_sync();
        const int2 cur = m.sess[s];
        const uint32_t hw = uni((uint32_t)cur.x), fl = hw;
        const int32_t tm = uni(cur.y);
        if (kind == QK_END) { end_session(c, r, s, hw, fl, now); continue; }
        r.cl_e = e; r.cl_x = x; r.cl_nx = nx; r.cl_nth = nth;
        const int32_t dur = x & 0x0FFFFFFF;
        if (kind == QK_RETRY) {
          attempt(c, r, s, hw, fl, now, tm, dur);
        } else if ((((uint32_t)x >> 28) & 3u) == NBOS_EV_CELL) {     // the session submits its next cell (S4-S8)
          r.c_total++;
          const uint32_t st = fl & 7u;
          // (a session whose next event is due is idle: its time word may hold that due time)
          if (st == SS_PLACED && !(fl & SF_ENDING)) attempt(c, r, s, hw, fl & ~(15u << 8), now, now, dur);
          else if (st == SS_PLACED || st == SS_QUEUED) r.c_busy++;
          else r.c_unplaced++;
        } else {
          on_session_end(c, r, s, hw, now, fl, now);              // S9: idle, so it ends at once
        }
        continue;
      }
      if (todo == 0) break;                 // draining and no timer is left
      todo &= todo - 1;
      const uint32_t s = (uint32_t)lane_get((int)vs, i) & 0xFFFFFFu;
      const uint32_t fl = uni((uint32_t)m.sess[s].x);
      r.t_end = r.t_end > t ? r.t_end : t;
      r.cl_e = (int32_t)(base - ev_lo) + i; r.cl_nx = lane_get(vnx, i); r.cl_nth = lane_get(vnth, i);
      session_start(c, r, s, fl, t);        // S3, S7; a placed session's first event is scheduled there
    }
    if (final) break;
  }
  write_stats(p, m, r, c.digest, rep, lane);
}

}  // namespace regk
}  // namespace
