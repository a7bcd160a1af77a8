// nbos_kernel_batch.hpp — replay of the Batch baseline (the paper's "Baselines" section): every cell is a job of its
// own, first come first served, a container per job. One workgroup (one wave64) per replay, any cluster
// size up to NBOS_MAX_HOSTS.
//
// Hosts: a bitmap per number of held GPUs ("level"; slots beyond G count as held, hosts that are off or being provisioned
// as full), 64 hosts to a word, level 8 left out: lane 8 l + w holds the word of hosts 64 w .. 64 w + 63 on level l,
// for each set of 512 hosts (NS of them) a pair of registers. A job takes the ready host with the fewest held GPUs (ties:
// lowest index): the first bit of the first lane that has one, found by two bit scans, and it fits there or nowhere.
// A job or a completion flips one bit in each of two lanes. On up to 64 hosts (NW = 1) lane l holds the one word of
// level l, and level 8 is there as well: every host is in exactly one lane, so that a completion's two lanes are a ballot
// and that ballot shifted by g. Many replays of a small cluster share a compute unit and are bound by its scalar unit,
// not by latency: 46 scalar instructions per job and completion in place of 67 take 4,096 replays of 16, 30 and 64 hosts
// with 3,000 cells from 2.86, 2.56 and 3.44 ms to 2.34, 2.08 and 2.81 (with a key per host 2.35, 2.31 and 3.35; with all
// that follows 1.61, 1.61 and 2.75).
// Completions: the earliest ones, in the order of their times, in registers (qt, qk: entry i in lane i, qe of them,
// at most 63): all running jobs that finish up to win_t. With more than MID_CAP sessions those that finish up to mid_t are
// in a list in LDS as well (mid_t[], mid_k[], in no order), the others are found in the session records only: a refill of
// the registers looks through a few hundred of the list, once per about 40 jobs, and the list is made anew from all
// records once per few hundred.
// Two jobs of one session in a tile of 64 events: the second is dropped if the first outlasts its arrival. With at most
// MID_CAP sessions (FEW) that is common, and a start looks for its session's other lanes then and there (two comparisons,
// seven scalar instructions); with more it is rare, and such arrivals leave the loop of starts for a look at the record
// (as all did before: 4,096 replays of 2,000 cells, 3 and 25 sessions on 16 hosts 1.67 and 1.36 ms, now 0.90 and 0.90;
// 400 sessions on 30 hosts, 256 replays of 20,000 cells, 6.36 and 6.20).
// Hosts being provisioned come up in the order of their index (all take the same time): next_up, ready[].
// Sessions in LDS: time[] and meta[] of the latest job: finish, host | (g - 1) << 27.
//
// The CPU reference keeps a queue, runs completions and "host ready" as timers and looks at the queue after each
// instant. First come, first served means that jobs start in the order in which they arrive, so a job can be followed to
// its start before the next arrival is looked at: it first meets the scheduler at T0 = max(its arrival, the start of the
// job before it), with everything applied that happens to the hosts up to T0. It starts there if a host has the GPUs
// idle; else nothing starts until it does, it asks for one more host (once), and starts at the first instant
// after which a host has them. An arrival is dropped if its session's previous job finishes later than that, and
// that job's start is known by then. There is no queue.
//
// Bound by the latency of the serial chain of jobs (one wave per replay). On a lone wave an instruction takes 5 clocks, a
// scalar one that reads what the vector side has just produced 20 more, a branch 12 to 25: hence bit scans where
// a minimum over the keys of all hosts was taken (and the rows of the hosts with a completion read again to refresh
// them); a job leaves its start and host in its lane, and records, sums, waits and digest are made from those for 64 jobs
// at a time. 512 hosts, 250,000 jobs, 256 replays: 152.4 ms with a key per host, a minimum over the keys and the queue, 84.4
// with this. By the path profile (500,000 jobs) 53 % are the loop of starts, 600 clocks per job and completion with the
// marks, 30 % the one job in ten that leaves it (it waits, or has to be preceded by a refill), 15 % refills.
// Control flow is uniform throughout: a store that one lane would do is done by all lanes.
#pragma once
#include "nbos_common.hpp"

namespace {
namespace batchk {

constexpr int G_SHIFT = 27;
constexpr uint32_t HOST_MASK = 1023u;
constexpr int Q_CAP = WAVE - 1;                       // completions in registers: lane 63 holds NEVER
constexpr uint32_t SLOW = 1u << 31;                   // (of an arrival) an earlier arrival of its session is in the tile
constexpr int32_t ALL = NEVER - 1;                    // win_t when no running job is left out
constexpr int MID_CAP = 512;                          // jobs in the list in LDS

struct Lds {
  uint32_t *hist;               // 32 bins, and behind them a word per lane for the lanes that an LDS atomic is not for
  int32_t *stage_t;             // [WAVE + 4] completions on their way into the registers; one place for lanes with none
  uint32_t *stage_k;
  int32_t *time;
  uint32_t *meta;
  int32_t *mid_t;               // [MID_CAP + 4] finish and meta word of the jobs in the list
  uint32_t *mid_k;
  int32_t *ready;               // [hosts] when a host that was added comes up
};

// NW: words of 64 hosts per level (1, 8, or 16 in two sets of 8). FEW: at most MID_CAP sessions
template <int NW, bool FEW>
struct Ctx {
  static constexpr int NS = NW > 8 ? 2 : 1;
  static constexpr int PER = NW > 8 ? 8 : NW;         // lanes per level
  static constexpr bool ALL_LEVELS = 9 * PER <= WAVE;  // full hosts have lanes, too
  const KParams &p;
  Lds m;
  int lane;
  int n_sess;
  uint32_t lo[NS], hi[NS];      // the levels, see above
  int32_t qt;                   // completions: finish,
  uint32_t qk;                  // and the session's meta word
  // the tile of events: arrival, container start + duration, session | (g - 1) << 16 | SLOW; and of the jobs that
  // have started: when, where
  int32_t vt, vfd;
  uint32_t vjob;
  uint32_t vsid;                // (FEW) the session
  int32_t vstart;
  uint32_t vhost;
  uint64_t power;               // see digest_powers
};

struct State {
  uint32_t c_total, c_started, c_imm, n_dec;
  int32_t qe, q_t;              // completions: how many, the next one's time (NEVER: none listed)
  uint32_t q_k;                 // ... and meta word
  int32_t win_t, win;           // all that finish up to win_t are listed; the window the next refill takes
  int32_t mid_t, mid_n;         // the list in LDS: all that finish up to mid_t >= win_t (with few sessions: not looked at)
  int32_t mid_win;
  int32_t next_up, up_t;        // the next host to come up and when (NEVER: none is being provisioned)
  int32_t n_on;
  int32_t now;                  // no job to come meets the scheduler before this: the latest one did, or has started, at this time
  // a job that has started, finishes within the lists' windows and finds no room there (p_f < 0: none)
  int32_t p_f;
  uint32_t p_k;
  uint64_t jobs, todo;          // arrivals of the tile that have not been dropped; those of them that are still to come
  uint64_t saved;               // jobs of the tile whose records are written (FEW: that are not their session's latest any more)
  uint64_t folded;              // ... whose decisions are in the digest
  uint64_t digest;
  int64_t prov;
  int32_t latest_up, t_end;
  int32_t status;               // NBOS_OK, or NBOS_E_RANGE once a time leaves the int32 range
};

// the host (set, word, bit) that the lanes of `flip` stand for moves between the levels of those lanes
template <int NW, bool FEW>
__device__ __forceinline__ void flip_host(Ctx<NW, FEW> &c, uint64_t flip, uint32_t h) {
#pragma unroll
  for (int s = 0; s < c.NS; s++) {
    const uint64_t here = c.NS == 1 || (int)(h >> 9) == s ? flip : 0ull;
    const uint64_t bit = (uint64_t)(in_mask(here) ? 1u : 0u) << (h & 63u);
    c.lo[s] ^= (uint32_t)bit;
    c.hi[s] ^= (uint32_t)(bit >> 32);
  }
}

// the g GPUs that a job held on host h are idle again (a host that comes up: all G); returns the host's lane from now on
template <int NW, bool FEW>
__device__ __forceinline__ int give_back(Ctx<NW, FEW> &c, uint32_t h, int g) {
  uint32_t lo = c.lo[0], hi = c.hi[0];
  if constexpr (Ctx<NW, FEW>::NS == 2) { lo = h >> 9 ? c.lo[1] : lo; hi = h >> 9 ? c.hi[1] : hi; }
  const uint32_t there = (uint32_t)((((uint64_t)hi << 32) | lo) >> (h & 63u)) & 1u;
  if constexpr (Ctx<NW, FEW>::ALL_LEVELS) {
    const uint32_t from = (uint32_t)wballot(there != 0u), to = from >> g;
    flip_host(c, from | to, h);
    return __builtin_ctz(to);
  }
  const uint32_t w = (h >> 6) & 7u;
  const uint64_t from = wballot(there != 0u) & (0x0101010101010101ull << w);      // no lane: the host was full
  const uint64_t full = from == 0 ? 1ull << w : 0ull;          // (g = 8 is a full host: then `from` is 0)
  const uint64_t to = (from >> (8 * (g & 7))) | (full << ((64 - 8 * g) & 63));
  flip_host(c, from | to, h);
  return (int)__builtin_ctzll(to);
}

// nothing happens to the hosts before this time
__device__ __forceinline__ int32_t due_time(const State &r) { return min(min(r.q_t, r.up_t), r.win_t + 1); }

// Which of the n times at `times` lie in [from, from + win]? They and their keys come to lie side by side in stage_t and
// stage_k (the first 64); returned are how many there are, and the earliest time beyond (as a distance from `from`; 2^31
// or more: none). Times before `from` wrap to large distances. Both arrays are read four at a time.
template <int NW, bool FEW>
__device__ __forceinline__ int scan_window(const Ctx<NW, FEW> &c, const int32_t *times, const uint32_t *keys, int n, int32_t from, uint32_t win, uint32_t &left) {
  const int4 *time4 = (const int4 *)times, *key4 = (const int4 *)keys;
  int cnt = 0;
  uint32_t mn = 0xFFFFFFFFu;
  for (int q0 = 0; 4 * q0 < n; q0 += WAVE) {
    const int q = q0 + c.lane, at = min(q, (n - 1) >> 2);
    const int4 d = time4[at], e = key4[at];
    const int32_t t[4] = {d.x, d.y, d.z, d.w}, k[4] = {e.x, e.y, e.z, e.w};
    uint64_t b[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const uint32_t x = (uint32_t)t[j] - (uint32_t)from;
      const bool in = 4 * q + j < n, hit = in & (x <= win);
      b[j] = wballot(hit);
      mn = in & !hit ? umin(mn, x) : mn;
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int to = min(cnt + lane_rank(b[j]), WAVE), place = in_mask(b[j]) ? to : WAVE;
      c.m.stage_t[place] = t[j];
      c.m.stage_k[place] = (uint32_t)k[j];
      cnt += __builtin_popcountll(b[j]);
    }
  }
  left = wave_min(mn);
  return cnt;
}

// A window of `win` from `from` on holds cnt jobs, too many; t: when 64 of them end. The window to look at next, for about
// `aim` of them: in proportion, but no narrower than up to the earliest of the 64 and narrower than up to the latest. All 64
// at one instant (`crowd` from then on): the window before it. (Windows cut in proportion alone take a dozen passes to get
// down to one instant with a hundred completions: traces on a grid of ten minutes, 256 replays of 20,000 cells, 200, 300 and
// 520 hosts 5.42, 5.82 and 7.79 ms, with this 4.04, 4.14 and 5.51.)
__device__ __forceinline__ uint32_t narrower(uint32_t win, int cnt, int aim, int32_t t, int32_t from, int32_t &crowd) {
  const uint32_t x = (uint32_t)t - (uint32_t)from, lo = wave_min(x), hi = ~wave_min(~x);
  const uint32_t share = (uint32_t)((float)win * ((float)aim / (float)cnt));      // (aim < cnt: below win)
  crowd = lo == hi ? from + (int32_t)lo : crowd;
  return lo == hi ? lo - (lo != 0u ? 1u : 0u) : umin(share > lo ? share : lo, hi - 1u);
}

// The list in LDS anew: the running jobs that finish within a window from `from` on, at most MID_CAP (the window adapts
// to find 192 to 384); more at one instant: none, and the registers are refilled from the records.
template <int NW, bool FEW>
__device__ __forceinline__ void list_jobs(Ctx<NW, FEW> &c, State &r, int32_t from) {
  const int4 *time4 = (const int4 *)c.m.time, *key4 = (const int4 *)c.m.meta;
  const int quads = (c.n_sess + 3) >> 2;
  uint32_t win = (uint32_t)r.mid_win;
  int cnt;
  uint32_t left;
  int32_t crowd = -1;
  for (;;) {
    win = umin(win, (uint32_t)(ALL - from));
    cnt = 0;
    uint32_t mn = 0xFFFFFFFFu;
    int4 next = time4[min(c.lane, quads - 1)], next_k = key4[min(c.lane, quads - 1)];
    for (int q0 = 0; q0 < quads; q0 += WAVE) {
      const int q = q0 + c.lane;
      const int4 d = next, e = next_k;
      next = time4[min(q + WAVE, quads - 1)]; next_k = key4[min(q + WAVE, quads - 1)];
      const bool in = q < quads;                       // (the places beyond the last session hold time 0, which is before `from`)
      const int32_t t[4] = {d.x, d.y, d.z, d.w}, k[4] = {e.x, e.y, e.z, e.w};
      uint64_t b[4];
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const uint32_t x = (uint32_t)t[j] - (uint32_t)from;
        b[j] = wballot(in & (x <= win));
        mn = in & (x > win) ? umin(mn, x) : mn;
      }
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int to = min(cnt + lane_rank(b[j]), MID_CAP), place = in_mask(b[j]) ? to : MID_CAP;
        c.m.mid_t[place] = t[j];
        c.m.mid_k[place] = (uint32_t)k[j];
        cnt += __builtin_popcountll(b[j]);
      }
    }
    left = wave_min(mn);
    if (cnt == 0 && left < 0x80000000u) {
      from += (int32_t)left;
      win = from == crowd ? 0u : win;
      continue;
    }
    if (cnt <= MID_CAP) break;
    if (win == 0) break;
    wave_sync();
    win = narrower(win, cnt, 300, c.m.mid_t[c.lane], from, crowd);
  }
  wave_sync();
  r.mid_n = cnt <= MID_CAP ? cnt : 0;
  r.mid_t = cnt > MID_CAP ? from - 1 : left < 0x80000000u ? from + (int32_t)win : ALL;
  if (crowd < 0) r.mid_win = cnt < MID_CAP * 3 / 8 ? (int32_t)umin(win + (win + 1) / 2 + 1, 1u << 26) : cnt > MID_CAP * 3 / 4 ? (int32_t)(win - win / 4) : (int32_t)win;
}

// The list in the registers is empty and time goes on beyond win_t, at most to t: the completions of the next window come in.
// More than fit into the registers at one instant: they are all applied at once if they are due at t, or left until they are.
template <int NW, bool FEW>
__device__ __forceinline__ void refill(Ctx<NW, FEW> &c, State &r, int32_t t) {
  wave_sync();
  int32_t from = r.win_t + 1;
  uint32_t win = (uint32_t)r.win, left, most;
  int cnt, n;
  const int32_t *times;
  const uint32_t *keys;
  int32_t crowd = -1;                          // more than fit end at this instant
  r.qe = 0; r.q_t = NEVER;
  c.qt = NEVER;
  for (;;) {
    times = c.m.time; keys = c.m.meta; n = c.n_sess;
    most = (uint32_t)(ALL - from);            // (from <= ALL: a finish is below NEVER)
    if constexpr (!FEW) {
      if (r.mid_t < from) list_jobs(c, r, from);
      if (r.mid_t >= from) { times = c.m.mid_t; keys = c.m.mid_k; n = r.mid_n; most = (uint32_t)(r.mid_t - from); }
    }
    win = umin(win, most);
    cnt = scan_window(c, times, keys, n, from, win, left);
    if (cnt == 0) {
      from += left < 0x80000000u ? (int32_t)left : (int32_t)most + 1;      // nothing (listed) up to there
      if (from > ALL) { r.win_t = ALL; return; }
      win = from == crowd ? 0u : (uint32_t)r.win;
      continue;
    }
    if (cnt <= Q_CAP) break;
    wave_sync();
    if (win != 0) win = narrower(win, cnt, 40, c.m.stage_t[c.lane], from, crowd);
    else crowd = from;
    if (crowd == from) {
      const bool now = t >= from;
      r.win_t = now ? from : from - 1;
      r.mid_t = max(r.mid_t, r.win_t);
      if (!now) return;
      for (int s0 = 0; s0 < n; s0 += WAVE) {
        const int s = min(s0 + c.lane, n - 1);
        const uint32_t k = keys[s];
        for (uint64_t w = wballot((s0 + c.lane < n) & (times[s] == from)); w != 0; w &= w - 1) {
          const uint32_t one = (uint32_t)lane_get((int)k, (int)__builtin_ctzll(w));
          give_back(c, one & HOST_MASK, (int)((one >> G_SHIFT) & 7u) + 1);
        }
      }
      return;
    }
  }
  r.win_t = from + (int32_t)win;
  r.mid_t = max(r.mid_t, r.win_t);
  // (a window cut short by the end of the list, or by a crowd, says nothing about the next one)
  if (cnt > 7 * WAVE / 8) r.win = (int32_t)(win - win / 4);
  else if (cnt < WAVE / 2 && (int32_t)win == r.win) r.win = (int32_t)umin(win + (win + 1) / 2 + 1, 1u << 26);
  else if (win < most && crowd < 0) r.win = (int32_t)win;
  wave_sync();
  const bool take = c.lane < cnt;
  const int32_t f = c.m.stage_t[c.lane], t_own = take ? f : NEVER;
  const uint32_t k = c.m.stage_k[c.lane];
  const int rank = timer_ranks(c.lane, cnt, t_own, (uint32_t)c.lane);
  const int dst = (take ? rank : c.lane) << 2;
  c.qt = __builtin_amdgcn_ds_permute(dst, t_own);
  c.qk = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)k);
  r.qe = cnt;
  r.q_t = lane_get(c.qt, 0); r.q_k = (uint32_t)lane_get((int)c.qk, 0);
}

// a job that finishes at f goes into the list in the registers (there is room)
template <int NW, bool FEW>
__device__ __forceinline__ void insert_completion(Ctx<NW, FEW> &c, State &r, int32_t f, uint32_t k) {
  const int pos = __builtin_popcountll(wballot(c.qt <= f));
  const int32_t st = __builtin_amdgcn_update_dpp(c.qt, c.qt, 0x138, 0xF, 0xF, false);          // wave_shr:1
  const uint32_t sk = (uint32_t)__builtin_amdgcn_update_dpp((int)c.qk, (int)c.qk, 0x138, 0xF, 0xF, false);
  const bool up = c.lane > pos, here = c.lane == pos;
  c.qt = here ? f : up ? st : c.qt;
  c.qk = here ? k : up ? sk : c.qk;
  r.qe++;
  r.q_t = lane_get(c.qt, 0); r.q_k = (uint32_t)lane_get((int)c.qk, 0);
}

// The job that has started finishes at p_f <= mid_t, and there was no room where that belongs: the list in LDS is given
// up, or (if the registers are still full) the latest instant in the registers, and that list with it.
template <int NW, bool FEW>
__device__ __forceinline__ void make_room(Ctx<NW, FEW> &c, State &r) {
  const int32_t f = r.p_f;
  r.p_f = -1;
  if (f <= r.win_t) {
    if (r.qe == Q_CAP) {
      const int32_t last = lane_get(c.qt, Q_CAP - 1);
      r.qe = __builtin_popcountll(wballot(c.qt < last));
      c.qt = c.lane < r.qe ? c.qt : NEVER;
      r.q_t = lane_get(c.qt, 0);
      r.win_t = last - 1;
      r.mid_t = r.win_t;
    }
    if (f <= r.win_t) insert_completion(c, r, f, r.p_k);
  } else {
    r.mid_t = r.win_t;
  }
}

// the next completion leaves the list
template <int NW, bool FEW>
__device__ __forceinline__ void pop_completion(Ctx<NW, FEW> &c, State &r) {
  c.qt = __builtin_amdgcn_update_dpp(c.qt, c.qt, 0x130, 0xF, 0xF, false);                // wave_shl:1
  c.qk = (uint32_t)__builtin_amdgcn_update_dpp((int)c.qk, (int)c.qk, 0x130, 0xF, 0xF, false);
  r.qe--;
  r.q_t = lane_get(c.qt, 0); r.q_k = (uint32_t)lane_get((int)c.qk, 0);
}

// The ready host with the fewest held GPUs, lowest index first: its lane (level 8 or beyond: all are full).
// The choice of the set comes back in `set`.
template <int NW, bool FEW>
__device__ __forceinline__ int best_lane(const Ctx<NW, FEW> &c, int &set) {
  const uint64_t a = wballot((c.lo[0] | c.hi[0]) != 0u);
  set = 0;
  if constexpr (Ctx<NW, FEW>::ALL_LEVELS) return (int)__builtin_ctzll(a);     // (a host is in some lane)
  int L = a != 0 ? (int)__builtin_ctzll(a) : WAVE;
  if constexpr (Ctx<NW, FEW>::NS == 2) {
    const uint64_t b = wballot((c.lo[1] | c.hi[1]) != 0u);
    const int L1 = b != 0 ? (int)__builtin_ctzll(b) : WAVE;
    set = (L1 >> 3) < (L >> 3) ? 1 : 0;
    L = set ? L1 : L;
  }
  return L;
}
template <int NW, bool FEW>
__device__ __forceinline__ bool fits(const Ctx<NW, FEW> &, int L, int g) { return L / Ctx<NW, FEW>::PER + g <= NGPU; }

// The records of the tile's jobs that have started since this was last done (before anyone looks at the records: a refill,
// a second arrival of a session in the tile, the next tile).
template <int NW, bool FEW>
__device__ __forceinline__ void save_records(Ctx<NW, FEW> &c, State &r) {
  const uint64_t started = r.jobs & ~r.todo;
  wave_sync();
  const bool mine = in_mask(started & ~r.saved);
  const int s = (int)(c.vjob & 0xFFFFu);
  *(mine ? &c.m.time[s] : c.m.stage_t + WAVE) = job_finish(c.vstart, c.vfd);
  *(mine ? &c.m.meta[s] : c.m.stage_k + WAVE) = c.vhost | (((c.vjob >> 16) & 7u) << G_SHIFT);
  if constexpr (!FEW) r.saved = started;
}

// The decisions of the tile's jobs in `jobs` go into the digest (they are the latest ones), and into the log.
template <int NW, bool FEW>
__device__ __forceinline__ void fold_jobs(Ctx<NW, FEW> &c, State &r, uint64_t *dlog, uint64_t jobs) {
  const uint32_t lo = c.vhost | ((uint32_t)NBOS_D_BATCH_START << 12) | (c.vjob << 16);
  r.digest = fold_decisions(r.digest, c.power, jobs, lo, (uint32_t)c.vstart);
  if (__builtin_expect(dlog != nullptr, 0)) {
    int64_t at = (int64_t)r.n_dec;
    for (uint64_t w = jobs; w != 0; w &= w - 1, at++) {
      const int j = (int)__builtin_ctzll(w);
      const uint64_t code = ((uint64_t)(uint32_t)lane_get(c.vstart, j) << 32) | (uint32_t)lane_get((int)lo, j);
      if (at < c.p.dlog_stride) dlog[at] = code;
    }
  }
  r.n_dec += (uint32_t)__builtin_popcountll(jobs);
  r.folded |= jobs;
}

// the job of session s finds no host at time T: it asks for one more host
template <int NW, bool FEW>
__device__ __forceinline__ void ask_for_host(Ctx<NW, FEW> &c, State &r, uint64_t *dlog, uint32_t s, int32_t T) {
  if (!(c.p.flags & NBOS_F_SCALE_OUT) || r.n_on >= c.p.Hmax) return;
  const int32_t up = add_in_range(T, c.p.boot);          // (a host that comes up at the end of the range ends the replay)
  r.status = up == NEVER ? (int32_t)NBOS_E_RANGE : r.status;
  const int h = r.n_on++;                              // hosts are added in order and never go
  r.prov -= (int64_t)c.p.G * T;
  c.m.ready[h] = up;
  r.up_t = r.next_up == h ? up : r.up_t;
  r.latest_up = max(r.latest_up, up);
  fold_jobs(c, r, dlog, r.jobs & ~r.todo & ~r.folded);
  const uint64_t code = decision_code(T, NBOS_D_BATCH_HOST, s, 0u, (uint32_t)h);
  r.digest = r.digest * DIGEST_PRIME + code;
  if (__builtin_expect(dlog != nullptr, 0)) {
    if ((int64_t)r.n_dec < c.p.dlog_stride) dlog[r.n_dec] = code;
  }
  r.n_dec++;
}

template <int NW, bool FEW>
__global__ void __launch_bounds__(WAVE) nbos_replay_batch_kernel(KParams p) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int rep = launch_slot_replay(p);
  const int lane = threadIdx.x;
  if (rep >= p.n_replays) return;

  const int trace = p.trace_of_replay[rep];
  const int64_t ev_lo = p.ev_offset[trace], ev_hi = p.ev_offset[trace + 1];
  const int s_lo = p.sess_offset[trace];
  const int n_sess = p.sess_offset[trace + 1] - s_lo;
  uint64_t *const dlog = p.dlog ? p.dlog + (int64_t)rep * p.dlog_stride : nullptr;

  Lds m;
  unsigned char *q = lds_raw;
  const size_t n4 = (size_t)((p.n_cap + 3) / 4 * 4);   // (read four at a time)
  m.hist = (uint32_t *)q;           q += (32 + WAVE) * 4;
  m.stage_t = (int32_t *)q;         q += (WAVE + 4) * 4;
  m.stage_k = (uint32_t *)q;        q += (WAVE + 4) * 4;
  m.time = (int32_t *)q;            q += n4 * 4;
  m.meta = (uint32_t *)q;           q += n4 * 4;
  m.mid_t = (int32_t *)q;           q += FEW ? 0 : (MID_CAP + 4) * 4;              // (and a word where nothing is kept)
  m.mid_k = (uint32_t *)q;          q += FEW ? 0 : (MID_CAP + 4) * 4;
  m.ready = (int32_t *)q;

  if (lane < 32) m.hist[lane] = 0;
  for (int s = lane; s < (int)n4; s += WAVE) { m.time[s] = 0; m.meta[s] = 0; }
  wave_sync();
  for (int s = lane; s < n_sess; s += WAVE) m.meta[s] = ((uint32_t)p.sess_gpus[s_lo + s] - 1u) << G_SHIFT;
  __syncthreads();

  Ctx<NW, FEW> c{p, m, lane, n_sess};
#pragma unroll
  for (int s = 0; s < c.NS; s++) {
    // the hosts that are there from the start are on the level of the slots that are not; the others count as full
    const int n = min(max(p.H0 - 512 * s - 64 * (lane % c.PER), 0), 64);
    const uint64_t on = n == 64 ? ~0ull : (1ull << n) - 1ull;
    const int level = lane / c.PER;
    const uint64_t bits = level == NGPU - p.G ? on : c.ALL_LEVELS & (level == NGPU) ? ~on : 0ull;
    c.lo[s] = (uint32_t)bits;
    c.hi[s] = (uint32_t)(bits >> 32);
  }
  c.qt = NEVER; c.qk = 0;
  c.vt = 0; c.vfd = 0; c.vjob = 0; c.vstart = 0; c.vhost = 0;
  c.power = digest_powers(lane);
  State r;
  memset(&r, 0, sizeof r);
  r.q_t = NEVER; r.up_t = NEVER;
  r.win_t = ALL; r.win = 1024;
  r.mid_t = ALL; r.mid_win = 1 << 17;
  r.p_f = -1;
  r.next_up = p.H0; r.n_on = p.H0;
  r.digest = 0xCBF29CE484222325ULL;
  // per lane: sums over jobs, their latest finish, the longest wait
  uint64_t sum_dur = 0, g_exec = 0, sum_wait = 0;
  uint32_t sum_g = 0;
  int32_t latest = 0, max_wait = 0;

  // the events: one per lane per tile, next tile in flight
  PROF_BEGIN();
  int32_t nt = 0, nd = 0, ns = 0;
  if (ev_lo < ev_hi) {
    const int64_t at = min(ev_lo + lane, ev_hi - 1);
    nt = p.ev_time[at]; nd = p.ev_dur[at]; ns = p.ev_sk[at];
  }
  for (int64_t cur = ev_lo; cur < ev_hi; cur += WAVE) {
    c.vt = nt;
    const int32_t vd = nd, vs = ns;
    if (cur + WAVE < ev_hi) {
      const int64_t at = min(cur + WAVE + lane, ev_hi - 1);
      nt = p.ev_time[at]; nd = p.ev_dur[at]; ns = p.ev_sk[at];
    }
    const bool is_cell = (cur + lane < ev_hi) & (((uint32_t)vs >> 24) == NBOS_EV_CELL);
    const uint32_t sid = (uint32_t)vs & 0xFFFFu;      // (every event of a trace has a session, below 2^16)
    wave_sync();
    const int32_t rt = m.time[sid];
    const uint32_t rm = m.meta[sid];
    // a cell whose session's previous job has started and outlasts it is dropped
    const bool drop = is_cell & (rt > c.vt);
    c.vfd = (int32_t)((uint32_t)p.batch_delay + (uint32_t)vd);
    c.vjob = sid | (((rm >> G_SHIFT) & 7u) << 16);
    if constexpr (FEW) {
      c.vsid = sid;
    } else {
      // lanes whose session has an earlier lane in the tile look again at their turn: every lane's mark goes to its session's
      // record, in bits that are 0 there, and the lowest lane's is the largest
      atomicMax(is_cell & !drop ? &m.meta[sid] : m.stage_k + WAVE, rm | ((uint32_t)(WAVE - lane) << 16));
      wave_sync();
      const uint32_t first = m.meta[sid];
      wave_sync();
      m.meta[sid] = rm;
      c.vjob |= ((first >> 16) & 127u) != (uint32_t)(WAVE - lane) ? SLOW : 0u;
    }
    r.c_total += (uint32_t)__builtin_popcountll(wballot(is_cell));
    r.todo = wballot(is_cell & !drop);
    r.jobs = r.todo;
    r.saved = 0; r.folded = 0;
    PROF(PC_TILE, 1);
    while (r.todo != 0) {
      [[maybe_unused]] const uint64_t prof_jobs0 = r.jobs & ~r.todo;
      if (__builtin_expect(r.p_f >= 0, 0)) make_room(c, r);
      // ---- jobs that start when they first meet the scheduler, the listed completions due before each applied on the
      // way: a loop with nothing else in it and one way out. `bad` is negative when it ends: no job of the tile is left (lane
      // 63's time is looked at then: no later than any job to come), the last one finds no room in the lists, or what does not fit.
      int32_t other_t = min(r.up_t, r.win_t + 1) - 1;
      int i, L, set, g;
      int32_t T, f, bad;
      uint32_t job;
      auto look_at_next = [&]() {
        i = (int)__builtin_ctzll(r.todo | (1ull << 63));
        job = (uint32_t)lane_get((int)c.vjob, i);
        T = r.now = max(lane_get(c.vt, i), r.now);
        f = (int32_t)((uint32_t)T + (uint32_t)lane_get(c.vfd, i));      // (below 2^32)
        while (r.q_t <= T) {
          const uint32_t k = r.q_k;
          pop_completion(c, r);
          give_back(c, k & HOST_MASK, (int)((k >> G_SHIFT) & 7u) + 1);
        }
        L = best_lane(c, set);
        g = (int)((job >> 16) & 7u) + 1;
        // (a long queue can push a job beyond the int32 time range: f + 1 is negative then)
        bad = (r.todo == 0 ? -1 : 0) | (int32_t)job | (NGPU - L / c.PER - g) | (other_t - T) | (int32_t)((uint32_t)f + 1u);
      };
      look_at_next();
      while (__builtin_expect(bad >= 0, 1)) {
        uint32_t wl = (uint32_t)lane_get((int)c.lo[0], L), wh = (uint32_t)lane_get((int)c.hi[0], L);
        if constexpr (Ctx<NW, FEW>::NS == 2) {
          const uint32_t vl = (uint32_t)lane_get((int)c.lo[1], L), vh = (uint32_t)lane_get((int)c.hi[1], L);
          wl = set ? vl : wl; wh = set ? vh : wh;
        }
        const uint32_t h = (uint32_t)__builtin_ctzll(((uint64_t)wh << 32) | wl) | ((uint32_t)(L % c.PER) << 6) | ((uint32_t)set << 9);
        if constexpr (Ctx<NW, FEW>::ALL_LEVELS) {
          const uint32_t from = 1u << L;
          flip_host(c, from | (from << g), h);
        } else {
          // from lane L to lane L + 8 g, which is not there for a host that is full now (8 g in two steps: a shift is by 63 at most)
          const uint64_t from = 1ull << L;
          flip_host(c, from | ((from << (4 * g)) << (4 * g)), h);
        }
        c.vstart = (int32_t)lane_set((uint32_t)c.vstart, (uint32_t)i, (uint32_t)T);
        c.vhost = lane_set(c.vhost, (uint32_t)i, h);
        r.todo &= r.todo - 1;
        if constexpr (FEW) {
          // of its session's lanes the earlier ones are not the latest job any more (nor the later ones, for now), and
          // arrivals that it outlasts are dropped
          const uint64_t same = wballot(c.vsid == (job & 0xFFFFu)), gone = same & wballot(c.vt < f) & r.todo;
          r.saved = (r.saved | same) & ~(1ull << i);
          r.todo ^= gone;
          r.jobs ^= gone;
        }
        if (f <= (FEW ? r.win_t : r.mid_t)) {
          const uint32_t k = h | ((uint32_t)(g - 1) << G_SHIFT);
          if (((r.win_t - f) | (Q_CAP - 1 - r.qe)) >= 0) {
            insert_completion(c, r, f, k);
          } else {
            const bool mid = !FEW & (f > r.win_t) & (r.mid_n < MID_CAP);
            if constexpr (!FEW) {
              const int at = mid ? r.mid_n : MID_CAP;
              c.m.mid_t[at] = f;
              c.m.mid_k[at] = k;
              r.mid_n += mid ? 1 : 0;
            }
            r.p_f = mid ? -1 : f;
            r.p_k = k;
            other_t = mid ? other_t : -1;
          }
        }
        look_at_next();
      }
      PROF(PC_ROUND, __builtin_popcountll((r.jobs & ~r.todo) ^ prof_jobs0));
      if ((r.todo == 0) | (r.p_f >= 0)) continue;
      // ---- one job that does not start like that ----
      save_records(c, r);
      const uint32_t s = job & 0xFFFFu;
      if (!FEW && __builtin_expect((job & SLOW) != 0u, 0)) {
        wave_sync();
        const uint64_t here = 1ull << i, gone = uni(m.time[s]) > lane_get(c.vt, i) ? here : 0ull;    // its previous job has not finished
        r.todo ^= gone;
        r.jobs ^= gone;
        c.vjob = in_mask(here) ? c.vjob & ~SLOW : c.vjob;
        PROF(PC_DROP, 1);
        continue;
      }
      bool asked = false;
      for (;;) {
        // what happens to the hosts up to T
        while (due_time(r) <= T) {
          if (r.win_t < min(r.q_t, r.up_t)) {
            PROF(PC_FAIL, 0);
            refill(c, r, min(T, r.up_t));
            PROF(PC_TIMER_OTHER, 1);
            continue;
          }
          const bool listed = r.q_t <= r.up_t;
          const uint32_t k = listed ? r.q_k : (uint32_t)r.next_up | ((uint32_t)(p.G - 1) << G_SHIFT);
          r.next_up += listed ? 0 : 1;
          if (__builtin_expect(listed, 1)) {
            pop_completion(c, r);
          } else {
            wave_sync();
            r.up_t = r.next_up < r.n_on ? uni(m.ready[r.next_up]) : NEVER;
          }
          give_back(c, k & HOST_MASK, (int)((k >> G_SHIFT) & 7u) + 1);
        }
        if (fits(c, best_lane(c, set), g)) break;             // it starts at T, in the loop above
        if (!asked) ask_for_host(c, r, dlog, s, T);         // (it starts before this path is left)
        asked = true;
        // the listed completions, instant by instant, for as long as none leaves a host with the GPUs idle
        other_t = min(r.up_t - 1, r.win_t);
        bool found = false;
        while (!found & (r.q_t <= other_t)) {
          T = r.q_t;
          do {
            const uint32_t k = r.q_k;
            pop_completion(c, r);
            found = found | fits(c, give_back(c, k & HOST_MASK, (int)((k >> G_SHIFT) & 7u) + 1), g);
          } while (r.q_t == T);
        }
        if (found) break;
        T = due_time(r);                                   // (at the end of a window nothing need happen: no harm)
        r.status = T == NEVER ? (int32_t)NBOS_E_RANGE : r.status;      // (cannot be: a job fits once the others are over)
        if (r.status != NBOS_OK) break;
      }
      // (a start beyond the time range ends the replay)
      r.status = (uint32_t)T + (uint32_t)lane_get(c.vfd, i) >= 0x7FFFFFFFu ? (int32_t)NBOS_E_RANGE : r.status;
      if (r.status != NBOS_OK) break;
      r.now = T;
      PROF(PC_FAIL, 1);
    }
    if (r.status != NBOS_OK) break;
    save_records(c, r);
    // the tile's jobs: digest, sums, waits (those that start at once are all in the histogram's bin of the container start)
    fold_jobs(c, r, dlog, r.jobs & ~r.folded);
    r.c_started += (uint32_t)__builtin_popcountll(r.jobs);
    const bool mine = in_mask(r.jobs);
    const uint32_t one = mine ? 1u : 0u, g = ((c.vjob >> 16) & 7u) + 1u;
    const uint32_t d = one * (uint32_t)vd, wait = one * (uint32_t)(c.vstart - c.vt);
    r.c_imm += (uint32_t)__builtin_popcountll(wballot(mine & (wait == 0u)));
    sum_dur += d;
    g_exec += g * d;                               // (8 * NBOS_MAX_DUR_MS is below 2^32)
    sum_g += one * g;
    sum_wait += wait;
    max_wait = max(max_wait, (int32_t)wait);
    latest = max(latest, mine ? job_finish(c.vstart, c.vfd) : 0);
    const int b = min(32 - __builtin_clz(wait + (uint32_t)p.batch_delay), 31);      // (of a wait of 0: not looked at)
    atomicAdd(&m.hist[wait != 0u ? b : 32 + lane], 1u);
    PROF(PC_TILE, 0);
  }
  if (ev_lo < ev_hi) {
    const int32_t tl = p.ev_time[ev_hi - 1];
    r.t_end = r.t_end > tl ? r.t_end : tl;
  }

  __syncthreads();
  const int64_t sum_dur_all = (int64_t)wave_sum64(sum_dur), g_exec_all = (int64_t)wave_sum64(g_exec), sum_g_all = (int64_t)wave_sum64(sum_g),
                sum_wait_all = (int64_t)wave_sum64(sum_wait);
  const int32_t longest = (int32_t)~wave_min(~(uint32_t)max_wait);
  const int32_t over = max((int32_t)~wave_min(~(uint32_t)latest), r.latest_up);
  const int32_t t_end = r.t_end > over ? r.t_end : over;
  nbos_stats *out = p.stats + rep;
  // the jobs that started at once: all in the bin of the container start
  const int b0 = p.batch_delay == 0 ? 0 : 32 - __builtin_clz((uint32_t)p.batch_delay);
  if (lane < 32) out->delay_hist[lane] = m.hist[lane] + (lane == b0 ? r.c_imm : 0u);
  if (lane == 0) {
    const int64_t sum_delay = sum_wait_all + (int64_t)r.c_started * p.batch_delay;
    out->status = r.status; out->n_decisions = r.n_dec;
    out->sessions_placed = 0; out->sessions_rejected = 0;
    out->cells_total = r.c_total; out->cells_immediate = r.c_imm; out->cells_started = r.c_started;
    out->cells_queued = r.c_started - r.c_imm; out->cells_aborted = 0;
    out->cells_dropped_busy = r.c_total - r.c_started; out->cells_dropped_unplaced = 0;
    out->executor_reused = 0; out->migrations = 0;
    out->scale_out_hosts = (uint32_t)(r.n_on - p.H0); out->scale_in_hosts = 0; out->peak_hosts = (uint32_t)r.n_on;
    out->migrations_warm = 0;
    out->max_delay_ms = r.c_started > 0 ? longest + p.batch_delay : 0; out->t_end_ms = t_end;
    out->sum_delay_ms = sum_delay; out->sum_tct_ms = sum_dur_all + sum_delay;
    out->gpu_ms_executed = g_exec_all; out->gpu_ms_committed = g_exec_all + sum_g_all * p.batch_delay;
    out->gpu_ms_provisioned = r.prov + (int64_t)r.n_on * p.G * t_end;
    out->reservation_gpu_ms = 0; out->sub_gpu_ms = 0; out->replica_ms = 0;
    out->digest = r.digest;
  }
  PROF_OUT(rep);
}

}  // namespace batchk
}  // namespace
