// nbos_kernel_batch.hpp — replay of the Batch baseline (the paper's "Baselines" section): every cell is a job of its
// own, first come first served, a container per job. One workgroup (one wave64) per replay, any cluster
// size up to NBOS_MAX_HOSTS.
//
// fin[h][8] in LDS: the "busy until" times of host h's GPUs, one row of 32 bytes per host, sorted ascending; slots
// beyond G hold NEVER. A GPU is held at time t iff fin > t; the host has g idle GPUs from fin[g-1] on. A host
// that is off holds NEVER everywhere, one that is being provisioned its ready time in all G slots: it has
// no idle GPU before it is ready, and needs no other mark.
// In registers, lane l and chunk j (j < NCH) for host h = 64 j + l:
//   key[j]  (slots with fin > T) << 10 | h at the time T of the last look; slots beyond G count too (the
//           same number on every host)
//   nx[j]   the earliest fin beyond that T: key[j] is good until then
// A job takes the ready host with the fewest held GPUs (ties: lowest index), i.e. the smallest key, and
// fits there or nowhere: its GPUs are idle iff (key >> 10) + g <= 8. So one minimum over the keys answers
// both questions, and a look at time T first brings those keys up to date whose nx has passed (the hosts of
// a completion or two per job). Allocating the g GPUs that have been free longest on a sorted row is one
// median per slot, lane = slot: new[k] = median(old[k], finish, old[k + g]).
// Sessions in LDS, 8 bytes each: time (busy until, or submit time while the job waits in the queue), and
// duration | (g - 1) << 27 | waiting. fifo: ring of waiting jobs (16-bit session ids), at most one per session.
//
// The CPU reference runs completions and "host ready" as timers and looks at the queue after each
// instant. Here nothing is queued as a timer. The job at the head of the queue first meets the scheduler
// at T0 = max(its submit time, the time the previous head got its GPUs). If some ready host has g idle
// GPUs at T0 it starts there. Otherwise nothing is allocated until it starts (it blocks the queue), so
// the busy-until times do not change while it waits and the instant it starts is known in closed form:
// E = min over hosts of f[g-1], which is the time of a completion or of a host turning ready, i.e. an
// instant at which the reference serves the queue. A GPU with f <= E is free at E exactly when the
// reference has applied every completion of that instant. The queue is advanced up to the time of each
// arriving event before the event is looked at (timers due at or before an arrival run before it), and to
// the end after the last one.
//
// Bound by the latency of the serial chain of jobs (one wave per replay): about 200 instructions and six LDS
// accesses per job on 512 hosts, 608 ns (256 replays of 250,000 jobs: 152 ms). The version before, whose jobs
// scanned the rows of every chunk that could take them, took 543 ms. Control flow is uniform throughout: a store
// that one lane would do is done by all lanes (same value, same address), as an exec-masked region costs 40
// clocks and makes the compiler rebuild the branches around it.
#pragma once
#include "nbos_common.hpp"

namespace {
namespace batchk {

constexpr int32_t WAITING = 1 << 30;
constexpr int G_SHIFT = 27;
constexpr int32_t DUR_MASK = (1 << G_SHIFT) - 1;      // a duration is at most NBOS_MAX_DUR_MS < 2^27

struct Lds {
  int32_t *fin;
  uint32_t *hist;               // 32 bins, and behind them a word per lane for the lanes that an LDS atomic is not for
  int2 *sess;
  uint16_t *fifo;
};

template <int NCH>
struct Ctx {
  const KParams &p;
  Lds m;
  int lane;
  int own_slot;                 // -1 in lane 0, elsewhere the lane's own word behind the histogram
  int ring;                     // ring capacity
  uint64_t *dlog;
  uint32_t key[NCH];
  int32_t nx[NCH];
  uint32_t vsid;                // session of this lane's event in the current tile (~0 if none)
  int32_t w_s, w_t, w_d;        // jobs read ahead from the queue, one per lane: session, its record
};

// (status is only ever set by a select: a conditional store to it next to one to head_E is merged into one store
// through a chosen pointer, which puts both into memory and every value that depends on them into vector registers)
struct State {
  uint32_t n_dec, c_total, c_started, c_imm, c_busy;
  int64_t sum_dur, g_exec, sum_g, sum_wait, prov;
  uint64_t digest;
  uint64_t dirty;               // lanes of the current tile whose prefetched record is stale
  int32_t q_head, q_n;          // ring: index of the head, jobs waiting (the head included)
  int32_t w_at, w_n;            // jobs read ahead: the next one, how many
  int32_t h_s, h_t, h_dur, h_g; // the head of the queue
  int32_t head_T;               // when the head looks for a host next: as it becomes the head, or once a host can
                                // give it its GPUs (NEVER: the queue is empty)
  int32_t last_T;               // when the last job got its GPUs
  int32_t n_on, max_wait;
  int32_t lazy_max, t_end;
  int32_t status;               // NBOS_OK, or NBOS_E_RANGE once a time leaves the int32 range
};

template <class C>
__device__ __forceinline__ void decide(C &c, State &r, int32_t now, uint32_t outcome, uint32_t s, uint32_t host) {
  const uint64_t code = decision_code(now, outcome, s, 0u, host);
  r.digest = r.digest * DIGEST_PRIME + code;
  if (__builtin_expect(c.dlog != nullptr, 0)) {
    if ((int64_t)r.n_dec < c.p.dlog_stride) c.dlog[r.n_dec] = code;
  }
  r.n_dec++;
}

// smallest key at time T: the host that takes the next job, if that fits (see fits)
template <int NCH>
__device__ __forceinline__ uint32_t best_host(Ctx<NCH> &c, int32_t T) {
  int32_t soonest = c.nx[0];
#pragma unroll
  for (int j = 1; j < NCH; j++) soonest = min(soonest, c.nx[j]);
  if (wballot(soonest <= T) != 0) {
    wave_sync();
#pragma unroll
    for (int j = 0; j < NCH; j++) {
      if (__builtin_expect(wballot(c.nx[j] <= T) != 0, 0)) {      // (the chunk's other keys come out as they were)
        const int4 *row = (const int4 *)(c.m.fin + NGPU * (j * WAVE + c.lane));
        const int4 a = row[0], b = row[1];
        const int32_t f[NGPU] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        uint32_t held = 0;
        int32_t next = NEVER;
#pragma unroll
        for (int k = NGPU - 1; k >= 0; k--) {
          held += f[k] > T ? 1u : 0u;
          next = f[k] > T ? f[k] : next;
        }
        c.key[j] = (held << 10) | (uint32_t)(j * WAVE + c.lane);
        c.nx[j] = next;
      }
    }
  }
  uint32_t best = c.key[0];
#pragma unroll
  for (int j = 1; j < NCH; j++) best = umin(best, c.key[j]);
  return wave_min(best);
}
__device__ __forceinline__ bool fits(uint32_t key, int g) { return (int)(key >> 10) + g <= NGPU; }

// earliest time at which some host has g idle GPUs if nothing new is allocated
template <int NCH>
__device__ __forceinline__ int32_t earliest_free(const Ctx<NCH> &c, int g) {
  wave_sync();
  int32_t y = NEVER;
#pragma unroll
  for (int j = 0; j < NCH; j++) y = min(y, c.m.fin[NGPU * (j * WAVE + c.lane) + g - 1]);
  return (int32_t)wave_min((uint32_t)y);
}

// The key and the next change of the host in chunk jh, lane `mine`: found by halving the chunks (a few uniform
// branches; touching the registers of all chunks takes five vector instructions for each).
template <int LO, int HI, int NCH>
__device__ __forceinline__ void note_allocation(Ctx<NCH> &c, int jh, bool mine, uint32_t key, int32_t finish) {
  if constexpr (HI - LO == 1) {
    c.key[LO] = mine ? key : c.key[LO];
    c.nx[LO] = mine ? min(c.nx[LO], finish) : c.nx[LO];
  } else {
    constexpr int MID = (LO + HI) / 2;
    if (jh < MID) note_allocation<LO, MID>(c, jh, mine, key, finish);
    else note_allocation<MID, HI>(c, jh, mine, key, finish);
  }
}

// the job of session s gets g GPUs of the host with this key at time T
template <int NCH>
__device__ __forceinline__ void start_job(Ctx<NCH> &c, State &r, uint32_t s, int32_t T, int32_t t_submit, int32_t dur, int g, uint32_t key) {
  const int h = (int)(key & 1023u);
  // a long queue can push a job beyond the int32 time range: the replay ends as invalid (the sum stays below 2^32)
  const uint32_t fin = (uint32_t)T + (uint32_t)c.p.batch_delay + (uint32_t)dur;
  r.status = fin >= 0x7FFFFFFFu ? (int32_t)NBOS_E_RANGE : r.status;
  const int32_t finish = (int32_t)fin;
  // the g GPUs of the row that have been free longest are held until `finish` (see the file header)
  wave_sync();
  int32_t *row = c.m.fin + NGPU * h;
  const int k = c.lane & 7;
  const int32_t own = row[k];
  int32_t up = row[(k + g) & 7];
  up = k + g < NGPU ? up : NEVER;
  note_allocation<0, NCH>(c, h >> 6, c.lane == (h & 63), key + ((uint32_t)g << 10), finish);
  r.dirty |= wballot(c.vsid == s);
  r.c_started++;
  r.sum_dur += dur;
  r.g_exec += (int64_t)g * dur;
  r.sum_g += g;
  if (T == t_submit) {
    r.c_imm++;                                    // its delay is the container start: histogram and sum follow at the end
  } else {
    const int32_t wait = T - t_submit, delay = wait + c.p.batch_delay;
    r.sum_wait += wait;
    r.max_wait = r.max_wait > wait ? r.max_wait : wait;
    const int b = min(32 - __builtin_clz((uint32_t)delay), 31);      // (delay > 0)
    atomicAdd(&c.m.hist[c.own_slot < 0 ? b : c.own_slot], 1u);
  }
  r.lazy_max = r.lazy_max > finish ? r.lazy_max : finish;
  r.last_T = T;
  decide(c, r, T, NBOS_D_BATCH_START, s, (uint32_t)h);
  row[k] = med3(own, finish, up);                 // (every eighth lane the same)
  c.m.sess[s] = make_int2(finish, (g - 1) << G_SHIFT);
}

// The head finds no host at time T: it asks for one more host, and its start time is worked out (a host has the
// GPUs idle then: it does not come here a second time).
template <int NCH>
__device__ __forceinline__ void head_waits(Ctx<NCH> &c, State &r, int32_t T) {
  int32_t first_free = earliest_free(c, r.h_g);
  if ((c.p.flags & NBOS_F_SCALE_OUT) && r.n_on < c.p.Hmax) {
    const int64_t up = (int64_t)T + c.p.boot;
    r.status = up >= 0x7FFFFFFFLL ? (int32_t)NBOS_E_RANGE : r.status;
    const int32_t ra = (int32_t)up;
    const int h = r.n_on++;                       // hosts are added in order and never go
    r.prov -= (int64_t)c.p.G * T;
    c.m.fin[NGPU * h + (c.lane & 7)] = (c.lane & 7) < c.p.G ? ra : NEVER;      // all its GPUs are idle once it is up
#pragma unroll
    for (int j = 0; j < NCH; j++) c.nx[j] = h - c.lane == j * WAVE ? ra : c.nx[j];
    r.lazy_max = r.lazy_max > ra ? r.lazy_max : ra;
    decide(c, r, T, NBOS_D_BATCH_HOST, (uint32_t)r.h_s, (uint32_t)h);
    first_free = first_free < ra ? first_free : ra;
  }
  r.status = first_free < T ? (int32_t)NBOS_E_RANGE : r.status;      // (cannot be; the loop might not end)
  r.head_T = first_free;
}

// the next waiting job becomes the head; jobs are read ahead from the ring, up to 64 at a time
template <int NCH>
__device__ __forceinline__ void next_head(Ctx<NCH> &c, State &r) {
  if (r.w_at == r.w_n) {
    wave_sync();
    r.w_n = r.q_n < WAVE ? r.q_n : WAVE;
    r.w_at = 0;
    int at = r.q_head + min(c.lane, r.w_n - 1);
    at = at >= c.ring ? at - c.ring : at;
    c.w_s = c.m.fifo[at];
    const int2 rec = c.m.sess[c.w_s];
    c.w_t = rec.x; c.w_d = rec.y;
  }
  const int32_t d = lane_get(c.w_d, r.w_at);
  r.h_s = lane_get(c.w_s, r.w_at);
  r.h_t = lane_get(c.w_t, r.w_at);
  r.h_dur = d & DUR_MASK;
  r.h_g = ((d >> G_SHIFT) & 7) + 1;
  r.w_at++;
  r.head_T = max(r.h_t, r.last_T);
}

// an arrival that cannot start yet waits at the end of the queue
template <int NCH>
__device__ __forceinline__ void join_queue(Ctx<NCH> &c, State &r, uint32_t s, int32_t t, int32_t dur, int g) {
  int tail = r.q_head + r.q_n;
  tail = tail >= c.ring ? tail - c.ring : tail;
  c.m.fifo[tail] = (uint16_t)s;
  c.m.sess[s] = make_int2(t, dur | ((g - 1) << G_SHIFT) | WAITING);
  r.dirty |= wballot(c.vsid == s);
  r.q_n++;
}

template <int NCH>
__global__ void __launch_bounds__(WAVE) nbos_replay_batch_kernel(KParams p) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int rep = launch_slot_replay(p);
  const int lane = threadIdx.x;
  if (rep >= p.n_replays) return;

  const int trace = p.trace_of_replay[rep];
  const int64_t ev_lo = p.ev_offset[trace], ev_hi = p.ev_offset[trace + 1];
  const int s_lo = p.sess_offset[trace];
  const int n_sess = p.sess_offset[trace + 1] - s_lo;

  Lds m;
  unsigned char *q = lds_raw;
  m.fin = (int32_t *)q;             q += (size_t)NCH * WAVE * NGPU * 4;
  m.hist = (uint32_t *)q;           q += (32 + WAVE) * 4;
  m.sess = (int2 *)q;               q += (size_t)p.n_cap * 8;
  m.fifo = (uint16_t *)q;

  for (int i = lane; i < NCH * WAVE * NGPU; i += WAVE) m.fin[i] = (i >> 3) < p.H0 && (i & 7) < p.G ? 0 : NEVER;
  if (lane < 32) m.hist[lane] = 0;
  for (int s = lane; s < n_sess; s += WAVE) m.sess[s] = make_int2(0, ((int)p.sess_gpus[s_lo + s] - 1) << G_SHIFT);
  __syncthreads();

  Ctx<NCH> c{p, m, lane, lane == 0 ? -1 : 32 + lane, p.n_cap + 1, p.dlog ? p.dlog + (int64_t)rep * p.dlog_stride : nullptr};
#pragma unroll
  for (int j = 0; j < NCH; j++) {
    const int h = j * WAVE + lane;
    c.key[j] = ((h < p.H0 ? (uint32_t)(NGPU - p.G) : (uint32_t)NGPU) << 10) | (uint32_t)h;
    c.nx[j] = NEVER;
  }
  c.w_s = 0; c.w_t = 0; c.w_d = 0;
  State r;
  memset(&r, 0, sizeof r);
  r.digest = 0xCBF29CE484222325ULL;
  r.head_T = NEVER;
  r.n_on = p.H0;

  // the events: one per lane per tile, next tile in flight; after the last one the queue is served to its end
  int64_t base = ev_lo;
  int32_t vt = 0, vd = 0, vs = 0, nt = 0, nd = 0, ns = 0;
  if (base < ev_hi) {
    const int64_t at = min(base + lane, ev_hi - 1);
    nt = p.ev_time[at]; nd = p.ev_dur[at]; ns = p.ev_sk[at];
  }
  bool final = false;
  while (!final) {
    uint64_t todo = 0;
    int2 rec = make_int2(0, 0);             // prefetched session record of this lane's event
    if (base < ev_hi) {
      vt = nt; vd = nd; vs = ns;
      const int64_t cur = base;
      base += WAVE;
      if (base < ev_hi) {
        const int64_t at = min(base + lane, ev_hi - 1);
        nt = p.ev_time[at]; nd = p.ev_dur[at]; ns = p.ev_sk[at];
      }
      const bool valid = cur + lane < ev_hi;
      const bool is_cell = valid && ((uint32_t)vs >> 24) == NBOS_EV_CELL;
      const uint32_t sid = (uint32_t)vs & 0xFFFFFFu;
      c.vsid = is_cell ? sid : 0xFFFFFFFFu;
      wave_sync();
      rec = m.sess[sid];                    // (every event of a trace has a session)
      // a cell whose session's job has started and outlasts it is dropped, whatever happens until then
      const bool drop = is_cell && !(rec.y & WAITING) && rec.x > vt;
      r.dirty = 0;
      r.c_total += (uint32_t)__builtin_popcountll(wballot(is_cell));
      r.c_busy += (uint32_t)__builtin_popcountll(wballot(drop));
      todo = wballot(is_cell && !drop);
      if (ev_hi - cur <= WAVE) {
        const int32_t tl = lane_get(vt, (int)(ev_hi - cur - 1));
        r.t_end = r.t_end > tl ? r.t_end : tl;
      }
    } else {
      final = true;
    }
    // one iteration per look at a job: the head of the queue if it meets the scheduler at or before the
    // next arrival (what is due at or before an arrival comes first), else the arrival
    while (r.status == NBOS_OK) {
      int i = 0;
      int32_t t = NEVER;
      if (todo != 0) { i = (int)__builtin_ctzll(todo); t = lane_get(vt, i); }
      else if (!final || r.q_n == 0) break;
      uint32_t s;
      int32_t T, t_submit, dur;
      int g;
      if (r.head_T <= t) {
        T = r.head_T; s = (uint32_t)r.h_s; t_submit = r.h_t; dur = r.h_dur; g = r.h_g;
      } else {
        todo &= todo - 1;
        s = (uint32_t)lane_get(vs, i) & 0xFFFFFFu;
        int32_t tm = lane_get(rec.x, i), gq = lane_get(rec.y, i);
        if (__builtin_expect(((r.dirty >> i) & 1u) != 0, 0)) {
          wave_sync();
          const int2 now = m.sess[s];
          tm = uni(now.x); gq = uni(now.y);
        }
        if (__builtin_expect(tm > t || (gq & WAITING), 0)) { r.c_busy++; continue; }   // its previous job has not finished
        T = t; t_submit = t; dur = lane_get(vd, i);
        g = ((gq >> G_SHIFT) & 7) + 1;
        if (r.q_n > 0) { join_queue(c, r, s, t, dur, g); continue; }
      }
      const uint32_t key = best_host(c, T);
      if (__builtin_expect(fits(key, g), 1)) {
        start_job(c, r, s, T, t_submit, dur, g, key);
        if (r.q_n > 0) {                          // it was the head
          r.q_head = r.q_head + 1 == c.ring ? 0 : r.q_head + 1;
          r.q_n--;
          r.head_T = NEVER;
          if (r.q_n > 0) next_head(c, r);
        }
      } else {
        if (r.q_n == 0) {
          join_queue(c, r, s, t, dur, g);
          r.h_s = (int32_t)s; r.h_t = t; r.h_dur = dur; r.h_g = g;
          r.w_at = 0; r.w_n = 0;
        }
        head_waits(c, r, T);
      }
    }
    if (r.status != NBOS_OK) break;
  }

  __syncthreads();
  const int32_t t_end = r.t_end > r.lazy_max ? r.t_end : r.lazy_max;
  nbos_stats *out = p.stats + rep;
  // the jobs that started at once: all in the bin of the container start
  const int b0 = p.batch_delay == 0 ? 0 : 32 - __builtin_clz((uint32_t)p.batch_delay);
  if (lane < 32) out->delay_hist[lane] = m.hist[lane] + (lane == b0 ? r.c_imm : 0u);
  if (lane == 0) {
    const int64_t sum_delay = r.sum_wait + (int64_t)r.c_started * p.batch_delay;
    out->status = r.status; out->n_decisions = r.n_dec;
    out->sessions_placed = 0; out->sessions_rejected = 0;
    out->cells_total = r.c_total; out->cells_immediate = r.c_imm; out->cells_started = r.c_started;
    out->cells_queued = r.c_started - r.c_imm; out->cells_aborted = 0;
    out->cells_dropped_busy = r.c_busy; out->cells_dropped_unplaced = 0;
    out->executor_reused = 0; out->migrations = 0;
    out->scale_out_hosts = (uint32_t)(r.n_on - p.H0); out->scale_in_hosts = 0; out->peak_hosts = (uint32_t)r.n_on;
    out->migrations_warm = 0;
    out->max_delay_ms = r.c_started > 0 ? r.max_wait + p.batch_delay : 0; out->t_end_ms = t_end;
    out->sum_delay_ms = sum_delay; out->sum_tct_ms = r.sum_dur + sum_delay;
    out->gpu_ms_executed = r.g_exec; out->gpu_ms_committed = r.g_exec + r.sum_g * p.batch_delay;
    out->gpu_ms_provisioned = r.prov + (int64_t)r.n_on * p.G * t_end;
    out->reservation_gpu_ms = 0; out->sub_gpu_ms = 0; out->replica_ms = 0;
    out->digest = r.digest;
  }
}

}  // namespace batchk
}  // namespace
