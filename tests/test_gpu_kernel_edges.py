"""The kernels at the edges of what each instance is compiled for, against the CPU oracle, bit for bit
(all outputs are integers: no tolerance)."""
import numpy as np
import pytest

from helpers import events_to_arrays
from paper_2503_20591_amd import tracegen as tg
from test_gpu_parity import as_batch, assert_same, gpu_run, rp  # noqa: F401  (rp: the fixture)

pytestmark = pytest.mark.gpu


def crowded(seed, hosts, G, sessions_per_host, cells_per_session, gap_s=5.0, dur_s=300.0, with_end=False):
    """A trace that fills ``hosts`` hosts of ``G`` GPUs: queues, blocked heads, several completions between events."""
    return tg.make_trace(seed, hosts * sessions_per_host, hosts * sessions_per_host * cells_per_session, ramp_ms=60_000,
                         gpus=lambda r, n: np.minimum(tg.gpus_uniform(r, n), G).astype(np.uint8),
                         gap=lambda r, s: tg.exp_ms(r, gap_s, s), dur=lambda r, s: tg.lognormal_ms(r, dur_s, 1.0, s),
                         with_end=with_end)


@pytest.mark.parametrize("grow", [False, True], ids=["fixed", "grow"])
@pytest.mark.parametrize("hosts,G", [(1, 8), (2, 1), (63, 8), (64, 3), (64, 8), (65, 8), (128, 2), (129, 1), (256, 4), (257, 3), (512, 2),
                                     (513, 1), (768, 2), (769, 3), (1024, 1), (1024, 2)])
def test_batch_kernel_at_its_chunk_edges(rp, oracle, hosts, G, grow):  # noqa: F811
    # 64 hosts to a word, 512 to a set of registers; of 8 slots per host those beyond G are held for ever (on up to 64
    # hosts the full ones have a lane of their own)
    b = tg.pack(tg.base_config(hosts_initial=hosts, hosts_max=hosts, gpus_per_host=G),
                [crowded(7, hosts, G, 3, 3), crowded(8, hosts, G, 2, 2)], [0, 1, 0], [1000, 1000, 1000], f"edge{hosts}")
    as_batch(b, delay=15_000, scale_out=grow)
    if grow:
        b.config.update(hosts_initial=max(1, hosts - 40), hosts_max=hosts, boot_delay_ms=20_000)
    st, logs = gpu_run(rp, b, log=True)
    assert_same(rp, oracle, b, st, logs)
    assert st["cells_queued"].max() > 0


def on_a_grid(seed, hosts, sessions, step_ms, flags, caps):
    """Every time of the trace is a multiple of ``step_ms``: the coarser, the more timers are due at one instant."""
    on_grid = lambda v: np.maximum(v // step_ms, 1) * step_ms  # noqa: E731
    tr = tg.make_trace(seed, sessions, sessions * 6, ramp_ms=300_000, gpus=lambda r, n: tg.gpus_uniform(r, n),
                       gap=lambda r, s: on_grid(tg.exp_ms(r, 40.0, s)), dur=lambda r, s: on_grid(tg.lognormal_ms(r, 200.0, 1.0, s)),
                       with_end=True)
    tr = (tr[0] // step_ms * step_ms, *tr[1:])
    return tg.pack(tg.base_config(hosts_initial=hosts, hosts_max=hosts, flags=flags), [tr], [0] * len(caps), list(caps), "refill")


def jobs_run(b, log):
    """Start and end of every job of a Batch replay, by the decision log and the trace (a cell that arrives before the
    session's job ends is dropped)."""
    delay, cells = b.config["batch_start_delay_ms"], [[] for _ in range(len(b.sess_gpus))]
    for t, d, sk in zip(b.ev_time.tolist(), b.ev_dur.tolist(), b.ev_sk.tolist()):
        if sk >> 24 == tg.EV_CELL:
            cells[sk & 0xFFFFFF].append((t, d))
    start, end, over = [], [], [-1] * len(cells)
    for code in log.tolist():
        if code >> 12 & 15 == 10:
            s, t = code >> 16 & 0xFFFF, code >> 32
            cell = next(c for c in cells[s] if c[0] >= over[s])
            cells[s] = cells[s][cells[s].index(cell) + 1:]
            over[s] = t + delay + cell[1]
            start.append(t)
            end.append(over[s])
    return np.array(start), np.array(end)


@pytest.mark.parametrize("grow", [False, True], ids=["fixed", "grow"])
@pytest.mark.parametrize("hosts,sessions,step_ms,delay,more_than,at_once",
                         [(40, 60, 1, 0, 0, 1), (40, 512, 1, 15_000, 63, 1), (64, 513, 1, 0, 63, 1), (100, 2000, 1, 15_000, 63, 1),
                          (100, 400, 600_000, 0, 63, 64), (100, 3000, 600_000, 0, 63, 64), (600, 3000, 60_000, 15_000, 512, 64),
                          (600, 6000, 1_200_000, 0, 512, 513), (520, 5000, 1000, 0, 512, 2), (40, 700, 100_000, 15_000, 63, 10),
                          (3, 700, 100_000, 15_000, 0, 2)])
def test_batch_completions_in_order(rp, oracle, hosts, sessions, step_ms, delay, more_than, at_once, grow):  # noqa: F811
    # the list of completions in registers (63) and the one in LDS (512 jobs, only with more sessions than that): refilled,
    # pushed into, overrun, and hundreds of jobs that end at one instant; the first and the last case never fill the registers
    b = as_batch(on_a_grid(9, hosts, sessions, step_ms, 0, [1000]), delay=delay, scale_out=grow)
    if grow:
        b.config.update(hosts_initial=max(1, hosts // 2), hosts_max=hosts, boot_delay_ms=20_000)
    st, logs = gpu_run(rp, b, log=True)
    assert_same(rp, oracle, b, st, logs)
    start, end = jobs_run(b, logs[0])
    assert len(start) == st["cells_started"][0] > 0
    change = np.concatenate([np.ones(len(start), int), -np.ones(len(end), int)])
    order = np.lexsort((change, np.concatenate([start, end])))         # at one instant jobs end before others start
    most = np.cumsum(change[order]).max()
    assert most > more_than and (more_than > 0 or most <= 63)
    assert grow or np.unique(end, return_counts=True)[1].max() >= at_once      # (added hosts spread the starts)


@pytest.mark.parametrize("hosts", [10, 64, 100, 600])
@pytest.mark.parametrize("sizes", [(62, 63, 64, 65, 128, 390), (63, 64, 65, 511, 512, 513, 700, 700)], ids=["few", "listed"])
def test_batch_crowds_of_completions(rp, oracle, hosts, sizes):  # noqa: F811
    # per size as many jobs that end at one instant (where the hosts take them all at once), a few before and after it, and
    # arrivals around it: crowds that just fit into the registers and the list, just do not, and two of them 1 ms apart
    rng, ev = np.random.default_rng(hosts), []
    for w, size in enumerate(sizes):
        at = 2_000_000 * w + 1_000_000
        ends = [at] * size + [at - 3, at - 1, at - 1, at + 1, at + 2] + ([at + 1] * 70 if w % 2 else [])
        for s, (start, end) in enumerate(zip(sorted(rng.integers(at - 900_000, at - 1000, len(ends))), rng.permutation(ends))):
            ev.append([int(start), tg.EV_CELL, s, int(end - start)])
        ev += [[at + int(d), tg.EV_CELL, len(ends) + k, 500 + k] for k, d in enumerate(sorted(rng.integers(-3, 4, 40)))]
    n = 1 + max(e[2] for e in ev)
    assert n <= 512 or sizes[-1] > 512
    t, d, sk = events_to_arrays(ev)
    gpus = np.where(rng.random(n) < 0.9, 1, 2).astype(np.uint8)
    b = tg.pack(tg.base_config(hosts_initial=hosts, hosts_max=hosts), [(t, d, sk, gpus)], [0, 0], [1000, 1000], "crowds")
    st, logs = gpu_run(rp, as_batch(b, delay=0, scale_out=False), log=True)
    assert_same(rp, oracle, b, st, logs, check=True)
    assert hosts < 100 or st["cells_started"].min() == len(ev)


@pytest.mark.parametrize("hosts", [1, 64, 65, 513])
@pytest.mark.parametrize("sessions", [1, 3, 60, 512, 513])
def test_batch_arrivals_of_one_session_in_a_tile(rp, oracle, hosts, sessions):  # noqa: F811
    # a session's next cell arrives up to 15 s (the container start) after the one before has ended, to the second: it is
    # dropped, or starts in the millisecond in which that one ends; both lanes of a tile of 64 events, or of two tiles
    on_grid = lambda v: np.maximum(v // 1000, 1) * 1000  # noqa: E731
    tr = tg.make_trace(31, sessions, max(sessions, 200) * 5 + 7, ramp_ms=60_000, gpus=tg.gpus_uniform,
                       gap=lambda r, s: on_grid(tg.exp_ms(r, 15.0, s)), dur=lambda r, s: on_grid(tg.exp_ms(r, 8.0, s)), with_end=True)
    b = tg.pack(tg.base_config(hosts_initial=hosts, hosts_max=hosts), [tr], [0, 0], [1000, 1000], "tile")
    st, logs = gpu_run(rp, as_batch(b, delay=15_000, scale_out=False), log=True)
    assert_same(rp, oracle, b, st, logs, check=True)
    assert st["cells_dropped_busy"].min() > 0


@pytest.mark.parametrize("grow", [False, True], ids=["fixed", "grow"])
@pytest.mark.parametrize("hosts,most", [(64, 16_140), (65, 15_935), (1024, 13_068)])
def test_batch_sessions_up_to_the_limit(rp, oracle, hosts, most, grow):  # noqa: F811
    # as many sessions as a call may have, and one more
    for sessions in (most, most + 1):
        rng = np.random.default_rng(hosts)
        t = np.sort(rng.integers(0, 600_000, 3_000)).astype(np.int32)
        d = rng.integers(1, 400_000, len(t)).astype(np.int32)
        sk = (rng.integers(sessions - 2_000, sessions, len(t)) | tg.EV_CELL << 24).astype(np.int32)
        b = tg.pack(tg.base_config(hosts_initial=hosts // 2 if grow else hosts, hosts_max=hosts),
                    [(t, d, sk, rng.integers(1, 9, sessions).astype(np.uint8))], [0], [1000], "most")
        b.config.update(flags=tg.F_BATCH_MODE | (tg.F_SCALE_OUT if grow else 0), boot_delay_ms=20_000)
        if sessions > most:
            with pytest.raises(rp.NbosError) as e:
                gpu_run(rp, b)
            assert e.value.code == rp.E_LIMIT
        else:
            st, logs = gpu_run(rp, b, log=True)
            assert_same(rp, oracle, b, st, logs)


def cell_timers_at_once(b, log):
    """The most cells that timers of one instant have started or given up, by the decision log (a closed loop's cells all
    come by timer, an open loop's if they do not arrive at that instant). All of these timers were pending before it."""
    time, sess, what = log >> np.uint64(32), (log >> np.uint64(16)) & np.uint64(0xFFFF), (log >> np.uint64(12)) & np.uint64(15)
    by_timer = np.isin(what, [4, 5, 6, 7, 12])
    if not b.config["flags"] & tg.F_CLOSED_LOOP:
        cell = b.ev_sk >> 24 == tg.EV_CELL
        arrivals = b.ev_time[cell].astype(np.uint64) << np.uint64(16) | b.ev_sk[cell].astype(np.uint64) & np.uint64(0xFFFF)
        by_timer &= ~np.isin(time << np.uint64(16) | sess, arrivals)
    return int(np.unique(time[by_timer], return_counts=True)[1].max(initial=0))


@pytest.mark.parametrize("closed", [False, True], ids=["open", "closed"])
@pytest.mark.parametrize("hosts,sessions,step_ms", [(256, 1024, 1), (256, 1025, 1), (256, 1028, 1000), (257, 2049, 60_000),
                                                    (320, 4099, 1), (300, 3000, 600_000), (65, 1300, 1000)])
def test_refill_of_the_sorted_timers(rp, oracle, hosts, sessions, step_ms, closed):  # noqa: F811
    # many more timers than the 64 sorted ones, alone in their millisecond or hundreds at one instant; the helper
    # waves take part in the scan from 256 hosts and more than 1,024 sessions on
    b = on_a_grid(5, hosts, sessions, step_ms, tg.F_MIGRATE | (tg.F_CLOSED_LOOP if closed else 0), [1500, 4000])
    st, logs = gpu_run(rp, b, log=True)
    assert_same(rp, oracle, b, st, logs)
    assert closed or st["cells_queued"].max() > 64
    # on the coarse grids more than 64 timers of one instant wait outside the 64 sorted ones
    assert step_ms < 60_000 or max(cell_timers_at_once(b, log) for log in logs) > 128


@pytest.mark.parametrize("hosts,sessions,step_ms,flags", [(64, 1200, 10_000, 0), (64, 1200, 10_000, tg.F_SCALE_IN), (8, 500, 10_000, tg.F_MIGRATE),
                                                          (33, 700, 10_000, tg.F_MIGRATE), (64, 1200, 10_000, tg.F_MIGRATE),
                                                          (33, 700, 600_000, tg.F_MIGRATE), (8, 300, 10_000, tg.F_MIGRATE | tg.F_SCALE_OUT),
                                                          (64, 1200, 10_000, tg.F_MIGRATE | tg.F_SCALE_OUT)])
def test_refill_of_one_instant_in_the_register_kernel(rp, oracle, hosts, sessions, step_ms, flags):  # noqa: F811
    # retries fall on the grid of the trace (10 s apart): more than 64 timers of one instant wait in the session records,
    # the earliest is taken alone, and timers pushed for that instant before it fires (an END deferred to a cell's finish,
    # the retry of a session with a lower number) come before it or wait behind it. Each case on the 10 s grid was
    # answered in another order while all such timers were left to wait.
    b = on_a_grid(5, hosts, sessions, step_ms, flags, [4000, 20_000, 100_000])
    if flags & tg.F_SCALE_OUT:
        b.config["hosts_max"] = min(64, hosts + 6)
    st, logs = gpu_run(rp, b, log=True)
    assert_same(rp, oracle, b, st, logs)
    assert st["cells_queued"].max() > 64
    assert step_ms < 60_000 or max(cell_timers_at_once(b, log) for log in logs) > 128


@pytest.mark.parametrize("flags", [0, tg.F_MIGRATE, tg.F_MIGRATE | tg.F_SCALE_OUT, tg.F_MIGRATE | tg.F_STICKY_EXECUTOR],
                         ids=["plain", "migrate", "grow", "sticky"])
@pytest.mark.parametrize("hosts,sessions,cells,longest", [(3, 1, 1, False), (8, 3, 60, False), (9, 7, 57, True), (24, 20, 45, False),
                                                          (33, 32, 97, True), (64, 64, 65, True), (64, 60, 1000, False)])
def test_starts_at_once_in_the_register_kernel(rp, oracle, hosts, sessions, cells, longest, flags):  # noqa: F811
    # sums over the cells that start at once are made per tile of 64 events: first and last tiles of any fill, the
    # longest cells on all GPUs of a host (the largest GPU time a lane can bring)
    tr = tg.make_trace(11, sessions, cells, ramp_ms=60_000,
                       gpus=(lambda r, n: np.full(n, 8, np.uint8)) if longest else tg.gpus_uniform,
                       gap=lambda r, s: tg.exp_ms(r, 100.0, s),
                       dur=lambda r, s: np.full(s, tg.MAX_DUR_MS, np.int64) if longest else tg.exp_ms(r, 20.0, s))
    b = tg.pack(tg.base_config(hosts_initial=hosts, hosts_max=min(hosts + 5, 64), flags=flags), [tr], [0, 0], [2000, 5000], "at_once")
    st, logs = gpu_run(rp, b, log=True)
    assert_same(rp, oracle, b, st, logs)
    assert st["cells_immediate"].max() > 0


@pytest.mark.parametrize("flags", [0, tg.F_SCALE_IN, tg.F_CLOSED_LOOP], ids=["plain", "shrink", "closed"])
@pytest.mark.parametrize("hosts,G", [(3, 8), (8, 3), (9, 8), (33, 2), (64, 8)])
def test_retries_skipped_where_cells_do_not_migrate(rp, oracle, hosts, G, flags):  # noqa: F811
    # without migration a queued cell waits for its session's own three hosts: retries before they can have the GPUs
    # idle are skipped, and the ones that are left start, fail again or give the cell up at the same times
    tr = crowded(21, hosts, G, 4, 5, gap_s=60.0, dur_s=90.0, with_end=True)
    b = tg.pack(tg.base_config(hosts_initial=hosts, hosts_max=hosts, min_hosts=max(3, hosts // 2), gpus_per_host=G, flags=flags),
                [tr], [0, 0], [1500, 6000], "own")
    st, logs = gpu_run(rp, b, log=True)
    assert_same(rp, oracle, b, st, logs)
    assert st["cells_queued"].max() > 0 and st["cells_started"].max() > st["cells_immediate"].max()
