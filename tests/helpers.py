"""Shared test plumbing: golden loading and trace assembly (no policy arithmetic)."""
import json
import os

import numpy as np

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")


def load_golden(name):
    with open(os.path.join(GOLDEN, name)) as f:
        return json.load(f)


def events_to_arrays(events):
    """[[time, kind, session, dur], ...] -> (ev_time, ev_dur, ev_sk) int32 arrays."""
    ev = np.asarray(events, dtype=np.int64).reshape(-1, 4)
    return (ev[:, 0].astype(np.int32), ev[:, 3].astype(np.int32),
            (ev[:, 2] | (ev[:, 1] << 24)).astype(np.int32))


def code_of(time, outcome, session, slot, host):
    return host | (slot << 10) | (outcome << 12) | (session << 16) | (time << 32)


def digest_of(codes):
    d = 0xCBF29CE484222325
    for c in codes:
        d = (d * 0x100000001B3 + int(c)) & 0xFFFFFFFFFFFFFFFF
    return d


def late_in_a_closed_loop(how, left, first_dur=1):
    """A closed loop near the end of the int32 time range: (config, events, GPUs) with two sessions (0 and 4) whose
    cells come days late, each after four day-long ones that follow one another at once, when three other sessions hold
    all GPUs of the hosts of both. Session 0's last cell, of ``first_dur`` ms, is submitted ``left`` ms before the last
    time there is, session 4's 5 s later. ``how``: 'migrate' (to the one idle host), 'grow' (onto a new host) or 'warm'
    (to the idle host, which has one pre-warmed container)."""
    from paper_2503_20591_amd import tracegen as tg
    day, end, now = 86_400_000, 2**31 - 1, 2**31 - 1 - left
    cfg = dict(tg.base_config(hosts_initial=3 if how == "grow" else 4, hosts_max=4,
                              flags=tg.F_CLOSED_LOOP | {"migrate": tg.F_MIGRATE, "grow": tg.F_SCALE_OUT,
                                                        "warm": tg.F_MIGRATE | tg.F_WARM_POOL}[how]),
               migration_delay_ms={"migrate": 600_000, "grow": 1_000, "warm": 2_000}[how], boot_delay_ms=600_000 if how == "grow" else 0,
               retry_interval_ms=1000, max_retries=2, warm_pool_per_host=1, warm_migration_delay_ms=1_000,
               prewarm_delay_ms=600_000 if how == "warm" else 0)
    latest = end - 1 - (day + 2 * 1000 + 600_000 + 2_000)          # a trace's last event
    ev = [[0, 0, s, 0] for s in range(5)]
    for s, at, dur in ((0, now, first_dur), (4, now + 5_000, 1)):
        ev += [[10 + i, 1, s, day] for i in range(4)]              # at 10 + i days: three days late at the end
        ev += [[at - 3 * day + 3, 1, s, dur]]
    for s in (1, 2, 3):                                            # a day, and on to the last second but one
        ev += [[latest - 10, 1, s, day], [latest - 10, 1, s, end - 2 - (latest - 10 + day)]]
    return cfg, sorted(ev), [8] * 5


def late_batch_host(up, lead=0):
    """A Batch queue whose last request for a host, made when none is being provisioned, asks for one that comes up at ``up``:
    (config, events, GPUs). All jobs need a whole host, hosts take 12 h to come up. The jobs arrive 48 h before ``up``; two days
    of waiting bring the fourth request to 12 h before ``up``, and the job that makes it runs a minute later on a host that
    is over by then. ``lead``: short jobs of another session at the trace's start."""
    from paper_2503_20591_amd import tracegen as tg
    hour, minute = 3_600_000, 60_000
    cfg = dict(tg.base_config(hosts_initial=1, hosts_max=5, flags=tg.F_BATCH_MODE | tg.F_SCALE_OUT), boot_delay_ms=12 * hour,
               batch_start_delay_ms=0)
    # hosts asked for at 0, 12, 24, 36 h; jobs start at 0 (host 0), 12 (1), 24 (0 again, and 2), 36 (1 again, and 3), 36 h 1 min
    durations = [24 * hour, 24 * hour, 23 * hour, 12 * hour + minute, 11 * hour, 11 * hour, 1]
    arrive = up - 48 * hour
    ev = [[2 * i, 1, 7, 1] for i in range(lead)]
    ev += [[arrive, 1, s, d] for s, d in enumerate(durations)]
    return cfg, ev, [8] * 8
