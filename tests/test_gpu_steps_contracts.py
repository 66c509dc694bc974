"""What callers of the block-local step loops are promised, where the loops
run differently from an iteration's separate kernels: blocks that start while
others of their launch end, limits, counters, tables and buffers of every
size."""
import numpy as np
import pytest
import torch

import workloads
from paper_2503_17608_amd import multistream
from tests.gpu_helpers import assert_events_match, run_oracle, session_for

pytestmark = pytest.mark.gpu

LOCAL = dict(sort_policy="partition", init_partition=True, streams=1)


def _electrons(n, energy):
    w = workloads.electron_showers_1gev_field(n)
    w.primaries["T"] = energy
    return w


@pytest.mark.parametrize("slots", [(1 << 23) + 1, (1 << 24) + 4567])
def test_more_blocks_than_compute_units(slots):
    """Above 2^23 slots a launch has more blocks than compute units, so blocks start while others end; an event
    that fills one block beyond its share of the live tracks makes its secondaries wait."""
    w = _electrons(5, 20000.0)
    e_ref, l_ref, steps = run_oracle(w)
    s = session_for(w, n_slots=slots, n_initializers=1 << 20, graph_iterations=8, **LOCAL)
    s.set_tuning(fuse_interactions=True)
    s.push(w.primaries)
    c = s.run()
    assert c["steps"] == steps and c["alive"] == 0 and c["queued"] == 0
    edep, led = s.tallies_by_event(np.arange(w.n_events))
    s.close()
    assert_events_match(w, edep, led, e_ref, l_ref, slots)


def test_sessions_that_share_the_gpu():
    """Three sessions whose launches each have a block per compute unit: a block of one waits for the end of
    another's, so blocks of a launch start while others end."""
    w = _electrons(48, 1000.0)
    e_ref, l_ref, steps = run_oracle(w)
    sessions = []
    for slots in (1 << 14, 1 << 15, 20001):
        s = session_for(w, n_slots=slots, max_events=4, stream=torch.cuda.Stream(), graph_iterations=8, **LOCAL)
        s.set_tuning(fuse_interactions=True)
        sessions.append(s)
    edep, led, n, _ = multistream.run_event_parallel(sessions, w.primaries, chunk_events=4)
    for s in sessions:
        s.close()
    assert n == steps
    ids = range(w.n_events)
    assert_events_match(w, np.stack([edep[i] for i in ids]), np.array([led[i] for i in ids], dtype=l_ref.dtype),
                        e_ref, l_ref, "three sessions")
