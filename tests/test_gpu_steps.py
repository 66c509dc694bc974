"""Block-local step loops (partition policy with every launch fused, or no
schedule asked for):
one iteration against the per-action kernels, bit for bit, and whole showers
against the oracle where the loops can go wrong -- slot counts that end
inside a chunk or a block, more tracks than slots (secondaries wait on the
blocks' stacks and in the initializer buffer), tables that do not fit beside
the lists -- and which schedules run as such loops."""
import numpy as np
import pytest

import workloads
from tests.gpu_helpers import assert_events_match, random_states, run_oracle, session_for, to_lib_tracks

pytestmark = pytest.mark.gpu

FIELDS = {"none": (0.0, 0.0, 0.0), "x": (1.0, 0.0, 0.0), "oblique": (0.3, -0.7, 1.1)}
LOCAL = dict(sort_policy="partition", init_partition=True, streams=1)
WORK = ("pre_step", "along_neutral", "along_charged", "along_field", "field_paused", "field_substeps", "compton",
        "photoelectric", "pair", "moller", "bhabha", "bremsstrahlung", "annihilation")


def _one_iteration(w, states, slots, precision, msc, cap, local):
    s = session_for(w, n_slots=slots, precision=precision, max_events=4, msc=msc, max_substeps=cap,
                    n_initializers=4 * len(states), **LOCAL)
    rows = np.array([s.register_event(10 + i) for i in range(4)], dtype=np.uint32)
    s.inject(to_lib_tracks(states, rows[np.arange(len(states)) % 4]))
    if local:
        s.set_tuning(fuse_interactions=True)
        s.step(1)
    else:
        s.iterate(1, no_init=True)
    t = s.read_tracks(slots)
    t = np.concatenate([t[t["type"] >= 0], s.read_secondaries()])
    work = s.counters()["work"]
    led = s.read_all()[1]
    s.close()
    return t[np.argsort(t["key"], kind="stable")], [work[k] for k in WORK], led


@pytest.mark.parametrize("precision", ["f64", "mixed"])
@pytest.mark.parametrize("field,msc,cap,n,slots", [
    ("x", False, 10, 20000, 20000),        # no vacant slot: every secondary waits
    ("x", True, 1, 20000, 70001),          # every step of more than one evaluation pauses
    ("oblique", False, 0, 5000, 6143),     # no cap; the last block's slots end inside a chunk
    ("none", True, 10, 20000, 1 << 17),    # straight charged steps
    ("none", False, 10, 1, 1),             # one slot
    ("x", False, 10, 65, 127),
])
def test_one_iteration_equals_the_action_kernels(precision, field, msc, cap, n, slots):
    w = workloads.electron_showers_1gev_field(1)
    w.stack = workloads.sampling_stack(50, 40.0, FIELDS[field])
    states = random_states(w, n, np.random.default_rng(n + slots), f32=precision == "mixed")
    ref, work_ref, led_ref = _one_iteration(w, states, slots, precision, msc, cap, False)
    t, work, led = _one_iteration(w, states, slots, precision, msc, cap, True)
    assert work == work_ref
    assert np.array_equal(led, led_ref) or all(
        np.array_equal(led[f], led_ref[f]) for f in led.dtype.names if f != "escaped")
    assert len(t) == len(ref)
    for f in t.dtype.names:
        if f != "row":
            assert np.ascontiguousarray(t[f]).tobytes() == np.ascontiguousarray(ref[f]).tobytes(), f


@pytest.mark.parametrize("slots,drain", [(1, 0), (64, 0), (257, 0xFFFFFFFF), (1000, 0), (8191, 2048), (300001, 0)])
def test_showers_equal_the_oracle(slots, drain):
    w = workloads.electron_showers_1gev_field(4 if slots > 1 else 1)
    if slots == 1:
        w.primaries["T"] = 20.0
    e_ref, l_ref, steps = run_oracle(w)
    s = session_for(w, n_slots=slots, n_initializers=1 << 18, graph_iterations=8, **LOCAL)
    s.set_tuning(fuse_interactions=True, drain_threshold=drain)
    for _ in range(2):
        c0 = s.counters()["steps"]
        s.push(w.primaries)
        c = s.run(10_000_000)
        assert c["steps"] - c0 == steps and c["alive"] == 0 and c["queued"] == 0
        edep, led = s.tallies_by_event(np.arange(w.n_events))
        assert_events_match(w, edep, led, e_ref, l_ref, (slots, drain))
        s.release(np.arange(w.n_events, dtype=np.uint64))
    s.close()


def test_tables_that_do_not_fit_beside_the_lists():
    """Sixteen materials: 185 kB of tables in FP64.  The step loops run as separate kernels that read them
    through the caches, and the drain is left out."""
    w = workloads.electron_showers_1gev_field(2)
    w.stack.materials = [workloads.LEAD, workloads.LIQUID_ARGON] * 8
    e_ref, l_ref, steps = run_oracle(w)
    s = session_for(w, n_slots=8192, graph_iterations=4, lds_tables=0, **LOCAL)
    s.set_tuning(fuse_interactions=True, drain_threshold=0xFFFFFFFF)
    s.push(w.primaries)
    c = s.run(1_000_000)
    edep, led = s.tallies_by_event(np.arange(w.n_events))
    s.close()
    assert c["steps"] == steps and c["work"]["drain"] == 0 and c["work"]["along_field"] > 0
    assert_events_match(w, edep, led, e_ref, l_ref, "sixteen materials")


def test_overflow_of_the_initializer_buffer_is_reported():
    from paper_2503_17608_amd import emstep
    w = workloads.electron_showers_1gev_field(40)
    s = session_for(w, n_slots=64, n_initializers=8, **LOCAL)
    s.set_tuning(fuse_interactions=True)
    s.push(w.primaries)
    with pytest.raises(emstep.EmsError) as e:
        s.run(1_000_000)
    assert e.value.status == emstep.ERR_CAPACITY
    s.close()


@pytest.mark.parametrize("n_events,max_events,order", [(1, 1, "one"), (7, 40, "reversed"), (3000, 3000, "shuffled"),
                                                       (40, 40, "twice")])
def test_events_are_read_in_the_callers_order(n_events, max_events, order):
    """Deposits and ledgers of listed events (through both halves of the staging buffer for 3000 events of 100
    slabs, 2.5 MB) are the rows of the whole-table read, bit for bit."""
    w = workloads.electron_showers_1gev_field(n_events)
    w.primaries["T"] = 5.0
    w.primaries["event"] += 5
    s = session_for(w, n_slots=4096, max_events=max_events, n_initializers=1 << 16, **LOCAL)
    s.set_tuning(fuse_interactions=True)
    s.push(w.primaries)
    s.run(100_000)
    e_all, l_all, ev_all = s.read_all()
    ids = np.arange(5, 5 + n_events)
    ids = {"one": ids, "reversed": ids[::-1], "shuffled": np.random.default_rng(1).permutation(ids),
           "twice": np.repeat(ids, 2)}[order]
    edep, led = s.tallies_by_event(ids)
    at = {int(x): i for i, x in enumerate(ev_all)}
    rows = np.array([at[int(x)] for x in ids])
    assert edep.tobytes() == e_all[rows].tobytes() and led.tobytes() == l_all[rows].tobytes()
    one_e, one_l = s.read_edep(int(ids[0]))
    assert one_e.tobytes() == edep[0].tobytes() and one_l.tobytes() == led[0].tobytes()
    assert edep.sum() > 0
    for bad in ([4], [5, 5 + n_events], [-1], np.array([-1])):
        with pytest.raises(KeyError):
            s.tallies_by_event(bad)
    s.close()


@pytest.mark.parametrize("tuning,streams,local", [
    (None, 4, True),                       # no schedule asked for: the library's choice
    (dict(), 4, False),                    # any tuning: no policy means masked kernels
    (dict(sort_policy="none", fuse_interactions=True), 1, False),
    (dict(sort_policy="partition"), 4, False),
    (dict(sort_policy="partition", fuse_interactions=True), 4, True),
])
def test_schedules_that_run_as_block_local_loops(tuning, streams, local):
    from paper_2503_17608_amd import emstep
    w = workloads.electron_showers_1gev_field(3)
    e_ref, l_ref, steps = run_oracle(w)
    s = session_for(w, n_slots=5001, n_initializers=1 << 18, sort_policy="none", graph_iterations=0, streams=streams)
    if tuning is not None:
        s.set_tuning(**tuning)
    s.profile(emstep.role_mask("drain"))   # the loops' launches
    s.push(w.primaries)
    c = s.run(10_000_000)
    assert (s.profile_read().get("drain", (0.0, 0))[1] > 0) == local
    assert c["steps"] == steps and c["alive"] == 0 and c["queued"] == 0
    edep, led = s.tallies_by_event(np.arange(3, dtype=np.uint64))
    assert_events_match(w, edep, led, e_ref, l_ref, (tuning, streams))
    s.close()
