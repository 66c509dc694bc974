"""What callers of the block-local step loops are promised, where the loops
run differently from an iteration's separate kernels: blocks that start while
others of their launch end, limits, counters, tables and buffers of every
size."""
import numpy as np
import pytest
import torch

import workloads
from paper_2503_17608_amd import multistream
from tests.gpu_helpers import (assert_events_match, assert_same_as, random_states, run_oracle, session_for,
                               to_lib_tracks)

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


def _many_materials(n_events, n_materials):
    w = _electrons(n_events, 1000.0)
    w.stack.materials = [workloads.LEAD, workloads.LIQUID_ARGON] * (n_materials // 2)
    i = np.arange(w.stack.n_slabs)
    w.stack.slab_material = ((2 * i + i % 2) % n_materials).astype(np.int32)
    return w


@pytest.mark.parametrize("precision,materials,slots,policy,fused,drain,field", [
    ("f64", 16, 8192, "partition", True, 0xFFFFFFFF, True),
    ("f64", 16, 8192, "partition", False, 2000, True),
    ("f64", 14, 777, "queue", True, 500, True),
    ("f64", 16, 4096, "none", False, 2000, False),
    ("f64", 6, 1 << 23, "partition", True, 0xFFFFFFFF, True),    # the lists of 32768 slots leave less room
    ("mixed", 32, 8192, "radix", True, 2000, True),
])
def test_drain_with_tables_beyond_lds(precision, materials, slots, policy, fused, drain, field):
    """Tables that do not fit into LDS beside a block's lists: the drain reads them through the caches.  The
    results are the oracle's (mixed precision: those of a run without a drain)."""
    from paper_2503_17608_amd import emstep
    w = _many_materials(12, materials)
    if not field:
        w.stack.B = (0.0, 0.0, 0.0)
    s = session_for(w, n_slots=slots, n_initializers=1 << 18, precision=precision, sort_policy=policy,
                    graph_iterations=0, streams=1, lds_tables=0)
    s.set_tuning(fuse_interactions=fused, drain_threshold=drain)
    s.profile(emstep.role_mask("drain"))
    s.push(w.primaries)
    c = s.run()
    assert s.profile_read().get("drain", (0.0, 0))[1] > 0
    edep, led = s.tallies_by_event(np.arange(w.n_events))
    if precision == "f64":
        e_ref, l_ref, steps = run_oracle(w)
        assert_events_match(w, edep, led, e_ref, l_ref, (materials, policy))
    else:
        s.profile(0)
        s.release(np.arange(w.n_events, dtype=np.uint64))
        s.set_tuning(drain_threshold=0)
        s.push(w.primaries)
        steps = s.run()["steps"] - c["steps"]
        assert_same_as(w, edep, led, *s.tallies_by_event(np.arange(w.n_events)), (materials, policy))
    assert c["steps"] == steps and c["alive"] == 0 and c["queued"] == 0
    s.close()


@pytest.mark.parametrize("slots", [1, 63, 65, 16385, 40007, (1 << 23) + 65])
def test_drain_at_ragged_slot_counts(slots):
    """A drain deals the slots out to its blocks 64 at a time: slot counts that end inside a row of blocks, inside
    64 slots, or fill fewer blocks than there are compute units."""
    w = _electrons(3, 1000.0 if slots > 1 else 20.0)
    e_ref, l_ref, steps = run_oracle(w)
    s = session_for(w, n_slots=slots, n_initializers=1 << 18, sort_policy="radix", init_partition=True, streams=1)
    for drain in (0xFFFFFFFF, 1000):
        s.set_tuning(fuse_interactions=True, drain_threshold=drain)
        s.push(w.primaries)
        c0 = s.counters()["steps"]
        c = s.run()
        assert c["steps"] - c0 == steps and c["alive"] == 0 and c["queued"] == 0 and c["work"]["drain"] > 0
        edep, led = s.tallies_by_event(np.arange(w.n_events))
        assert_events_match(w, edep, led, e_ref, l_ref, (slots, drain))
        s.release(np.arange(w.n_events, dtype=np.uint64))
    s.close()


def _iterations_needed(s, w):
    """Iterations of the separate kernels (a profile of one of them keeps the loops away) until `w` has ended."""
    from paper_2503_17608_amd import emstep
    s.profile(emstep.role_mask("bremsstrahlung", "interactions"))
    s.push(w.primaries)
    for n in range(1, 100000):
        c = s.step(1)
        if c["alive"] == 0 and c["queued"] == 0 and c["pending_primaries"] == 0:
            break
    s.profile(0)
    s.profile_read()
    s.release(np.arange(w.n_events, dtype=np.uint64))
    return n


@pytest.mark.parametrize("n,slots,drain_steps,max_substeps", [(1, 1 << 14, 1, 10), (1, 1 << 14, 3, 1), (100, 8192, 50, 10)])
def test_a_round_of_a_drain_is_worth_an_iteration(n, slots, drain_steps, max_substeps):
    """In a round of drain_steps every track makes up to four steps, so a drain from the first iteration on ends
    within 1 / drain_steps as many launches as the separate kernels need iterations."""
    w = _electrons(n, 1000.0)
    s = session_for(w, n_slots=slots, n_initializers=1 << 18, sort_policy="radix", streams=1, max_substeps=max_substeps)
    s.set_tuning(fuse_interactions=True)
    limit = -(-_iterations_needed(s, w) // drain_steps)
    s.set_tuning(drain_threshold=0xFFFFFFFF, drain_steps=drain_steps)
    s.push(w.primaries)
    c = s.run(limit)
    assert c["alive"] == 0 and c["queued"] == 0
    s.close()


@pytest.mark.parametrize("n,slots,tuned", [(1, 1 << 14, True), (1, 1 << 14, False), (20, 64, True), (100, 8192, True)])
def test_a_limit_that_suffices_for_the_separate_kernels_suffices(n, slots, tuned):
    from paper_2503_17608_amd import emstep
    w = _electrons(n, 1000.0)
    e_ref, l_ref, steps = run_oracle(w)
    s = session_for(w, n_slots=slots, n_initializers=1 << 18, **(LOCAL if tuned else {}))
    if tuned:
        s.set_tuning(fuse_interactions=True)
    limit = _iterations_needed(s, w)
    steps0 = s.counters()["steps"]
    s.push(w.primaries)
    with pytest.raises(emstep.EmsError) as e:
        s.run(16)                   # far fewer than the showers are deep
    assert e.value.status == emstep.ERR_STATE
    s.run()
    s.release(np.arange(w.n_events, dtype=np.uint64))
    s.push(w.primaries)
    c = s.run(limit)
    assert c["steps"] - steps0 == 2 * steps and c["alive"] == 0 and c["queued"] == 0
    edep, led = s.tallies_by_event(np.arange(w.n_events))
    s.close()
    assert_events_match(w, edep, led, e_ref, l_ref, (n, slots, tuned))


def test_null_stream_with_graph_batches():
    """Graph batches need a stream of their own; a run that is drained from its first iteration has none."""
    from paper_2503_17608_amd import emstep
    w = _electrons(3, 1000.0)
    e_ref, l_ref, steps = run_oracle(w)
    s = session_for(w, n_slots=4096, graph_iterations=8, stream=torch.cuda.default_stream(), **LOCAL)
    assert s.stream.cuda_stream == 0
    s.set_tuning(fuse_interactions=True)
    s.push(w.primaries)
    with pytest.raises(emstep.EmsError) as e:
        s.run()
    assert e.value.status == emstep.ERR_INVALID_ARG
    s.set_tuning(drain_threshold=0xFFFFFFFF)
    c = s.run()
    assert c["steps"] == steps and c["alive"] == 0
    edep, led = s.tallies_by_event(np.arange(w.n_events))
    s.close()
    assert_events_match(w, edep, led, e_ref, l_ref, "null stream")


@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_live_tracks_are_counted_at_the_start_of_the_last_iteration(precision):
    from paper_2503_17608_amd import emstep
    w = _electrons(6, 500.0)
    seen = []
    for local in (True, False):
        s = session_for(w, n_slots=1 << 16, precision=precision, **LOCAL)
        s.set_tuning(fuse_interactions=True)
        if not local:
            s.profile(emstep.role_mask("interactions"))
        s.push(w.primaries)
        seen.append([s.step(n)["alive"] for n in (1, 1, 1, 5, 8, 1, 33, 2, 64, 16, 16, 1, 1, 40, 100, 1)])
        s.close()
    assert seen[0] == seen[1] and max(seen[0]) > 100 and seen[0][0] == 6 and seen[0][-1] == 0


@pytest.mark.parametrize("slots", [1, 3, 64])
def test_stepping_by_the_counters_ends_with_the_last_track(slots):
    """A caller that steps until nothing is alive, queued or pending has stepped everything, also where tracks
    wait for a slot."""
    w = _electrons(2, 60.0)
    e_ref, l_ref, steps = run_oracle(w)
    for n in (1, 3):
        s = session_for(w, n_slots=slots, n_initializers=1 << 14, streams=1)
        s.push(w.primaries)
        for _ in range(100000):
            c = s.step(n)
            if c["alive"] == 0 and c["queued"] == 0 and c["pending_primaries"] == 0:
                break
        assert c["steps"] == steps
        edep, led = s.tallies_by_event(np.arange(w.n_events))
        s.close()
        assert_events_match(w, edep, led, e_ref, l_ref, (slots, n))


def test_unknown_event_of_a_list_that_is_too_long():
    """An unknown event is refused when it is met, whatever length the list is said to have."""
    from paper_2503_17608_amd import emstep
    w = _electrons(2, 20.0)
    s = session_for(w, n_slots=1024, **LOCAL)
    s.push(w.primaries)
    s.run()
    ids = np.array([0, 77], dtype=np.uint64)
    for n in (2, 1 << 40, (1 << 64) - 1):
        assert emstep._lib.ems_release_events(s._h, emstep._ptr(ids), n) == emstep.ERR_INVALID_ARG
        assert emstep._lib.ems_read_events(s._h, emstep._ptr(ids), n, None, None) == emstep.ERR_INVALID_ARG
    s.release(np.arange(2, dtype=np.uint64))
    s.close()


def test_event_lists_of_every_kind():
    """Ids as an array of any integer type, a column, floats, a list, a generator, a tensor; a negative id names no
    event, also where its 64 bits would; a closed session is the library's error, not a missing event."""
    from paper_2503_17608_amd import emstep
    w = _electrons(3, 20.0)
    w.primaries["event"] = np.array([2 ** 64 - 5, 7, 3], dtype=np.uint64)[w.primaries["event"].astype(int)]
    s = session_for(w, n_slots=1024, **LOCAL)
    s.push(w.primaries)
    s.run()
    e_ref, l_ref = s.tallies_by_event(np.array([7, 3], dtype=np.uint64))
    for ids in (np.array([7, 3], np.int64), np.array([7, 3], np.uint8), np.array([7, 9, 3, 9])[::2],
                np.array([[7], [3]]), np.array([7.0, 3.0]), [7, 3], (x for x in (7, 3)), torch.tensor([7, 3])):
        edep, led = s.tallies_by_event(ids)
        assert edep.tobytes() == e_ref.tobytes() and led.tobytes() == l_ref.tobytes()
    s.tallies_by_event([2 ** 64 - 5])
    for bad in (np.array([7, -5]), [-5], np.array([4], np.uint64), [2 ** 64]):
        with pytest.raises(KeyError):
            s.tallies_by_event(bad)
    for bad in (np.array(7), np.array([[7, 3]])):
        with pytest.raises(TypeError):
            s.tallies_by_event(bad)
    s.close()
    with pytest.raises(emstep.EmsError):
        s.tallies_by_event([7])


@pytest.mark.parametrize("n,energy,slots,tuning", [
    (20, 1000.0, 1 << 14, dict(sort_policy="partition", fuse_interactions=True)),
    (200, 1000.0, 1024, dict(sort_policy="partition", fuse_interactions=True)),
    (200, 1000.0, 1 << 14, None),
    (8, 100000.0, 4096, None),
    (1, 100000.0, 4096, dict(sort_policy="radix", fuse_interactions=True, drain_threshold=0xFFFFFFFF)),
    (8, 100000.0, 4096, dict(sort_policy="radix", fuse_interactions=True, drain_threshold=0xFFFFFFFF)),
])
def test_a_buffer_that_suffices_for_the_separate_kernels_suffices(n, energy, slots, tuning):
    """The initializer buffer as large as the most secondaries that wait while separate kernels run (a drain: a
    tenth of it, which its own stacks make up for)."""
    from paper_2503_17608_amd import emstep
    w = _electrons(n, energy)
    streams = 1 if tuning else 4
    s = session_for(w, n_slots=slots, streams=streams, init_partition=tuning is not None)
    s.set_tuning(**{k: v for k, v in (tuning or {}).items() if k != "drain_threshold"})
    s.profile(emstep.role_mask("bremsstrahlung", "interactions"))
    s.push(w.primaries)
    most = 0
    while True:
        c = s.step(1)
        most = max(most, c["queued"])
        if c["alive"] == 0 and c["queued"] == 0 and c["pending_primaries"] == 0:
            break
    e_ref, l_ref = s.tallies_by_event(np.arange(w.n_events))
    s.close()
    s = session_for(w, n_slots=slots, streams=streams, init_partition=tuning is not None,
                    n_initializers=max(1, most // 10 if tuning and "drain_threshold" in tuning else most))
    if tuning:
        s.set_tuning(**tuning)
    s.push(w.primaries)
    assert s.run()["steps"] == c["steps"]
    assert_same_as(w, *s.tallies_by_event(np.arange(w.n_events)), e_ref, l_ref, (n, energy, slots))
    s.close()


def test_a_cleared_tuning_leaves_the_schedule_to_the_library():
    from paper_2503_17608_amd import emstep
    w = _electrons(2, 200.0)
    s = session_for(w, n_slots=4096)
    new = s.tuning()

    def loops():
        s.profile(emstep.role_mask("drain"))
        s.push(w.primaries)
        s.run()
        n = s.profile_read().get("drain", (0.0, 0))[1]
        s.profile(0)
        s.release(np.arange(2, dtype=np.uint64))
        return n > 0

    assert loops()
    s.set_tuning(block={"compton": 128}, tail_threshold=5, phase_sort=(0, 1), fuse_along=False)
    assert not loops()
    s.clear_tuning()
    assert s.tuning() == new and loops()
    s.close()


@pytest.mark.parametrize("n_slabs,n_events", [(1, 3), (127, 1), (129, 5), (2000, 1), (65534, 5)])
def test_events_of_wide_stacks_are_read_whole(n_slabs, n_events):
    """Rows of one to 65534 slabs (several blocks per row; four rows fill half of the staging buffer)."""
    from paper_2503_17608_amd import emstep
    s = emstep.Session(4096, max_events=n_events, max_slabs=n_slabs, max_materials=1, streams=1)
    s.load(np.arange(n_slabs + 1) * (70.0 / n_slabs), np.zeros(n_slabs, np.int32), 20.0, (1.0, 0.0, 0.0),
           [workloads.LEAD], 0.1)
    p = np.zeros(8 * n_events, dtype=emstep.PRIMARY_DTYPE)
    p["event"], p["key"], p["type"], p["T"] = np.arange(len(p)) % n_events, np.arange(len(p)), 1, 5.0
    p["u"][:, 2] = 1.0
    p["slab"] = np.linspace(0, n_slabs - 1, len(p)).astype(np.int32)
    p["r"][:, 2] = (p["slab"] + 0.5) * (70.0 / n_slabs)
    s.push(p)
    s.run()
    e_all, l_all, ev_all = s.read_all()
    ids = np.arange(n_events)[::-1]
    rows = [list(ev_all).index(i) for i in ids]
    edep, led = s.tallies_by_event(ids)
    assert edep.tobytes() == e_all[rows].tobytes() and led.tobytes() == l_all[rows].tobytes()
    assert np.all(edep.max(1) > 0) and (edep[:, -1] > 0).any() and (edep[:, 0] > 0).any()
    one_e, one_l = s.read_edep(0)
    assert one_e.tobytes() == edep[-1].tobytes() and one_l.tobytes() == led[-1].tobytes()
    s.close()


def _after(w, states, slots, precision, max_events, iterations, local):
    """Tracks by key, ledgers and deposits after `iterations` of the loops in one launch, or of separate kernels."""
    s = session_for(w, n_slots=slots, precision=precision, max_events=max_events, n_initializers=4 * len(states),
                    **LOCAL)
    rows = np.array([s.register_event(10 + i) for i in range(4)], dtype=np.uint32)
    t = to_lib_tracks(states, rows[np.arange(len(states)) % 4])
    t["type"][np.arange(len(t)) % 60 != 0] = -1      # 5 of a block's 274 slots: none of its tracks has to wait
    s.inject(t)
    s.set_tuning(fuse_interactions=True)
    if local:
        s.step(iterations)
    else:
        s.iterate(iterations)
    t = s.read_tracks(slots)
    t = np.concatenate([t[t["type"] >= 0], s.read_secondaries()])
    edep, led = s.tallies_by_event(np.arange(10, 14))
    s.close()
    return t[np.argsort(t["key"], kind="stable")], edep, led


@pytest.mark.parametrize("precision", ["f64", "mixed"])
@pytest.mark.parametrize("max_events,iterations", [(4, 1), (4, 7), (2000, 7)])    # 4 rows fit a block's LDS, 2000 do not
def test_iterations_in_one_launch_equal_the_separate_kernels(precision, max_events, iterations):
    """Seven iterations in step: tracks bit for bit, whole numbers equal; deposits and escapes are sums of at most
    10^5 terms in another order, each rounded to 1.1e-16."""
    w = _electrons(1, 1000.0)
    states = random_states(w, 60000, np.random.default_rng(iterations), f32=precision == "mixed")
    ref, e_ref, l_ref = _after(w, states, 70001, precision, max_events, iterations, False)
    t, edep, led = _after(w, states, 70001, precision, max_events, iterations, True)
    assert len(t) == len(ref)
    for f in t.dtype.names:
        if f != "row":
            assert np.ascontiguousarray(t[f]).tobytes() == np.ascontiguousarray(ref[f]).tobytes(), f
    for f in led.dtype.names:
        if f != "escaped":
            assert np.array_equal(led[f], l_ref[f]), f
    assert np.all(np.abs(edep - e_ref) <= 1.2e-11 * e_ref) and edep.sum() > 0
    assert np.all(np.abs(led["escaped"] - l_ref["escaped"]) <= 1.2e-11 * l_ref["escaped"])


@pytest.mark.parametrize("policy", ["partition", "radix"])
def test_phase_tables_with_separate_kernels(policy):
    """Masked and sorted iterations in one run (sort points off in some occupancy buckets), interactions apart so
    that they run as separate kernels."""
    w = _electrons(20, 1000.0)
    e_ref, l_ref, steps = run_oracle(w)
    s = session_for(w, n_slots=1 << 14, sort_policy=policy, graph_iterations=4, streams=1)
    for masks in ((0, 0xFFFFFFFF), (0xFFFFFFFF, 0), (0x0000003F, 0xFFFFFFC0), (0x00000FC0, 0x000001FF)):
        s.set_tuning(phase_sort=masks, fuse_interactions=False)
        s.push(w.primaries)
        s.run()
        edep, led = s.tallies_by_event(np.arange(w.n_events))
        s.release(np.arange(w.n_events, dtype=np.uint64))
        assert_events_match(w, edep, led, e_ref, l_ref, (policy, masks))
    s.close()
