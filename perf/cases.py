"""The work whose time on one GPU this repository is judged by.

A user of the library opens a session (track slots, buffers and tables
resident on the GPU), pushes the primaries of some events, runs them to the
end and reads every event's deposits and ledger; a server does the same with
events that keep arriving; and the reordering of slots by a small key can be
called on its own.  Each case below is one such call, whole: primaries start
on the host, results end on the host.

`listed` names the cases, `draw` gives further ones of the same ranges,
`prepare` holds what a program has in hand before the call, `run` is one call
and returns all its results, `work` is what a call cannot do without, and
`exact` is its result computed without this repository's code where that
exists.

Every random number of a transport is keyed by its track, so a case's results
depend on its inputs alone, not on slots, policies, batching or timing: whole
numbers repeat exactly, and deposits to the rounding of the order in which
they are summed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import workloads
from paper_2503_17608_amd import emstep

# The settings of the repository's benchmark: slots partitioned by action before
# the interactions, initializers filled from both ends, one launch for the
# interactions and one for the along-steps, captured graphs, one stream, the
# last tracks drained.
TUNED = dict(policy="partition", partition=True, graph=8, streams=1, fuse=True, drain=-1, det=False, msc=False)
# A session opened with nothing but its size.
PLAIN = dict(policy="none", partition=False, graph=0, streams=4, fuse=False, drain=0, det=False, msc=False)


def _shower(name, events, per, species, e, slots, *, layers=50, field=1.0, cut=0.1, cone=0.0, precision="f64",
            **settings):
    return dict(name=name, kind="shower", events=events, per_lo=per[0], per_hi=per[1], species=species, e_lo=e[0],
                e_hi=e[1], slots=slots, layers=layers, field=field, cut=cut, cone=cone, precision=precision,
                **{**TUNED, **settings})


def listed():
    gev = (1000.0, 1000.0)
    return [
        # one electron of 1 GeV on its own: the latency of the smallest request
        _shower("one_electron_1gev", 1, (1, 1), 1, gev, 1 << 14),
        # the small no-field workload: 1000 electrons of 10 MeV, 20 layers, 1 MeV cut, in few slots
        _shower("electrons_10mev_1000", 1000, (1, 1), 1, (10.0, 10.0), 4096, layers=20, field=0.0, cut=1.0, graph=4),
        # a production batch of odd sizes: 777 electrons of 1 GeV in a slot array that divides by nothing
        _shower("electrons_1gev_777_ragged", 777, (1, 1), 1, gev, 100003),
        # the benchmark's batch: 10^4 electrons of 1 GeV in a 1 T field, FP64
        _shower("electrons_1gev_10000", 10000, (1, 1), 1, gev, 1 << 20),
        # mixed species over two decades of energy in a cone, mixed precision
        _shower("cone_mixed_5000_f32", 5000, (1, 1), 3, (100.0, 10000.0), 1 << 20, cone=5.0, precision="mixed"),
        # events of the size of a collider's: 1300 electrons of 10 GeV each, the largest batch
        _shower("collider_16_events", 16, (1300, 1300), 1, (10000.0, 10000.0), 1 << 21),
        # events of very different sizes up to 100 GeV, in a slot array larger than the caches
        _shower("batched_16_events", 16, (1, 500), 3, (10.0, 100000.0), 1 << 22),
        # a test beam without field and with multiple scattering: charged tracks step straight
        _shower("msc_no_field_5001", 5001, (1, 1), 3, (10.0, 500.0), 1 << 18, layers=20, field=0.0, msc=True),
        # a session as the library opens it when only its size is given: masked kernels on four streams
        _shower("library_defaults_500", 500, (1, 1), 1, gev, 1 << 17, **PLAIN),
        # reproducible runs: secondaries appended in a fixed order
        _shower("deterministic_300", 300, (1, 1), 1, gev, 1 << 16, det=True, drain=0),
        # a server: events arrive four at a time while earlier ones are stepping, mixed precision
        dict(name="serving_48_events", kind="serve", events=48, per_lo=1, per_hi=200, e_lo=10.0, e_hi=10000.0,
             slots=1 << 20, wave=4, iterations=8, precision="mixed", cut=0.1),
        # the reordering on its own: a permutation of slots by a small key, keys and result on the GPU
        dict(name="sort_keys_1000003", kind="sort", n=1000003, policy="partition"),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choices(("shower", "serve", "sort"), (8, 1, 1))[0]
    if kind == "sort":
        # up to the 2^23 keys that the entry point takes
        return dict(kind="sort", n=int(_log_uniform(rng, 1, 1 << 23)), policy=rng.choice(("partition", "radix")))
    if kind == "serve":
        return dict(kind="serve", events=rng.randint(4, 60), per_lo=1, per_hi=rng.randint(2, 200), e_lo=10.0,
                    e_hi=_log_uniform(rng, 100.0, 10000.0), slots=int(_log_uniform(rng, 1 << 16, 1 << 21)),
                    wave=rng.randint(1, 8), iterations=rng.choice((4, 8, 16)),
                    precision=rng.choice(("f64", "mixed")), cut=0.1)
    # the energy of the whole batch, then slots to suit it (a batch of e MeV
    # takes about 9 e track-steps, and few slots step fewer at a time), then
    # how it is divided over events, primaries and energies
    total = _log_uniform(rng, 100.0, 5.0e7)
    slots = int(_log_uniform(rng, max(1024.0, total / 100.0), max(65536.0, 1.2 * total / 100.0, 1 << 21)))
    if rng.random() < 0.4:
        slots = max(1024, 1 << (slots.bit_length() - 1))
    energy = min(max(_log_uniform(rng, 10.0, 1.0e5), total / 2.0e4), total)
    primaries = max(1, int(total / energy))
    events = min(primaries, int(_log_uniform(rng, 1, 10000)))
    per = max(1, primaries // events)
    spread = rng.random() < 0.5
    settings = rng.choices((TUNED, PLAIN, {**TUNED, "det": True, "drain": 0}, {**TUNED, "policy": "radix"}),
                           (12, 1, 1, 1))[0]
    field = rng.choice((0.0, 1.0, 1.0, 2.0))
    return dict(kind="shower", events=events, per_lo=1 if spread else per, per_hi=per, species=rng.choice((0, 1, 1, 2, 3)),
                e_lo=max(10.0, energy / 10.0) if spread else energy, e_hi=energy, slots=slots,
                layers=rng.choice((20, 50, 50)), field=field, cut=rng.choice((0.1, 0.1, 1.0)),
                cone=rng.choice((0.0, 5.0)), precision=rng.choice(("f64", "f64", "mixed")),
                **{**settings, "msc": rng.random() < 0.2})


def _primaries(case, seed):
    """The primaries of a case in event order: on the front face's centre, in a cone about +z."""
    rng = np.random.default_rng(seed)
    counts = rng.integers(case["per_lo"], case["per_hi"] + 1, case["events"])
    n = int(counts.sum())
    p = np.zeros(n, dtype=emstep.PRIMARY_DTYPE)
    p["event"] = np.repeat(np.arange(case["events"], dtype=np.uint64), counts)
    p["key"] = rng.integers(0, 1 << 63, n, dtype=np.uint64)
    species = case.get("species", 3)
    p["type"] = rng.integers(0, 3, n) if species == 3 else species
    p["T"] = case["e_lo"] * (case["e_hi"] / case["e_lo"]) ** rng.random(n)
    cos = 1.0 - rng.random(n) * (1.0 - math.cos(math.radians(case.get("cone", 0.0))))
    phi, sin = 2.0 * math.pi * rng.random(n), np.sqrt(np.maximum(0.0, 1.0 - cos * cos))
    p["u"] = np.stack([sin * np.cos(phi), sin * np.sin(phi), cos], 1)
    return p


def _session(case, seed, energy, n_primaries):
    """A session with the case's stack loaded.  At the widest point of a shower about a hundred tracks
    per GeV are in flight; those beyond the slots wait in the initializer buffer."""
    layers = case.get("layers", 50)
    stack = workloads.sampling_stack(layers, 40.0 if layers == 50 else 10.0, (case.get("field", 1.0), 0.0, 0.0))
    tuned = case.get("policy", "partition") != "none"
    s = emstep.Session(case["slots"], precision=case["precision"],
                       n_initializers=int(max(16 * case["slots"], 0.2 * energy + (1 << 16))),
                       n_primaries=max(n_primaries, 1 << 16), max_events=case["events"], max_slabs=stack.n_slabs,
                       max_materials=len(stack.materials), sort_policy=case.get("policy", "partition"),
                       init_partition=case.get("partition", True), seed=seed & 0xFFFFFFFF,
                       graph_iterations=case.get("graph", 8), streams=case.get("streams", 1),
                       msc=case.get("msc", False), deterministic=case.get("det", False))
    s.load(stack.z_planes, stack.slab_material, stack.half_width, stack.B, stack.materials, case["cut"])
    if tuned:
        # the benchmark's choices: no reordering before the along-steps, and
        # the drain below 65536 tracks at 2^20 slots, in proportion below
        drain = case.get("drain", -1)
        if drain < 0:
            drain = max(256, min(65536, 65536 * case["slots"] // (1 << 20)))
        s.set_tuning(fuse_interactions=case.get("fuse", True), phase_sort=(0, 0xFFFFFFFF),
                     drain_threshold=drain if case["kind"] == "shower" else 0)
    return s


def _keys(case, seed):
    """Sort keys on the GPU: action codes (partition), or action, type and material (radix)."""
    bins = 16 if case["policy"] == "partition" else 128
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(0, bins, (case["n"],), dtype=torch.uint8, device="cuda", generator=gen)


def prepare(case, seed):
    if case["kind"] == "sort":
        s = emstep.Session(1024, n_initializers=1024, n_primaries=1024, max_events=1, streams=1)
        return dict(case=case, session=s, keys=_keys(case, seed),
                    perm=torch.empty(case["n"], dtype=torch.int32, device="cuda"))
    p = _primaries(case, seed)
    s = _session(case, seed, float(p["T"].sum()), len(p))
    state = dict(case=case, session=s, events=np.arange(case["events"], dtype=np.uint64), primaries=p)
    if case["kind"] == "serve":
        edge = np.flatnonzero(np.diff(p["event"])) + 1
        state["requests"] = np.split(p, edge)
    return state


def _results(edep, ledger):
    return {"edep": edep, **{f: np.ascontiguousarray(ledger[f]) for f in ledger.dtype.names}}


def _serve(state):
    case, s = state["case"], state["session"]
    edep, ledger = np.zeros((case["events"], s.n_slabs)), np.zeros(case["events"], dtype=emstep.LEDGER_DTYPE)
    waiting, in_flight = 0, 0
    while waiting < case["events"] or in_flight:
        for _ in range(case["wave"]):
            if waiting < case["events"]:
                s.push(state["requests"][waiting])
                waiting += 1
                in_flight += 1
        s.launch(case["iterations"])
        for ev in s.poll_completed():
            edep[int(ev)], ledger[int(ev)] = s.read_edep(int(ev))
            s.release(int(ev))
            in_flight -= 1
    return _results(edep, ledger)


def run(state):
    case, s = state["case"], state["session"]
    if case["kind"] == "sort":
        s.sort_device(state["keys"], state["perm"], case["policy"])
        return state["perm"]
    if case["kind"] == "serve":
        return _serve(state)
    s.push(state["primaries"])
    s.run(10_000_000)
    edep, ledger = s.tallies_by_event(state["events"])
    s.release(state["events"])
    return _results(edep, ledger)


def work(case):
    """A transport reads its primaries and writes its tallies; between them every track-step is arithmetic, about
    a thousand operations in 64 bits: ten Philox rounds, a logarithm and the cross sections of the step limit, a
    fourth-order step with its distances to six faces, the inverse range and the choice of the process."""
    if case["kind"] == "sort":
        return {"bytes": 5.0 * case["n"], "flops": 0.0}
    lo, hi = case["e_lo"], case["e_hi"]
    mean = lo if hi == lo else (hi - lo) / math.log(hi / lo)
    primaries = 0.5 * (case["per_lo"] + case["per_hi"]) * case["events"]
    # track-steps per MeV, from the oracle: 8.8 above a cut of 0.1 MeV, 2.5 above 1 MeV
    steps = primaries * mean * (8.8 if case["cut"] < 0.5 else 2.5)
    return {"bytes": 80.0 * primaries + case["events"] * (8.0 * 2 * case.get("layers", 50) + 72.0),
            "flops": 1000.0 * steps}


def exact(case, seed):
    """The sort's permutation.  A transport has no value here: it is a chain of random decisions, each drawn at
    the end of the one before, so 64-bit code with other roundings (or the mixed precision's) takes another turn
    somewhere in a large batch, and stepping the histories one by one in Python takes minutes."""
    if case["kind"] != "sort":
        return None
    return np.argsort(_keys(case, seed).cpu().numpy(), kind="stable").astype(np.int32)
