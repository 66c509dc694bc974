"""The autotuner's search on made-up run times (no GPU): the block-local step
loops -- partition with both fusions -- are timed whatever the separate
kernels' searches came to."""
import numpy as np
import pytest

from paper_2503_17608_amd import autotune


class Session:
    """Run time by policy for the separate kernels, and another one for partition with everything fused."""

    def __init__(self, policy_s, loops_s):
        self.policy_s, self.loops_s = policy_s, loops_s
        self.t = dict(sort_policy="none", fuse_interactions=False, fuse_along=True, drain_threshold=0)
        self.timed = []

    def set_tuning(self, **kw):
        self.t.update(kw)

    def profile(self, mask):
        pass

    def profile_read(self):
        return {}

    def loops(self):
        return self.t["sort_policy"] == "partition" and self.t["fuse_interactions"] and self.t["fuse_along"]

    def run(self):
        self.timed.append(self.loops())
        drain = 0.9 if self.t["drain_threshold"] == 16384 else 1.0
        if self.loops():
            return self.loops_s * drain
        return self.policy_s[self.t["sort_policy"]] * (0.8 if self.t["fuse_interactions"] else 1.0) * drain


SEPARATE = {"none": 1.0, "partition": 2.0, "radix": 1.5, "queue": 3.0}


@pytest.mark.parametrize("loops_s,policies,want", [
    (0.3, tuple(SEPARATE), "partition"),        # partition alone is the slowest but one
    (0.9, tuple(SEPARATE), "none"),             # slower than the masked kernels, fused and drained
    (0.3, ("none", "radix"), "none"),           # a caller that leaves partition out does not get it
])
def test_loops_are_a_candidate_of_their_own(monkeypatch, loops_s, policies, want):
    monkeypatch.setattr(autotune, "_run", lambda s, sample, events: s.run())
    monkeypatch.setattr(autotune, "phase_table", lambda s, sample, events: ((1, 2), {"choice": {"0": [1, 1]}}))
    s = Session(SEPARATE, loops_s)
    res = autotune.autotune(s, np.zeros(1, dtype=[("event", "<u8")]), policies=policies)
    assert any(s.timed) == ("partition" in policies)
    assert res["sort_policy"] == want == s.t["sort_policy"]
    assert res["fuse_interactions"] and res["drain_threshold"] == 16384 == s.t["drain_threshold"]
    if want == "partition":
        assert s.loops() and res["fuse_along"] and res["phase_table"]["choice"]
