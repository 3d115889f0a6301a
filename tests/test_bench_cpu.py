"""The benchmark's comparison with the oracle, on a stand-in workload (no GPU)."""
import types

import numpy as np
import torch

import bench

B, STEPS, D = 2, 6, 8


class Work:
    """y holds garbage until launch() writes a step's rows, as a torch.empty does."""

    def __init__(self):
        self.cfg = types.SimpleNamespace(B=B, layers=1, steps=STEPS)
        self.want = np.random.default_rng(0).standard_normal((B * STEPS, D)).astype(np.float32)
        self.y = torch.full((B * STEPS, D), 1e3)
        self.launched = set()

    def launch(self, step):
        s = step % STEPS
        self.launched.add(s)
        self.y[s * B:(s + 1) * B] = torch.from_numpy(self.want[s * B:(s + 1) * B])


def test_parity_of_steps_the_timed_run_did_not_reach():
    """Fewer steps than the oracle's sample: every sampled token is compared, on rows that a
    launch has written."""
    work = Work()
    for i in range(2):
        work.launch(i)
    outputs = {t: work.want[t].astype(np.float64) for t in range(B * STEPS - 1)}
    rec = bench.parity_from_oracle(work, outputs, 1e-5)
    assert rec["max_rel_l2"] == 0.0 and rec["tokens_checked"] == len(outputs)
    assert work.launched == set(range(STEPS))


def test_parity_sees_a_wrong_token():
    work = Work()
    outputs = {t: work.want[t].astype(np.float64) for t in range(B * STEPS)}
    outputs[7] = outputs[7] * 1.5
    assert bench.parity_from_oracle(work, outputs, 1e-5)["max_rel_l2"] > 0.3


def test_parity_sees_a_nan():
    work = Work()
    outputs = {t: work.want[t].astype(np.float64) for t in range(B * STEPS)}
    work.want[4, 1] = np.nan                              # what the launch writes
    assert not bench.parity_from_oracle(work, outputs, 1e-5)["max_rel_l2"] <= 1e-5
