"""The batch evaluation's tilings and launch order: runs of very different
scan lengths and populations together (long scans take fewer clients per
workgroup, the longest workgroups are launched first) evolve exactly as each
alone, for small, odd and large common client counts."""
import numpy as np
import pytest

import pmp_inputs as gi

pytestmark = pytest.mark.gpu

RUNS = [(100, 2, 64, 64), (333, 3, 128, 32), (520, 130, 192, 64), (90, 20, 64, 16),
        (1100, 6, 64, 32)]


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available()
    import paper_1610_10061_amd as pm
    pm.lib()
    return pm


@pytest.fixture(scope="module")
def alone(pm):
    out = []
    for k, (n, p, P, NT) in enumerate(RUNS):
        inst = pm.Instance(gi.euclid_instance(n, k), p)
        ga = pm.GA(inst, P, NT, 3, seed=k)
        ga.step(3)
        out.append((ga.best(), ga.state()))
    return out


@pytest.mark.parametrize("clients", [0, 1, 16, 100, 512, 5000])
def test_tilings_do_not_change_the_runs(pm, alone, monkeypatch, clients):
    if clients:
        monkeypatch.setenv("PMP_BATCH_CLIENTS", str(clients))
    insts = [pm.Instance(gi.euclid_instance(n, k), p) for k, (n, p, _, _) in enumerate(RUNS)]
    gas = [pm.GA(inst, P, NT, 3, seed=k)
           for k, (inst, (_, _, P, NT)) in enumerate(zip(insts, RUNS))]
    batch = pm.Batch(gas)
    batch.step(3)
    batch.check()
    for ga, (best, state) in zip(gas, alone):
        mask, cost, stats = ga.best()
        np.testing.assert_array_equal(mask, best[0])
        assert cost == best[1]
        for key in ("chromosome_evals", "scan_total", "crossover_taken", "mutation_taken"):
            assert stats[key] == best[2][key]
        for a, b in zip(ga.state(), state):
            np.testing.assert_array_equal(a, b)
