"""The reduction of the client tiles' partial sums and the error bits it hands
over: tile counts around its wave split (one wave, a wave per four tiles, 16
waves, more tiles than 16 waves take in one round) and populations around its
64 chromosomes per workgroup, bit-exact against the oracle; a waiting call
reports its own errors only."""
import numpy as np
import pytest

import oracle
import pmp_inputs as gi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available()
    import paper_1610_10061_amd as pm
    pm.lib()
    return pm


@pytest.mark.parametrize("clients,P", [(150, 1), (40, 63), (30, 64), (9, 65), (2, 130), (1, 7)])
def test_tile_counts_and_populations(pm, monkeypatch, clients, P):
    d = gi.euclid_instance(150, 4)
    p = 11
    monkeypatch.setenv("PMP_CLIENTS_PER_BLOCK", str(clients))
    inst = pm.Instance(d, p)
    masks = gi.random_population(P, 150, p, seed=P)
    fit, scan = np.zeros(P, np.int64), np.zeros(P, np.int64)
    pm.pmp_eval_population(inst.handle, masks, fit, scan)
    cost, scans = oracle.objective(d, masks, p, scan=True)
    np.testing.assert_array_equal(fit, cost)
    np.testing.assert_array_equal(scan, scans)


def test_waiting_calls_report_their_own_errors(pm):
    import torch
    d = gi.euclid_instance(90, 5)
    inst = pm.Instance(torch.from_numpy(d).cuda(), 7)

    def dev(p):
        m = gi.random_population(70, 90, p, seed=p)
        return torch.from_numpy(m.view(np.int64)).cuda().view(torch.uint64)

    good, bad = dev(7), dev(6)
    want = oracle.objective(d, gi.random_population(70, 90, 7, seed=7), 7)
    fit = torch.empty(70, dtype=torch.int64, device="cuda")
    for evaluate in (pm.pmp_eval_population, pm.pmp_eval_population_noalloc):
        with pytest.raises(pm.PmpError) as err:
            evaluate(inst.handle, bad, fit)
        assert err.value.status == 4
        evaluate(inst.handle, good, fit)  # the bits of the call before are gone
        np.testing.assert_array_equal(fit.cpu().numpy(), want)
        inst.check()
        evaluate(inst.handle, bad, fit, asynchronous=True)
        with pytest.raises(pm.PmpError):
            inst.check()
        inst.check()
