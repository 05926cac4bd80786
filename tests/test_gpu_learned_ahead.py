"""Learned runs whose next population is made in the resolve step's launch
(an even number of crossover steps, an even number of mutation attempts, the
attempts evaluated at once) against the attempt-by-attempt schedule, which
samples each generation by itself: the same populations, group bests, scores,
network parameters and counters, whatever the calls' lengths, with the
network set and taken away between generations."""
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


# crossover steps, mutation attempts: (4, 4) and (2, 2) are made ahead,
# (3, 4), (4, 3) and (3, 3) are not
@pytest.mark.parametrize("X,Y", [(4, 4), (2, 2), (3, 4), (4, 3), (3, 3)])
@pytest.mark.parametrize("mode", ["graph", "kernels"])
def test_population_made_ahead_equals_sampled(pm, monkeypatch, X, Y, mode):
    d = gi.euclid_instance(130, 11)
    p, P, NT, G = 13, 96, 32, 60
    out = []
    for spec in ("1", "0"):
        monkeypatch.setenv("PMP_GA_MODE", mode)
        monkeypatch.setenv("PMP_GA_SPEC", spec)
        print("made ahead", X, Y, mode, spec, flush=True)
        kw = dict(candidates=16, learned_iters=2, explore_permille=100, train_every=1, lr=1e-3)
        inst = pm.Instance(d, p)
        ga = pm.GA(inst, P, NT, G, 3, crossover_iters=X, mutation_iters=Y)
        model = pm.Model(4)
        seen = []
        ga.step(3)  # plain
        ga.set_model(model, **kw)
        for steps in (1, 8, 3, 17):
            ga.step(steps)
            pop, fit, gm, gc = ga.state()
            np.testing.assert_array_equal(fit, oracle.objective(d, pop, p))
            rep = ga.replay()
            seen += [pop, fit, gm, gc, model.params(), rep["scores"], rep["swap"],
                     rep["weight"], rep["target"]]
        ga.set_model(None)
        ga.step(9)  # plain again
        ga.set_model(model, **kw)
        ga.step(100)  # past the run's end
        seen += list(ga.state()) + [model.params()]
        out.append((seen, ga.best()[2]))
        ga.close()
        inst.close()
    for a, b in zip(out[0][0], out[1][0]):
        np.testing.assert_array_equal(a, b)
    for k in ("chromosome_evals", "swap_tried", "swap_taken", "mutation_taken",
              "crossover_taken", "scan_total", "generations", "done"):
        assert out[0][1][k] == out[1][1][k], k
    assert out[0][1]["swap_taken"] > 0
