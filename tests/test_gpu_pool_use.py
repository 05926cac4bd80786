"""Objects closed by one thread while another steps runs and batches, whose
first steps capture graphs: the steps succeed and give the results they give
alone."""
import threading

import numpy as np
import pytest

import pmp_inputs as gi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available()
    import paper_1610_10061_amd as pm
    pm.lib()
    return pm


def test_steps_beside_closing_threads(pm):
    import torch
    d = torch.from_numpy(gi.euclid_instance(120, 3)).cuda()
    inst = pm.Instance(d, 8)

    def runs():
        return ([pm.GA(inst, 128, 64, 1000, seed) for seed in range(6)],
                [pm.GA(inst, 128, 64, 1000, 50 + seed) for seed in range(6)])

    def step(alone, batched):
        batch = pm.Batch(batched)
        for k in range(3):
            for ga in alone:
                ga.step(8)
            batch.step(4 + k)
        batch.check()
        return [ga.best()[1] for ga in alone + batched], [ga.state()[1] for ga in alone + batched]

    costs, fits = step(*runs())
    alone, batched = runs()
    torch.cuda.synchronize()
    stop, bad = threading.Event(), []

    def close(t):
        stream = torch.cuda.Stream()
        masks = torch.from_numpy(gi.random_population(64, 120, 8, seed=t).view(np.int64)).cuda()
        masks = masks.view(torch.uint64)
        fit = torch.empty(64, dtype=torch.int64, device="cuda")
        torch.cuda.current_stream().synchronize()
        n = 0
        while not stop.is_set() and n < 2000:
            try:
                x = pm.Instance(d, 8 + t, stream) if n % 2 else pm.Instance(d, 8, stream)
                if not n % 2 and t == 0:
                    x.eval(masks, fit, stream=stream, asynchronous=True)
                x.close()
            except pm.PmpError as e:
                bad.append(str(e))
                return
            n += 1

    threads = [threading.Thread(target=close, args=(t,)) for t in range(2)]
    for th in threads:
        th.start()
    try:
        costs2, fits2 = step(alone, batched)
    finally:
        stop.set()
        for th in threads:
            th.join()
    assert not bad, bad
    assert costs2 == costs
    for a, b in zip(fits, fits2):
        assert np.array_equal(a, b)
