"""Device memory kept between objects: instances made, used and destroyed from
several threads on their own streams (blocks change hands between them) give
the oracle's results; the memory kept is bounded."""
import threading

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


def test_threads_and_streams(pm):
    import torch
    shapes = [(60, 90, 5), (61, 90, 6), (120, 300, 20), (40, 1000, 9)]
    cases = []
    for t, (n, m, p) in enumerate(shapes):
        d = gi.euclid_instance(m, t)[:n].copy()
        masks = gi.random_population(100, m, p, seed=t)
        cases.append((torch.from_numpy(d).cuda(), p,
                      torch.from_numpy(masks.view(np.int64)).cuda().view(torch.uint64),
                      oracle.objective(d, masks, p)))
    torch.cuda.synchronize()
    wrong = []

    def work(t):
        stream = torch.cuda.Stream()
        for k in range(24):
            d, p, masks, want = cases[(t + k) % len(cases)]
            inst = pm.Instance(d, p, stream)
            fit = torch.empty(100, dtype=torch.int64, device="cuda")
            stream.wait_stream(torch.cuda.current_stream())
            inst.eval(masks, fit, stream=stream, asynchronous=k % 2 == 1)
            if k % 3 == 0:  # destroyed with its work still enqueued
                inst.close()
            stream.synchronize()
            if not np.array_equal(fit.cpu().numpy(), want):
                wrong.append((t, k))
            inst.close()

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not wrong


def test_kept_memory_is_bounded(pm):
    import torch
    pm.Instance(torch.zeros((8, 64), dtype=torch.int32, device="cuda"), 1).close()
    d = torch.zeros((2000, 4096), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for k in range(12):  # tables of 80 to 300 MB, no two of one size
        insts = [pm.Instance(d[: 1000 + 70 * k + 10 * q].repeat(1 + q, 1), 2) for q in range(4)]
        for i in insts:
            i.close()
    torch.cuda.empty_cache()
    torch.cuda.synchronize()
    assert free0 - torch.cuda.mem_get_info()[0] <= (1024 + 128) << 20
