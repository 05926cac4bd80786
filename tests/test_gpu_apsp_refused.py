"""Edge weights whose paths might not fit int32 are refused: d is left alone,
in a fraction of an accepted call's time, and the next call (on another stream)
is not disturbed."""
import time

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available()
    import paper_1610_10061_amd as pm
    pm.lib()
    return pm


def weights(n, seed):
    rng = np.random.default_rng([seed, n])
    w = rng.integers(1, 100, (n, n)).astype(np.int32)
    w[rng.random((n, n)) < 0.9] = -1
    return w


# one tile; the rounds enqueued without a wait (8 tiles) and one more
@pytest.mark.parametrize("n", [2, 64, 65, 512, 513, 700])
def test_refused_then_accepted(pm, n):
    import torch
    w = weights(n, 1)
    large = w.copy()
    large[0, 1] = 0x7FFFFFFE // (n - 1) + 1
    ok = w.copy()
    ok[0, 1] = 0x7FFFFFFE // (n - 1)
    d = torch.full((n, n), -7, dtype=torch.int32, device="cuda")
    with pytest.raises(pm.PmpError) as e:
        pm.pmp_apsp(torch.from_numpy(large).cuda(), d)
    assert e.value.status == pm.PMP_EUNSUPPORTED
    assert bool((d == -7).all())
    stream = torch.cuda.Stream()
    wd = torch.from_numpy(ok).cuda()
    torch.cuda.synchronize()
    pm.pmp_apsp(wd, d, stream)
    assert np.array_equal(d.cpu().numpy(), oracle.apsp(ok))


def test_refused_without_the_rounds(pm):
    import torch
    n = 3000
    w = torch.from_numpy(weights(n, 2)).cuda()
    d = torch.empty_like(w)

    def least(call):
        call()
        out = []
        for _ in range(7):
            t = time.perf_counter()
            call()
            out.append(time.perf_counter() - t)
        return min(out)

    accepted = least(lambda: pm.pmp_apsp(w, d))
    w[0, 1] = 0x7FFFFFFF

    def refuse():
        with pytest.raises(pm.PmpError):
            pm.pmp_apsp(w, d)

    assert least(refuse) < 0.4 * accepted
