"""Rounds of the blocked shortest paths: one to four tiles per side and edges
around them, paths that need every vertex (a long chain in random order, so
each tile's closing and both panel products matter), row strides on both
sides, the largest weights that fit, and refused weights, which leave the
output alone.  Bit-exact against the oracle."""
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


def _chain(n, seed):
    """A directed chain over a random vertex order, and a few shortcuts."""
    rng = np.random.default_rng([seed, n])
    w = np.full((n, n), -1, np.int32)
    order = rng.permutation(n)
    w[order[:-1], order[1:]] = rng.integers(0, 5, n - 1)
    a, b = rng.integers(0, n, (2, n // 8 + 1))
    w[a, b] = rng.integers(100, 10_000, len(a))
    return w


@pytest.mark.parametrize("n", [3, 16, 63, 64, 65, 127, 128, 129, 192, 193, 256, 257, 321])
def test_chains(pm, n):
    w = _chain(n, 1)
    np.testing.assert_array_equal(pm.pmp_apsp(w), oracle.apsp(w))


def test_strides_and_largest_weights(pm):
    import torch
    n, ldw, ldd = 130, 133, 141
    w = _chain(n, 2)
    w[w > 100] = (2**31 - 2) // (n - 1)
    wd = torch.full((n, ldw), 3, dtype=torch.int32, device="cuda")
    wd[:, :n] = torch.from_numpy(w).cuda()
    out = torch.full((n, ldd), 77, dtype=torch.int32, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    assert pm.lib().pmp_apsp(wd.data_ptr(), ldw, n, out.data_ptr(), ldd, 1, st) == 0
    got = out.cpu().numpy()
    np.testing.assert_array_equal(got[:, :n], oracle.apsp(w))
    assert (got[:, n:] == 77).all()


def test_refused_weights_leave_the_output(pm):
    import torch
    w = torch.from_numpy(_chain(70, 3)).cuda()
    w[3, 5] = 2**31 - 1
    out = torch.full((70, 70), 5, dtype=torch.int32, device="cuda")
    with pytest.raises(pm.PmpError) as err:
        pm.pmp_apsp(w, out)
    assert err.value.status == pm.PMP_EUNSUPPORTED
    assert bool((out == 5).all())
    w[3, 5] = -1
    np.testing.assert_array_equal(pm.pmp_apsp(w, out).cpu().numpy(), oracle.apsp(w.cpu().numpy()))
