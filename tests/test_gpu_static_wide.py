"""Instances of 28673 to 32768 facilities, where the static sums' launch needs
a little more than 64 KB of LDS: made, and their tables those of a stable sort
by distance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available()
    import paper_1610_10061_amd as pm
    pm.lib()
    return pm


@pytest.mark.parametrize("m", [28672, 28673, 30001, 32768, 32769])
def test_tables(pm, m):
    import torch
    n, p = 3, 11
    d = np.random.default_rng(m).integers(0, 2**18, (n, m)).astype(np.int32)
    inst = pm.Instance(torch.from_numpy(d).cuda(), p)
    pi, delta, ds = inst.tables()
    order = np.argsort(d, axis=1, kind="stable")[:, :m - p + 1]
    want = np.take_along_axis(d, order, axis=1)
    np.testing.assert_array_equal(pi, order.astype(np.uint16))
    np.testing.assert_array_equal(ds, want)
    np.testing.assert_array_equal(delta, np.diff(want, axis=1, prepend=0))
    inst.check()
