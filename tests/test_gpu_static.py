"""Static sums of the preprocessing (column sums, total, near counts), read
back as features 10, 11 and 13: one and many counting workgroups, rows of one
and of many counted entries, odd facility numbers (two counts share a word),
more facilities than a column block, a single client; synchronous and
asynchronous.  Bit-exact against the oracle's definitions."""
import numpy as np
import pytest

import pmp_inputs as gi
from oracle import learned

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available()
    import paper_1610_10061_amd as pm
    pm.lib()
    return pm


@pytest.mark.parametrize("n,m,p", [(1, 5, 2), (3, 65, 64), (700, 65, 2), (130, 255, 1),
                                   (257, 257, 40), (90, 1025, 3), (1200, 901, 4), (400, 4095, 9)])
@pytest.mark.parametrize("asynchronous", [False, True])
def test_features_from_static_sums(pm, n, m, p, asynchronous):
    import torch
    rng = np.random.default_rng([n, m, p])
    d = rng.integers(0, 2**20, (n, m)).astype(np.int32)
    dd = torch.from_numpy(d).cuda()
    inst = pm.Instance(dd, p, asynchronous=asynchronous)
    masks = gi.random_population(1, m, p, seed=1)
    got = pm.pmp_features(inst.handle, masks)[0]
    colsum, total, near, L = learned.static_sums(d, p)
    np.testing.assert_array_equal(got[:, 10], learned._q(colsum, m, float(max(total, 1))))
    np.testing.assert_array_equal(got[:, 11], learned._q(near, m, float(n) * float(L)))
    inst.check()


def test_host_rows_with_and_without_gaps(pm):
    import ctypes
    d = gi.euclid_instance(70, 3)
    wide = np.full((70, 77), -1, np.int32)
    wide[:, :70] = d
    want = pm.Instance(d, 4).tables()
    out = ctypes.c_void_p()
    assert pm.lib().pmp_preprocess(wide.ctypes.data, 77, 70, 70, 4, 0, None,
                                   ctypes.byref(out)) == 0
    for a, b in zip(pm.pmp_instance_tables(out), want):
        np.testing.assert_array_equal(a, b)
    pm.pmp_instance_destroy(out)
