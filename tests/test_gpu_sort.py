"""The row sort of the preprocessing against numpy's stable argsort: row widths
at the edges of its shapes (waves x vectors x 64, and the widest row sorted in
LDS), distances of every pass count (no pass, one digit, several digits, keys
of one word and of two, the largest int32), heavy ties, rows of different
widths of distances in one matrix, device input with a row stride."""
import numpy as np
import pytest

import pmp_inputs as gi

pytestmark = pytest.mark.gpu

BITS = [0, 1, 6, 7, 8, 9, 14, 16, 17, 22, 25, 31]


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available()
    import paper_1610_10061_amd as pm
    pm.lib()
    return pm


def _matrix(m, seed):
    """One row per bit width (the widest value present), a row of few
    distinct values, a descending one and one of equal values."""
    rng = np.random.default_rng([seed, m])
    rows = []
    for b in BITS:
        r = rng.integers(0, 1 << b, size=m) if b else np.zeros(m, np.int64)
        if b:
            r[rng.integers(0, m)] = (1 << b) - 1
        rows.append(r)
    rows += [rng.integers(0, 3, m) * 70_000, np.arange(m)[::-1], np.full(m, 12345)]
    return np.stack(rows).astype(np.int32)


def _check(d, p, tables):
    pi, delta, ds = tables
    K = d.shape[1] - p + 1
    order = np.argsort(d, axis=1, kind="stable")[:, :K]
    sd = np.take_along_axis(d, order, 1)
    np.testing.assert_array_equal(pi, order)
    np.testing.assert_array_equal(ds, sd)
    np.testing.assert_array_equal(delta, np.diff(sd, axis=1, prepend=np.int32(0)))


@pytest.mark.parametrize("m", [2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 769, 1024, 1025, 1537,
                               2048, 2049, 2561, 3073, 4097, 5120, 5121, 6145, 7169, 8192, 8193,
                               10241, 12289, 14337, 16385, 18433, 20481, 23552, 23553])
def test_row_widths(pm, m):
    print("m", m, flush=True)
    d = _matrix(m, 1)
    for p in (1, max(1, m // 3)):
        _check(d, p, pm.Instance(d, p).tables())


def test_strided_device_rows(pm):
    import ctypes
    import torch
    m, ld, p = 300, 331, 7
    full = torch.full((15, ld), -5, dtype=torch.int32, device="cuda")  # the gap is never read
    d = _matrix(m, 2)
    full[:, :m] = torch.from_numpy(d).cuda()
    out = ctypes.c_void_p()
    assert pm.lib().pmp_preprocess(full.data_ptr(), ld, 15, m, p, 1,
                                   torch.cuda.current_stream().cuda_stream,
                                   ctypes.byref(out)) == 0
    _check(d, p, pm.pmp_instance_tables(out))
    pm.pmp_instance_destroy(out)


@pytest.mark.parametrize("m", [100, 9000, 23600])
def test_negative_distances_are_refused(pm, m):
    import torch
    d = np.array(gi.euclid_instance(40, 1)[:, :1].repeat(m, 1))
    d[39, m - 1] = -1
    for x in (d, torch.from_numpy(d).cuda()):
        with pytest.raises(pm.PmpError) as err:
            pm.Instance(x, 2)
        assert err.value.status == 1
    inst = pm.Instance(torch.from_numpy(d).cuda(), 2, asynchronous=True)
    with pytest.raises(pm.PmpError):
        inst.check()
