"""Walks past a row's first chunk (bit-exact against the oracle): rows that end
at, before and after a chunk, walks to a row's last position (one open
facility), chunks in which few and many chromosomes stop, the paired walk's
second half, tiles in device memory, and chromosomes without an open
facility, whose walk runs past the row and is reported."""
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


def _compare(pm, d, p, masks):
    P = masks.shape[0]
    inst = pm.Instance(d, p)
    fit, scan = np.zeros(P, np.int64), np.zeros(P, np.int64)
    pm.pmp_eval_population(inst.handle, masks, fit, scan)
    cost, scans = oracle.objective(d, masks, p, scan=True)
    np.testing.assert_array_equal(fit, cost)
    np.testing.assert_array_equal(scan, scans)


@pytest.mark.parametrize("m", [63, 64, 65, 128, 129, 191, 640])
def test_one_open_facility(pm, m):
    d = gi.euclid_instance(m, m)[: max(5, m // 3)]
    masks = gi.pack_masks([[j] for j in range(m)], m)  # every scan length 1..m
    _compare(pm, np.ascontiguousarray(d), 1, masks)


@pytest.mark.parametrize("m,p,far", [(130, 3, 0), (700, 2, 40), (1500, 5, 3), (200, 60, 100),
                                     (129, 40, 64), (8200, 4, 20)])
def test_few_and_many_stop_in_a_chunk(pm, m, p, far):
    """Random chromosomes, and `far` whose open facilities are all among the
    highest-numbered sites (ordered by the first client's distance, so whole
    rows keep them to the end)."""
    rng = np.random.default_rng([m, p])
    d = rng.integers(0, 3000, size=(37, m)).astype(np.int32)
    d += (np.arange(m, dtype=np.int32) * 7)[None, :]
    masks = gi.random_population(90, m, p, seed=m)
    if far:
        near_end = [rng.choice(np.arange(m - p - p // 2 - 1, m), p, replace=False)
                    for _ in range(far)]
        masks = np.concatenate([masks, gi.pack_masks([list(s) for s in near_end], m)])
    _compare(pm, d, p, masks)


@pytest.mark.parametrize("m,p", [(40, 20), (70, 3), (128, 2), (300, 4)])
def test_no_open_facility_is_reported(pm, m, p):
    inst = pm.Instance(gi.euclid_instance(m, 1), p)
    masks = gi.random_population(66, m, p, seed=1)
    masks[65] = 0
    fit = np.zeros(66, np.int64)
    with pytest.raises(pm.PmpError) as err:
        pm.pmp_eval_population(inst.handle, masks, fit)
    assert err.value.status == 4
    np.testing.assert_array_equal(fit[:65],
                                  oracle.objective(gi.euclid_instance(m, 1), masks[:65], p))


@pytest.mark.parametrize("m,p", [(255, 20), (256, 20), (257, 20), (320, 3), (1000, 100)])
@pytest.mark.parametrize("waves,P", [(4, 1), (8, 37), (16, 64), (16, 100)])
def test_both_chunk_reads(pm, monkeypatch, m, p, waves, P):
    """Chromosomes of four words and of five (the transposing read of the
    first chunk starts there), partly filled tiles, each wave count."""
    monkeypatch.setenv("PMP_EVAL_WAVES", str(waves))
    rng = np.random.default_rng([m, p, P])
    d = rng.integers(0, 2**31 - 1, size=(45, m)).astype(np.int32)
    _compare(pm, d, p, gi.random_population(P, m, p, seed=P))


@pytest.mark.parametrize("m,p", [(300, 238), (300, 237), (300, 280), (300, 299), (900, 895)])
def test_rows_shorter_than_a_chunk(pm, monkeypatch, m, p):
    """Rows of 2 to 64 entries through the single-client walk."""
    monkeypatch.setenv("PMP_EVAL_PAIRED", "0")
    d = np.random.default_rng([m, p]).integers(0, 50, size=(33, m)).astype(np.int32)
    _compare(pm, d, p, gi.random_population(70, m, p, seed=p))
