"""Host integers of the binding (dims, boxes, capacities): the forms it takes,
and numbers beyond 64 bits, which raise instead of wrapping around."""
import numpy as np
import pytest

import oracle
import paper_2505_21266_amd as dms

DIMS = (5, 4, 3)
FORMS = [(5, 4, 3), [5, 4, 3], np.array([5, 4, 3]), np.array([[5, 4, 3]]), np.array([[5], [4], [3]]), (5.9, 4.0, 3),
         np.array([5, 4, 3], np.int32), (np.int64(5), 4, np.uint8(3))]
REFUSED = [((1 << 64) + 5, 4, 3), [5, 4, -(1 << 63) - 1], (5, 1 << 63, 3)]


@pytest.mark.parametrize("form", FORMS, ids=[str(i) for i in range(len(FORMS))])
def test_three_integers(form):
    assert list(dms._arr3(form)[1]) == [5, 4, 3]
    # through a call: the host pairing on dims of this form
    v = np.random.default_rng(3).random(DIMS[::-1], dtype=np.float32)
    o = oracle.order(v)
    rec, _, _ = oracle.lower_stars(o, DIMS)
    crit, _ = oracle.critical_simplices(rec, DIMS)
    want = oracle.d0_pairs(o, rec, DIMS, crit[1])
    got = dms.d0_pairs_host(rec, o, form, crit[1])
    assert (got[0] == want[0]).all() and (got[1] == want[1]).all()


@pytest.mark.parametrize("bad", REFUSED, ids=[str(i) for i in range(len(REFUSED))])
def test_integers_beyond_64_bits(bad):
    with pytest.raises(OverflowError):
        dms._arr3(bad)
    with pytest.raises(OverflowError):
        dms.d0_pairs_host(np.zeros((60, 4), np.uint32), np.arange(60, dtype=np.int32), bad, np.zeros(0, np.int64))


def test_wrong_counts():
    for bad in ((5, 4), (5, 4, 3, 2), 5, np.zeros((3, 2), np.int64)):
        with pytest.raises((ValueError, TypeError)):
            dms._arr3(bad)
    with pytest.raises((ValueError, TypeError)):
        dms._arr3(("a", "b", "c"))


@pytest.mark.parametrize("cap", [(1, 2, 3, 4), [1, 2, 3, 4], np.array([[1, 2], [3, 4]]), np.arange(1, 5, dtype=np.uint32)],
                         ids=["tuple", "list", "square", "uint32"])
def test_capacities(cap):
    assert list(dms._int64s(cap, 4)) == [1, 2, 3, 4]


@pytest.mark.parametrize("cap", [(1 << 70, 0, 0, 0), [0, 0, 0, 1 << 63]], ids=["tuple", "list"])
def test_capacities_beyond_64_bits(cap):
    with pytest.raises(OverflowError):
        dms._int64s(cap, 4)


@pytest.mark.parametrize("values", [[0.5, 1.0], 3.0, np.zeros((2, 2, 2), np.float32), None],
                         ids=["list", "number", "array", "none"])
def test_pipeline_refuses_host_values(values):
    with pytest.raises(TypeError, match="GPU tensor"):
        dms.gradient_pipeline(values)
