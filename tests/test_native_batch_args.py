"""What the batch entry point hands to the library: the arrays hold an entry for every
problem, whatever the length and kind of the lists they are made from."""
import pytest
import torch

from paper_2203_09621_amd import _native as nat


class _Fake(torch.Tensor):
    """A CPU tensor that claims to lie on the device."""
    is_cuda = True


def _t(n):
    return torch.zeros(n, n, dtype=torch.float64).as_subclass(_Fake)


@pytest.fixture
def passed(monkeypatch):
    """The lists of the four pointer arrays of the last call."""
    seen = []

    def response(batch, *args):
        seen[:] = [list(a) for a in args[:4]]
        return 0

    monkeypatch.setattr(nat.LIB, "dmpt_batch_response", response)
    return seen


def _batch(count=3):
    return [_t(2 + p) for p in range(count)], [[_t(2 + p)] * (1 + p % 2) for p in range(count)]


@pytest.mark.parametrize("given", [0, 1, 2, 3])
def test_missing_p0_entries_are_null(passed, given):
    """P0 may be left out: a list shorter than the batch, or an empty one, is no error,
    and the problems past its end write no P0."""
    H0s, H1s = _batch()
    P0s = [_t(2 + p) for p in range(given)]
    nat.dmpt_batch_response(None, H0s, H1s, P0s=P0s)
    assert passed[2] == [t.data_ptr() for t in P0s] + [None] * (3 - given)


def test_too_many_p0_entries_are_refused(passed):
    H0s, H1s = _batch()
    with pytest.raises(IndexError):
        nat.dmpt_batch_response(None, H0s, H1s, P0s=[_t(2)] * 4)
    assert not passed


def test_iterators_are_walked_once(passed):
    H0s, H1s = _batch()
    P0s = [_t(2 + p) for p in range(3)]
    P1s = [[_t(2 + p)] * (1 + p % 2) for p in range(3)]
    nat.dmpt_batch_response(None, H0s, (iter(h) for h in H1s), P0s=iter(P0s),
                            P1s=(iter(p) for p in P1s))
    assert passed[1] == [t.data_ptr() for h in H1s for t in h]
    assert passed[2] == [t.data_ptr() for t in P0s]
    assert passed[3] == [t.data_ptr() for p in P1s for t in p]


@pytest.mark.parametrize("P1s", [[], [[_t(2)], [_t(3)], [_t(4)]]])
def test_too_few_p1_entries_are_refused(passed, P1s):
    H0s, H1s = _batch()
    with pytest.raises(ValueError):
        nat.dmpt_batch_response(None, H0s, H1s, P1s=P1s)
    assert not passed


@pytest.mark.parametrize("drop_h0,drop_h1", [(1, 0), (0, 1), (3, 4)])
def test_fewer_inputs_than_the_batch_holds_are_refused(passed, monkeypatch, drop_h0, drop_h1):
    monkeypatch.setattr(nat.LIB, "dmpt_batch_init", lambda *args: 0)
    monkeypatch.setattr(nat, "_stream", lambda s: None)
    H0s, H1s = _batch()
    batch = nat.dmpt_batch_init([2, 3, 4], [1, 1, 2], [len(h) for h in H1s])
    nat.dmpt_batch_response(batch, H0s, H1s)
    assert len(passed[0]) == 3 and len(passed[1]) == 4
    passed.clear()
    flat = [[h] for hs in H1s for h in hs]
    with pytest.raises(ValueError):
        nat.dmpt_batch_response(batch, H0s[:3 - drop_h0], flat[:4 - drop_h1])
    assert not passed
