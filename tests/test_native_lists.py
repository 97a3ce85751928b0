"""Tensor lists of the batch entry point: the pointers and the errors are those of the
tensors one by one."""
import ctypes

import pytest
import torch

from paper_2203_09621_amd import _native as nat


class _Fake(torch.Tensor):
    """A CPU tensor that claims to lie on the device."""
    is_cuda = True


def _t(*shape, dtype=torch.float64):
    return torch.zeros(*shape, dtype=dtype).as_subclass(_Fake)


def test_pointers_of_a_list():
    ts = [_t(n, n) for n in (1, 3, 2, 3)]
    assert list(nat._devs(ts, "H1")) == [nat._dev(t, "H1").value for t in ts]
    assert len(nat._devs([], "H1")) == 0


@pytest.mark.parametrize("bad", [None, 1.0, torch.zeros(2, 2, dtype=torch.float64),
                                 _t(2, 2, dtype=torch.float32), _t(2, 3), _t(2), _t(2, 2, 2),
                                 _t(4, 4)[::2, ::2], _t(2, 2, dtype=torch.int64)])
def test_bad_entries_raise_as_one_by_one(bad):
    with pytest.raises(TypeError) as one:
        nat._dev(bad, "P0")
    with pytest.raises(TypeError) as many:
        nat._devs([_t(2, 2), bad, _t(3, 3)], "P0")
    assert str(one.value) == str(many.value)


def test_problem_stats_of_an_array():
    st = (nat.DmptProblemStats * 3)()
    for i, x in enumerate(st):
        x.layers, x.d0_layer, x.converged, x.k = 20 + i, 18 + i, i % 2, 1 + i
        x.d1_layer[:] = [3 * i, 3 * i + 1, 3 * i + 2]
        x.idem0 = 0.5 + i
        x.idem1[:] = [i + 0.25, i + 0.125, float("inf")]
    assert nat._problem_stats(st) == [x.as_dict() for x in st]
    assert ctypes.sizeof(nat.DmptProblemStats) == 64
