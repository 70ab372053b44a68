"""The C struct of a Window is made again whenever a field's values change, in place too, and
a window that has been used still copies and pickles."""
import copy
import pickle

import numpy as np
import pytest
import torch

import paper_2608_02947_amd as atf


@pytest.mark.parametrize("kind", [list, tuple, np.array])
def test_window_struct_follows_its_values(kind):
    theta = [10.0 ** (-r / 8) for r in range(32)]
    w = atf.Window(64, 1e4, 2.0, inv_freq=kind(theta))
    first = atf.atf_window_table(w)
    assert w.as_c()[0] is w.as_c()[0]
    if kind is not tuple:
        w.inv_freq[3] = 0.5  # in place
        theta[3] = 0.5
        assert np.array_equal(atf.atf_window_table(w), atf.atf_window_table(atf.Window(64, 1e4, 2.0, inv_freq=theta)))
        assert not np.array_equal(atf.atf_window_table(w), first)
    w.k = 5.0
    assert np.array_equal(atf.atf_window_table(w), atf.atf_window_table(atf.Window(64, 1e4, 5.0, inv_freq=theta)))
    w.inv_freq = None
    w.k_profile = kind([3.0] * 32)
    assert np.array_equal(atf.atf_window_table(w), atf.atf_window_table(atf.Window(64, 1e4, 3.0)))
    for again in (copy.copy(w), copy.deepcopy(w), pickle.loads(pickle.dumps(w))):
        assert np.array_equal(atf.atf_window_table(again), atf.atf_window_table(w))
    with pytest.raises(ValueError):
        w.k_profile = kind([3.0] * 31)
        atf.atf_window_table(w)


class _Own:
    """A number of a type of its own, changed in place."""

    def __init__(self, x):
        self.x = x

    def __float__(self):
        return self.x


def _zero_d(x):
    return np.array(x)


def _tensor(x):
    return torch.tensor(x, dtype=torch.float64)


def _set(cell, x):
    """Change a mutable number in place."""
    if isinstance(cell, _Own):
        cell.x = x
    elif isinstance(cell, np.ndarray):
        cell.fill(x)
    else:
        cell.fill_(x)


@pytest.mark.parametrize("make", [_zero_d, _tensor, _Own])
def test_window_struct_follows_mutable_numbers(make):
    """A number that can change in place (a 0-d array or tensor, an object), in a scalar field
    or as an element of a list, a tuple or an object array."""
    table = atf.atf_window_table
    w = atf.Window(64, 1e4, make(2.0))
    assert np.array_equal(table(w), table(atf.Window(64, 1e4, 2.0)))
    _set(w.k, 5.0)
    assert np.array_equal(table(w), table(atf.Window(64, 1e4, 5.0)))

    theta = [10.0 ** (-r / 8) for r in range(32)]
    changed = theta[:3] + [0.5] + theta[4:]
    kinds = [list, tuple]
    if make is _Own:
        kinds.append(lambda cells: np.array(cells, dtype=object))
    for kind in kinds:
        for field in ("inv_freq", "k_profile"):
            cells = [make(x) for x in theta]
            w = atf.Window(64, 1e4, 2.0, **{field: kind(cells)})
            assert np.array_equal(table(w), table(atf.Window(64, 1e4, 2.0, **{field: theta})))
            _set(cells[3], 0.5)
            assert np.array_equal(table(w), table(atf.Window(64, 1e4, 2.0, **{field: changed})))


def test_window_struct_follows_a_tensor_given_as_a_list():
    th = torch.tensor([10.0 ** (-r / 8) for r in range(32)], dtype=torch.float64)
    w = atf.Window(64, 1e4, 2.0, inv_freq=list(th))  # 0-d views of it
    atf.atf_window_table(w)
    th[3] = 0.5
    assert np.array_equal(atf.atf_window_table(w), atf.atf_window_table(atf.Window(64, 1e4, 2.0, inv_freq=th)))


def test_window_struct_edited_by_a_caller_is_not_kept():
    w = atf.Window(64, 1e4, 2.0, inv_freq=[10.0 ** (-r / 8) for r in range(32)])
    first = atf.atf_window_table(w)
    cw, (th, _) = w.as_c()
    cw.k = 9.0
    assert np.array_equal(atf.atf_window_table(w), first)
    th = w.as_c()[1][0]
    th[3] = 0.5
    assert np.array_equal(atf.atf_window_table(w), first)


@pytest.mark.parametrize("number", [int, float, bool, np.float64, np.float32, np.int64])
def test_window_struct_is_kept_for_plain_numbers(number):
    w = atf.Window(64, 1e4, number(1), inv_freq=[number(1)] * 32, k_profile=(number(1),) * 32)
    assert w.as_c()[0] is w.as_c()[0]
