"""The C struct of a Window is made again whenever a field's values change, in place too, and
a window that has been used still copies and pickles."""
import copy
import pickle

import numpy as np
import pytest

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
