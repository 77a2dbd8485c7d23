"""Host checks of the binding's size helper."""
import ctypes

import pytest

from paper_2607_06763_amd import gdn_tree as G


def test_meta_bytes_takes_integers_only():
    """An equal argument of another type is refused whatever was asked before."""
    n = G.meta_bytes(2, 7)
    assert n == G.lib().gdn_tree_meta_bytes(2, 7) and n == G.meta_bytes(2, 7)
    with pytest.raises(ctypes.ArgumentError):
        G.meta_bytes(2.0, 7)
    with pytest.raises(ctypes.ArgumentError):
        G.meta_bytes(2, 7.0)
