"""Addresses that the binding computes instead of asking a view for them."""
import numpy as np
import pytest
import torch

from paper_2412_14838_amd import dkv


@pytest.mark.parametrize("t", [torch.zeros(5, 3, 4), torch.zeros(5, 8, dtype=torch.bfloat16), torch.zeros(9, 6, 2)[1:6, ::2],
                               torch.zeros(4, 5, 7).transpose(0, 1), torch.zeros(5, 0)])
def test_layer_ptr_is_the_address_of_the_view(t):
    for layer in (0, 1, 4, -1, -5, np.int64(3)):
        assert dkv.layer_ptr(t, layer) == t.data_ptr() + (t[layer].storage_offset() - t.storage_offset()) * t.element_size()
        assert type(dkv.layer_ptr(t, layer)) is int
    for layer in (5, -6):
        with pytest.raises(IndexError):
            dkv.layer_ptr(t, layer)
    assert dkv._ptr(None) is None and dkv._ptr(64) == 64 and dkv._ptr(t) == t.data_ptr()
