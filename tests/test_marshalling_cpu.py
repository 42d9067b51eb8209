"""Addresses that the binding computes instead of asking a view for them."""
import ctypes as C

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


def test_pack_zero_tail_validates_its_arguments():
    lib = dkv.load()
    d = dkv.dkv_desc(n_layers=2, n_q_heads=2, n_kv_heads=2, head_dim=64, window=16, pool_kernel=7, layer_max=64, mean_budget=16,
                     interval=2, dtype=dkv.DKV_BF16, n_seqs=1, total_tokens=300, max_seq_len=300)
    fake = C.c_void_p(0x1000)
    good = [fake, fake, fake, 10, None]
    for i, bad in ((0, None), (1, None), (2, None), (0, C.c_void_p(0x1004)), (1, C.c_void_p(0x1008)), (3, -1)):
        a = list(good)
        a[i] = bad
        assert lib.dkv_pack_zero_tail(C.byref(d), *a) == dkv.DKV_ERR_INVALID_ARG
    assert lib.dkv_pack_zero_tail(None, *good) == dkv.DKV_ERR_INVALID_ARG
