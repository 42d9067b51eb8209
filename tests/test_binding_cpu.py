"""The compiled stage calls take what the functions of the C ABI take, and refuse the rest. Calls that the library refuses on the
host: nothing is launched."""
import ctypes as C
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2412_14838_amd import dkv
from test_two_devices_cpu import STAND_INS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _desc(**kw):
    a = dict(n_layers=4, n_q_heads=4, n_kv_heads=2, head_dim=128, window=16, pool_kernel=7, layer_max=64, mean_budget=16, interval=2,
             dtype=dkv.DKV_BF16, n_seqs=1, total_tokens=300, max_seq_len=300)
    a.update(kw)
    return dkv.dkv_desc(**a)


def test_arguments_arrive_as_through_ctypes():
    """Every argument of a call in turn off by one step into what the library refuses: the same status as the plain C call's."""
    t = torch.zeros(4096, dtype=torch.uint8)
    at = t.data_ptr()
    good = [3, t, at, t, 80 * 128, 80 * 128, t, t, t, None, t, 1 << 40, 64]
    for i, bad in ((0, 4), (0, -1), (0, np.int64(9)), (1, None), (2, None), (2, at + 8), (3, None), (4, -1), (5, 127), (6, None), (7, None),
                   (8, None), (10, None), (11, 16)):
        a = list(good)
        a[i] = bad
        plain = [x.data_ptr() if isinstance(x, torch.Tensor) else (int(x) if isinstance(x, np.int64) else x) for x in a]
        d = _desc()
        want = dkv.load().dkv_decode_attention(C.byref(d), *plain)
        assert want < 0 and dkv.binding().dkv_decode_attention(d, *a) == want, (i, bad)


def test_what_is_no_argument_is_refused():
    t = torch.zeros(64, dtype=torch.uint8)
    b = dkv.binding()
    good = [_desc(), 1, t, t, 64]
    for i, bad in ((0, None), (0, b"short"), (1, 1.0), (1, "1"), (2, "x"), (2, 1.5), (4, object())):
        a = list(good)
        a[i] = bad
        with pytest.raises((TypeError, AttributeError)):
            b.dkv_apply_budgets(*a)
    with pytest.raises(TypeError):
        b.dkv_apply_budgets(*good[:-1])


def test_layers_of_a_call():
    t, d = torch.zeros(4096, dtype=torch.uint8), _desc()
    strides = (128, 300 * 128)
    with pytest.raises(dkv.DkvError) as e:                                # fewer queries than keys: null pointers, as ever
        dkv.dkv_score_window_layers(d, 0, [t], [t, t], *strides, t, t, t, 64)
    assert e.value.status == dkv.DKV_ERR_INVALID_ARG
    with pytest.raises(IndexError):
        dkv.dkv_score_window_layers(d, 0, [t, t, t], [t, t], *strides, t, t, t, 64)
    with pytest.raises(dkv.DkvError):
        dkv.dkv_score_window_layers(d, 0, [t] * 40, [t] * 40, *strides, t, t, t, 64)


def test_layers_may_come_from_any_iterable():
    """As ctypes took them: what is no sequence is read once. The status is that of a call the library refuses (32 layers of 4)."""
    t, d = torch.zeros(4096, dtype=torch.uint8), _desc()
    out = (128, 300 * 128, t, t, t, t, t)
    for make in (lambda n: (t for _ in range(n)), lambda n: map(lambda _: t, range(n)), lambda n: iter([t] * n), lambda n: dict.fromkeys(range(n), t).values(),
                 lambda n: torch.zeros(n, 4096, dtype=torch.uint8)):
        for call in (lambda q, k: dkv.dkv_score_window_layers(d, 0, q, k, *out[:5], stream=64),
                     lambda q, k: dkv.dkv_score_window_lse_layers(d, 0, q, k, *out[:3], make(32), t, t, stream=64),
                     lambda q, k: dkv.dkv_gather_kv_layers(d, 0, k, q, *out, 1 << 20, 1 << 18, 1 << 16, stream=64)):
            with pytest.raises(dkv.DkvError) as e:
                call(make(32), [t] * 32)
            assert e.value.status == dkv.DKV_ERR_INVALID_ARG
    with pytest.raises(IndexError):
        dkv.dkv_score_window_layers(d, 0, (t for _ in range(3)), [t, t], *out[:5], stream=64)


def test_a_descriptor_is_a_dkv_desc():
    """Bytes and other structures of its size are none, as through ctypes; a structure derived from it is one."""
    class Other(C.Structure):
        _fields_ = [("words", C.c_int32 * 15)]

    class Longer(dkv.dkv_desc):
        _fields_ = [("more", C.c_int32)]

    t, good = torch.zeros(64, dtype=torch.uint8), _desc()
    assert C.sizeof(Other) == C.sizeof(good)
    for bad in (bytes(good), bytearray(bytes(good)), memoryview(bytes(good)), np.frombuffer(bytes(good), np.int32), Other.from_buffer_copy(bytes(good))):
        with pytest.raises(TypeError):
            dkv.dkv_apply_budgets(bad, 5, t, t, 64)
    longer = Longer(*[getattr(good, name) for name, _ in dkv.dkv_desc._fields_], 7)
    for d in (good, longer):
        with pytest.raises(dkv.DkvError) as e:                            # 5 layers of 4
            dkv.dkv_apply_budgets(d, 5, t, t, 64)
        assert e.value.status == dkv.DKV_ERR_INVALID_ARG


class _Address(int):
    pass


def test_what_is_no_tensor_is_refused():
    """An address is a plain int, and the tensors of several layers are tensors: None and addresses among them are refused."""
    t, d = torch.zeros(4096, dtype=torch.uint8), _desc()
    for bad in (True, False, _Address(t.data_ptr()), np.int64(t.data_ptr())):
        with pytest.raises(AttributeError):
            dkv.dkv_apply_budgets(d, 5, bad, t, 64)
    for bad in (None, t.data_ptr(), True):
        with pytest.raises(AttributeError):
            dkv.dkv_score_window_layers(d, 0, [t, bad], [t, t], 128, 300 * 128, t, t, t, 64)
        with pytest.raises(AttributeError):
            dkv.dkv_score_window_layers(d, 0, [t, t], [bad, t], 128, 300 * 128, t, t, t, 64)


def test_a_list_may_change_while_it_is_read():
    """data_ptr() is Python code for what is no plain tensor: the list it empties is not read past its end."""
    t, d = torch.zeros(4096, dtype=torch.uint8), _desc()

    class Emptying:
        def __init__(self, of):
            self.of = of

        def data_ptr(self):
            self.of.clear()
            return t.data_ptr()

    layers = []
    layers += [Emptying(layers)] + [t] * 3
    with pytest.raises(dkv.DkvError) as e:                                # the three others are null pointers
        dkv.dkv_score_window_layers(d, 0, layers, [t] * 4, 128, 300 * 128, t, t, t, 64)
    assert e.value.status == dkv.DKV_ERR_INVALID_ARG and layers == []


def test_no_cpp_exception_reaches_python():
    """A list that would not fit memory a second time: the call refuses it (more layers than one takes), the process goes on."""
    program = r"""
import sys
sys.path.insert(0, "tests")
import resource, torch
from paper_2412_14838_amd import dkv
from test_binding_cpu import _desc
t = torch.zeros(4096, dtype=torch.uint8)
dkv.binding()
layers = [t] * 40000000                                                   # 320 MB
size = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (size + (64 << 20), resource.RLIM_INFINITY))
try:
    dkv.dkv_score_window_layers(_desc(), 0, layers, layers, 128, 300 * 128, t, t, t, 64)
except dkv.DkvError as e:
    print("refused", e.status)
"""
    run = subprocess.run([sys.executable, "-c", program], capture_output=True, text=True, cwd=ROOT, timeout=300)
    assert run.returncode == 0 and run.stdout.split() == ["refused", str(dkv.DKV_ERR_INVALID_ARG)], (run.returncode, run.stderr[-500:])


@pytest.mark.parametrize("layer", [2 ** 31 - 1, 2 ** 31 - 2, 4])
def test_layers_past_the_model_are_refused(layer):
    """Also where the first layer and their number add up past 2^31. Refused on the host: nothing is launched."""
    t, d = torch.zeros(4096 + 256, dtype=torch.uint8), _desc()
    t = t[-t.data_ptr() % 256:]                                           # as a workspace is aligned
    lib, at, room, ptrs = dkv.load(), t.data_ptr(), 1 << 40, (C.c_void_p * 2)(t.data_ptr(), t.data_ptr())
    block = 80 * 128
    for status in (
            lib.dkv_score_window_layers(C.byref(d), layer, 2, ptrs, ptrs, 128, 300 * 128, at, at, at, room, 64),
            lib.dkv_score_window_lse_layers(C.byref(d), layer, 2, ptrs, ptrs, 128, 300 * 128, at, ptrs, at, at, room, 64),
            lib.dkv_select_topk_layers(C.byref(d), layer, 2, at, at, at, at, at, room, 64),
            lib.dkv_gather_kv_layers(C.byref(d), layer, 2, ptrs, ptrs, 128, 300 * 128, at, at, at, at, at, 4 * block, 2 * block, block, 64),
            lib.dkv_decode_attention_layers(C.byref(d), layer, 2, at, at, at, 4 * block, 2 * block, block, at, at, at, None, at, room, 64)):
        assert status == dkv.DKV_ERR_INVALID_ARG


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_stream_of_a_call(tmp_path):
    """An address, an object with cuda_stream, or (None) torch's current stream at the time of the call: what the launch gets. The
    HIP calls go to stand-ins."""
    src, lib = tmp_path / "stand_ins.cpp", tmp_path / "libstand_ins.so"
    launch = "int hipLaunchKernel(const void*, d3, d3, void**, size_t, void*) { return 0; }"
    assert launch in STAND_INS
    src.write_text(STAND_INS.replace(launch, "static void* launched_on; void* stand_in_stream() { return launched_on; }\n"
                                     "int hipLaunchKernel(const void*, d3, d3, void**, size_t, void* s) { launched_on = s; return 0; }"))
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    program = r"""
import sys
sys.path.insert(0, "tests")
import ctypes as C, sys
stand_ins = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
stand_ins.stand_in_stream.restype = C.c_void_p
import torch
from paper_2412_14838_amd import dkv
from test_binding_cpu import _desc
now = [0, 0x500]
torch.cuda.current_device = lambda: now[0]
torch._C._cuda_getCurrentRawStream = lambda device: now[1] + device
class Stream:
    cuda_stream = 0x700
for stream in (0x300, 0, Stream()):
    dkv.dkv_apply_budgets(_desc(), 2, 0x1000, 0x1000, stream)
    print(stand_ins.stand_in_stream())
for now[:] in ([0, 0x500], [3, 0x600], [0, 0]):
    dkv.dkv_apply_budgets(_desc(), 2, 0x1000, 0x1000)
    print(stand_ins.stand_in_stream())
"""
    run = subprocess.run([sys.executable, "-c", program, str(lib)], capture_output=True, text=True, cwd=ROOT, timeout=300)
    assert run.returncode == 0, run.stderr[-800:]
    assert run.stdout.split() == [str(x or None) for x in (0x300, 0, 0x700, 0x500, 0x603, 0)]
