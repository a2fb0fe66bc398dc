"""The compiled binding of the calls in a model's loop, on tensors without memory (no GPU needed): whatever it does
not take must end in the Python binding's own exception.  Every case runs in a process of its own, since what
these tests are about is a process that dies."""
import subprocess
import sys

import pytest

SETUP = """
import ctypes
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
import paper_2505_20334_amd as laq
from paper_2505_20334_amd import binding

lib = laq.load_library()
address = lambda name: ctypes.cast(getattr(lib, name), ctypes.c_void_p).value
# (no device here: a device and a stream number as a GPU would give them)
binding._native.bind(address("laq_evict"), address("laq_workspace_bytes"), address("laq_decode_attention"),
                     address("laq_decode_workspace_bytes"), address("laq_qcache_store"), lambda: 0, lambda device: 0)
binding._stream = lambda stream: 0

def made(*sizes):
    return torch.empty(*sizes, dtype=torch.bfloat16, device="cuda")

with FakeTensorMode():
    q, k, step, rows = made(1, 8, 8, 128), made(1, 2, 512, 128), made(1, 8, 128), made(128, 128)
    try:
        %s
        print("no exception")
    except Exception as e:
        print("raised", type(e).__name__, str(e).split(chr(10))[0])
"""


def outcome(call):
    res = subprocess.run([sys.executable, "-c", SETUP % call], capture_output=True, text=True, timeout=110)
    assert res.returncode == 0, "the process ended with %d: %s" % (res.returncode, res.stderr[-600:])
    return res.stdout.strip().splitlines()[-1]


def test_it_is_built_and_loads():
    from paper_2505_20334_amd import binding
    binding.load_library()
    assert binding._native is not None


@pytest.mark.parametrize("value", ["None", "b'max'"])
@pytest.mark.parametrize("name", ["pool_mode", "choose"])
def test_a_mode_that_is_no_text(name, value):
    assert outcome("laq.laq_evict(q, k, k, [64], 7, %s=%s)" % (name, value)).startswith("raised ValueError")


BATCHED = {"evict": "laq.laq_evict(x, k, k, [64], 7), q", "decode": "laq.laq_decode_attention(x, rows, rows, [64], 2, 512), step"}


@pytest.mark.parametrize("name", ["evict", "decode"])
def test_a_tensor_without_an_address(name):
    call, batch = BATCHED[name].rsplit(", ", 1)
    assert outcome("torch.vmap(lambda x: %s)(%s.unsqueeze(0))" % (call, batch)).startswith("raised RuntimeError Cannot access data pointer")


def test_a_tensor_without_an_address_in_the_query_cache():
    call = "torch.vmap(lambda x: laq.laq_qcache_store(q, x, 0))(step.unsqueeze(0))"
    assert outcome(call).startswith("raised RuntimeError Cannot access data pointer")


OUT_OF_MEMORY = """
        from torch.utils._python_dispatch import TorchDispatchMode
        class NoMemory(TorchDispatchMode):
            def __torch_dispatch__(self, func, types, args=(), kwargs=None):
                if "empty" in str(func):
                    raise torch.OutOfMemoryError("no memory")
                return func(*args, **(kwargs or {}))
        with NoMemory():
            %s
"""


@pytest.mark.parametrize("call", ["laq.laq_evict(q, k, k, [64], 7)", "laq.laq_decode_attention(step, rows, rows, [64], 2, 512)"])
def test_an_allocation_that_fails_raises_what_torch_raises(call):
    assert outcome(OUT_OF_MEMORY % call) == "raised OutOfMemoryError no memory"


def test_calls_work_without_the_compiled_binding():
    code = ("import sys, warnings\nsys.modules['paper_2505_20334_amd._native'] = None\nimport torch\nimport paper_2505_20334_amd as laq\n"
            "with warnings.catch_warnings(record=True) as told:\n    warnings.simplefilter('always')\n    laq.load_library()\n"
            "assert any('_native' in str(w.message) for w in told)\n"
            "x = torch.zeros(1, 2, 64, 128)\n"
            "for call in (lambda: laq.laq_evict(x, x, x, [8], 7), lambda: laq.laq_qcache_store(x, x[:, :, 0], 0),\n"
            "             lambda: laq.laq_decode_attention(x[:, :, 0], x[0, 0], x[0, 0], [32], 2, 64)):\n"
            "    try:\n        call()\n    except ValueError as e:\n        assert 'must live on the GPU' in str(e)\n"
            "    else:\n        raise AssertionError\n")
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=110)
    assert res.returncode == 0, res.stderr[-600:]
