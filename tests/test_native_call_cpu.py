"""Argument checks of the binding's native host path (no device is touched: they fail before the library is called)."""
import os
import subprocess
import sys

import pytest
import torch

from paper_2311_10090_amd import binding


@pytest.fixture(scope="module")
def call():
    binding.load_library()
    return binding._call


@pytest.mark.parametrize("name,extra", [("reset", (1,)), ("step", ()), ("rollout", (4,)), ("rollout_ac", (4,)), ("set_policy", ()),
                                        ("set_critic", ()), ("set_gru_policy", ()), ("set_gru_critic", ())])
def test_bad_arguments_are_refused(call, name, extra):
    fn = getattr(call, name)
    pointers = {"reset": 1, "step": 4, "rollout": 5, "rollout_ac": 8, "set_policy": 6, "set_critic": 6, "set_gru_policy": 10,
                "set_gru_critic": 4}[name]
    with pytest.raises(TypeError):
        fn(0, 0, *extra, *(None,) * (pointers - 1))                      # one argument short
    for k in range(pointers):
        args = [None] * pointers
        args[k] = torch.zeros(4)                                         # host memory
        with pytest.raises(AssertionError):
            fn(0, 0, *extra, *args)
        args[k] = "not a tensor"
        with pytest.raises(TypeError):
            fn(0, 0, *extra, *args)


# Tensors without storage: what a call gets inside a function transform.  In a child process, because an exception that
# leaves a native function unhandled ends the process.
TRANSFORMED = """
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from paper_2311_10090_amd import binding
binding.load_library()
arguments = {"reset": ((1,), "f"), "step": ((), "bffb"), "rollout": ((4,), "fbfbf"), "rollout_ac": ((4,), "fbfffbff"),
             "set_policy": ((), "f" * 6), "set_critic": ((), "f" * 6), "set_gru_policy": ((), "f" * 10), "set_gru_critic": ((), "f" * 4)}
with FakeTensorMode():
    tensors = {"f": torch.empty(3, 4, device="cuda"), "b": torch.empty(3, 4, device="cuda", dtype=torch.uint8)}
    for name, (extra, types) in arguments.items():
        for k, kind in enumerate(types):
            def call(x):
                args = [None] * len(types)
                args[k] = x
                getattr(binding._call, name)(0, 0, *extra, *args)
                return x
            for transform in (torch.vmap,) + ((lambda f: torch.func.grad(lambda x: f(x).sum()),) if kind == "f" else ()):
                try:
                    transform(call)(tensors[kind])
                except RuntimeError as e:
                    assert "storage" in str(e), (name, k, e)
                else:
                    raise SystemExit("%s accepted argument %d" % (name, k))
print("refused")
"""


def test_tensors_without_storage_raise():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", TRANSFORMED], cwd=root, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("refused"), (r.returncode, r.stderr[-2000:])
