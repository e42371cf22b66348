"""Argument checks of the binding's native host path (no device is touched: they fail before the library is called)."""
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
