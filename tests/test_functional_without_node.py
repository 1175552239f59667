"""When the PyTorch entry points may run without an autograd node (CPU): never inside a derivative, a transform or a trace."""
import importlib.util

import pytest
import torch
from torch.autograd import forward_ad

from paper_2511_02043_amd import functional as fn


def test_only_without_derivatives_transforms_and_traces():
    x, g = torch.zeros(2), torch.zeros(2, requires_grad=True)
    seen = []

    def call(*tensors):
        seen.append(fn._without_node(tensors))
        return tensors[0] * 2

    call(x, None, x)
    call(x, None, g)
    with torch.no_grad():
        call(g)
    with torch.inference_mode():
        call(x)
    assert seen == [True, False, True, True]
    del seen[:]
    torch.vmap(call)(x)
    torch.func.grad(lambda t: call(t).sum())(x)
    torch.func.jvp(call, (x,), (x,))
    with forward_ad.dual_level():
        call(forward_ad.make_dual(x, x))
        call(x)
    with torch.no_grad():
        torch.jit.trace(call, (x,), check_trace=False)
    assert not any(seen) and len(seen) == 6, seen


@pytest.mark.parametrize("owner,name", [(torch._C, "_are_functorch_transforms_active"), (torch._C, "_get_tracing_state"), (forward_ad, "_current_level")])
def test_with_a_torch_that_has_not_the_name(owner, name, monkeypatch):
    """A state that cannot be asked for is one that may be there: the module is imported, and every call gets its node."""
    monkeypatch.delattr(owner, name)
    spec = importlib.util.spec_from_file_location(fn.__name__ + "_again", fn.__file__)
    again = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(again)
    assert not again._without_node((torch.zeros(2),))
