"""When the one-launch layout kernels may stand in for torch's operations: never
while something watches the operations, and never when torch cannot say."""
import pytest
import torch
from torch.autograd import forward_ad
from torch.fx.experimental.proxy_tensor import make_fx
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2605_20150_amd import raster


class Watch(TorchDispatchMode):
    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def seen(run):
    """What _watched says of the tensor that run hands to a function."""
    got = []

    def f(t):
        got.append(raster._watched(t))
        return t + 1

    run(f)
    return got[0]


def dual(f):
    with forward_ad.dual_level():
        f(torch.zeros(3))


def mode(f):
    with Watch():
        f(torch.zeros(3))


def device(f):
    with torch.device("cpu"):
        f(torch.zeros(3))


@pytest.mark.parametrize("name,run,want", [
    ("plain", lambda f: f(torch.zeros(3)), False),
    ("default device", device, False),
    ("autograd", lambda f: f(torch.zeros(3, requires_grad=True)), True),
    ("jit.trace", lambda f: torch.jit.trace(f, torch.zeros(3)), True),
    ("make_fx", lambda f: make_fx(f)(torch.zeros(3)), True),
    ("vmap", lambda f: torch.func.vmap(f)(torch.zeros(2, 3)), True),
    ("functionalize", lambda f: torch.func.functionalize(f)(torch.zeros(3)), True),
    ("forward mode", dual, True),
    ("dispatch mode", mode, True),
    ("negation not yet done", lambda f: f(torch._neg_view(torch.zeros(3))), True),
])
def test_watched_tensors(name, run, want):
    assert seen(run) is want


@pytest.mark.parametrize("owner,attr", [(torch._C, "_functorch"), (forward_ad, "_current_level"),
                                        (torch._C, "_len_torch_dispatch_stack"), (torch.compiler, "is_compiling")])
def test_a_torch_that_cannot_say_takes_the_general_path(monkeypatch, owner, attr):
    monkeypatch.delattr(owner, attr)
    assert raster._watched(torch.zeros(3)) is True
    assert raster._plain(torch.zeros(3)) is False
