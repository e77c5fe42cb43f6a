"""What the library's stand-ins for torch operations must leave to torch: every
state in which something sees those operations one by one."""
import pytest
import torch
from torch.overrides import TorchFunctionMode
from torch.utils._python_dispatch import TorchDispatchMode

from paper_1803_03949_amd.binding import torch_is_watched


class Functions(TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


class Dispatch(TorchDispatchMode):
    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def plain(f):
    f(torch.zeros(2))


def under_trace(f):
    torch.jit.trace(f, (torch.zeros(2),), check_trace=False)


def under_functions(f):
    with Functions():
        f(torch.zeros(2))


def under_functions_and_device(f):
    with Functions(), torch.device("cpu"):
        f(torch.zeros(2))


def under_device(f):
    with torch.device("cpu"):
        f(torch.zeros(2))


def under_dispatch(f):
    with Dispatch():
        f(torch.zeros(2))


def under_forward_mode(f):
    with torch.autograd.forward_ad.dual_level():
        f(torch.zeros(2))


def under_vmap(f):
    torch.func.vmap(f)(torch.zeros(3, 2))


def under_func_grad(f):
    torch.func.grad(lambda x: f(x).sum())(torch.zeros(2))


def under_functionalize(f):
    torch.func.functionalize(f)(torch.zeros(2))


@pytest.mark.parametrize("call,watched", [
    (under_vmap, True), (under_func_grad, True), (under_functionalize, True),
    (plain, False), (under_device, False), (under_trace, True), (under_functions, True),
    (under_functions_and_device, True), (under_dispatch, True), (under_forward_mode, True)])
def test_every_watcher_is_seen(call, watched):
    seen = []

    def f(x):
        seen.append(torch_is_watched())
        return x + 1

    call(f)
    assert seen == [watched]
    assert not torch_is_watched()
