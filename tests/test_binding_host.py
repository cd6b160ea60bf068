"""The binding's argument marshalling without a GPU: every call here is refused before anything is launched."""

import types

import numpy as np
import pytest
import torch

from paper_2105_09377_amd import binding as gs


def refused(status, call, *args, **kw):
    with pytest.raises(gs.GlensideError) as e:
        call(*args, **kw)
    assert e.value.status == status


@pytest.mark.parametrize("n0,n1", [(-1, -1), (-1, 1), (1, -2), (3, 1)])
def test_cartesian_dot_access_splits_that_do_not_exist(n0, n1):
    a = torch.zeros((4, 8), dtype=torch.bfloat16)
    # results of the shapes that "-1: all of them" would have
    lead = {1: (4,), -1: (4, 8), -2: (4, 8), 3: (4, 8)}
    out = torch.zeros(lead[n0] + lead[n1], dtype=torch.float32)
    refused(gs.GS_ERR_RANK, gs.cartesian_dot, a, a, n0, n1, out=out)
    refused(gs.GS_ERR_RANK, gs.cartesian_dot, a, a, n0, n1)


def long_name():
    """A name that no constant of this module holds."""
    return "".join(["activations", "_of_a_name", "_that_nothing_else_holds"])


class Changing:
    """An integer whose conversion empties the dict of tensors, as another thread might."""

    def __init__(self, tensors):
        self.tensors = tensors

    def __int__(self):
        self.tensors.clear()
        self.held = ["y" * len(long_name()) for _ in range(1000)]     # where the freed name was
        return 3


def test_program_eval_holds_what_it_was_given():
    tensors = {long_name(): torch.zeros((5, 4), dtype=torch.int8)}
    text = f"(pad {long_name()} 0 A A)"
    out = torch.zeros((11, 4), dtype=torch.int32)
    # the name is found and the result's shape follows from the tensor: only its type is wrong
    refused(gs.GS_ERR_DTYPE, gs.program_eval, text, tensors, {"A": Changing(tensors)}, out=out)
    assert tensors == {}


@pytest.mark.parametrize("shape", [(10, 4), (11, 3), (0,), ()])
def test_program_eval_into_a_result_that_is_too_short(shape):
    x = torch.zeros((5, 4), dtype=torch.int8)
    refused(gs.GS_ERR_SHAPE, gs.program_eval, "(pad x 0 A A)", {"x": x}, {"A": 3}, out=torch.zeros(shape, dtype=torch.int8))


def test_program_eval_into_a_result_of_another_shape():
    """The same elements in another shape pass that check (the type is what is refused here)."""
    x = torch.zeros((5, 4), dtype=torch.int8)
    refused(gs.GS_ERR_DTYPE, gs.program_eval, "(pad x 0 A A)", {"x": x}, {"A": 3}, out=torch.zeros((44,), dtype=torch.int32))


@pytest.mark.parametrize("mapping", [dict, types.MappingProxyType])
def test_program_eval_takes_any_mapping(mapping):
    x = torch.zeros((5, 4), dtype=torch.int8)
    refused(gs.GS_ERR_DTYPE, gs.program_eval, "(pad x 0 A A)", mapping({"x": x}), mapping({"A": 3}), out=torch.zeros((11, 4), dtype=torch.int32))


@pytest.mark.parametrize("not_a_mapping", [[("x", 1)], ["x"], 5])
def test_program_eval_takes_nothing_else(not_a_mapping):
    with pytest.raises((TypeError, AttributeError)):
        gs.program_eval("(pad x 0 1 1)", not_a_mapping, {})


def test_operators_and_activations_are_integers():
    x = torch.zeros((4, 8), dtype=torch.bfloat16)
    y = torch.zeros((1, 2, 6, 6), dtype=torch.bfloat16)
    w = torch.zeros((2, 2, 3, 3), dtype=torch.bfloat16)
    for call in (lambda c: gs.cartesian_dot(x, x, act=c), lambda c: gs.reduce(x, 1, c), lambda c: gs.conv2d_direct(y, w, act=c),
                 lambda c: gs.pair_reduce(x, x, c), lambda c: gs.windows_reduce(y, 2, (2, 2), (2, 2), op=c),
                 lambda c: gs.access_windows(y, 2, (2, 2), (2, 2), pad_mode=c), lambda c: gs.depthwise_conv2d(y, w[0], act=c)):
        for wrong in (1.0, "1", None):
            with pytest.raises(TypeError):
                call(wrong)
        refused(gs.GS_ERR_UNSUPPORTED, call, np.int64(77))


def test_sequences_of_integers_are_sized():
    y = torch.zeros((1, 2, 6, 6), dtype=torch.bfloat16)
    with pytest.raises(TypeError):
        gs.windows_reduce(y, 2, (i for i in (2, 2)), (2, 2))
    # what is sized is taken: the operator is what is refused
    for window in ([2, 2], torch.Size((2, 2)), np.array([2, 2]), torch.tensor([2, 2]), range(2, 4)):
        refused(gs.GS_ERR_UNSUPPORTED, gs.windows_reduce, y, 2, window, (2, 2), op=77)


def test_the_stack_names_every_layer():
    """Projections too, which are computed by the calls of the convolutions beside them."""
    from paper_2105_09377_amd.resnet import ResNet18Stack
    from paper_2105_09377_amd.synth import RESNET18_CONVS
    net = object.__new__(ResNet18Stack)
    net.spec = {name: rest for name, *rest in RESNET18_CONVS}
    names = net.layer_calls()
    assert names[:2] == ["conv1", "pool"] and names[-2:] == ["avg", "fc"]
    assert sorted(names[2:-2]) == sorted(n for n in net.spec if n != "conv1")
