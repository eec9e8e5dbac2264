"""The binding's native marshalling refuses what its Python descriptors refuse,
with the same errors, before any call reaches the library (CPU only)."""
from __future__ import annotations

import pytest
import torch

from paper_2602_00125_amd import binding as b


@pytest.mark.parametrize("call", [
    lambda t: b.linear_fwd(t, t, None, t), lambda t: b.linear_act_fwd(t, t, None, "relu", t),
    lambda t: b.linear_bwd(t, t, t, t), lambda t: b.matmul(t, t, t), lambda t: b.reduce_broadcast_grad(t, t),
    lambda t: b.act_bwd("gelu", t, t, t), lambda t: b.mse_loss(t, t, t), lambda t: b.sgd_step([t], [t], [t], 0.1),
    lambda t: b.adam_step([t], [t], [t], [t], 0.1, 0.9, 0.999, 1e-8, 1), lambda t: b.rmsprop_step([t], [t], [t], 0.1, 0.9, 1e-8),
    lambda t: b.conv2d_fwd(t, t, None, t), lambda t: b.conv2d_bwd(t, t, t, t)])
def test_host_tensors_are_refused(call):
    with pytest.raises(ValueError, match="device tensors"):
        call(torch.zeros(2, 2))
    with pytest.raises(AttributeError):
        call(3)


def test_lists_of_different_lengths_are_refused():
    with pytest.raises(AssertionError):
        b.sgd_step([], [torch.zeros(1)], [], 0.1)


def test_missing_descriptors_are_the_library_s_error():
    with pytest.raises(b.MtError) as e:
        b.linear_fwd(None, None, None, None, stream=0)
    assert e.value.name == "MT_ERR_NULL"


class _Made:
    """A tensor to the marshalling, with no memory behind it."""
    is_cuda, dtype, shape = True, torch.float32, (4,)
    live = 0

    def __init__(self):
        _Made.live += 1

    def __del__(self):
        _Made.live -= 1

    def stride(self):
        return (1,)

    def data_ptr(self):
        _Made.seen = max(_Made.seen, _Made.live)
        return 4096 * _Made.live


class _Makes:
    """A list whose tensors are made as it is read."""

    def __len__(self):
        return 2

    def __iter__(self):
        return (_Made() for _ in range(2))


def test_tensors_of_lists_are_held_until_the_call_returns():
    _Made.seen = 0
    with pytest.raises(b.MtError, match="step counts from 1"):  # refused before any memory is touched
        b.adam_step(_Makes(), _Makes(), _Makes(), _Makes(), 0.1, 0.9, 0.999, 1e-8, 0, stream=0)
    assert _Made.seen == 8 and _Made.live == 0


@pytest.mark.parametrize("call", [
    lambda t: b.sgd_step(t(), [], [], 0.1, stream=0), lambda t: b.adam_step([], t(), [], [], 0.1, 0.9, 0.999, 1e-8, 1, stream=0),
    lambda t: b.rmsprop_step([], [], t(), 0.1, 0.9, 1e-8, stream=0)])
def test_generators_are_refused(call):
    with pytest.raises(TypeError):
        call(lambda: (x for x in []))
