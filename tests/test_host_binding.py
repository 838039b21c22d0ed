"""The binding's helpers that need no GPU."""
import warnings

import pytest
import torch

import paper_2407_16847_amd as splat


def _named(x):
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")   # named tensors are a prototype feature
        return x.refine_names("B", "H", "L", "d")


@pytest.mark.parametrize("make", [
    lambda x: x, _named, lambda x: torch.nn.Parameter(x), lambda x: torch._neg_view(x),
    lambda x: x.as_strided(x.shape, (7, 60, 5, 1))], ids=["plain", "named", "parameter", "neg", "strides"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_an_output_made_by_a_call_is_plain(make, dtype):
    """Of its input an output takes shape and device only."""
    ref = make(torch.zeros(1, 3, 12, 5))
    out = splat._new(ref, dtype)
    assert type(out) is torch.Tensor and out.dtype == dtype and not out.requires_grad
    assert out.names == (None,) * 4 and not out.is_neg()
    assert out.shape == (1, 3, 12, 5) and out.stride() == (180, 60, 5, 1)
