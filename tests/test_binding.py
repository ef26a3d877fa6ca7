"""What the native marshalling of the list calls refuses, and how, without a GPU."""
import os

import pytest
import torch

import paper_2607_03441_amd as attt

X = torch.zeros(4, 8)
FULL = dict(x=X, dy=X, y=X, A=X, B=X, dA=X, dB=X, scale=1)


class Mapping:
    """Not a dict: hands out a new object at every access."""

    def __init__(self, d):
        self.d = d

    def __getitem__(self, k):
        v = self.d[k]
        return v.clone() if isinstance(v, torch.Tensor) else v


@pytest.fixture(autouse=True)
def built():
    if not os.path.exists(attt.lib_path()):
        pytest.fail("libattt.so is not built; run __graft_entry__.build()")


@pytest.mark.parametrize("call,error", [
    (lambda: attt.lora_forward([FULL]), ValueError),                       # not on a device
    (lambda: attt.lora_grad([FULL]), ValueError),
    (lambda: attt.lora_hot_swap([(X, X)]), ValueError),
    (lambda: attt.lora_sgd_step([dict(param=X, grad=X)], 0.1), ValueError),
    (lambda: attt.lora_grad([{}]), KeyError),
    (lambda: attt.lora_hot_swap([(X,)]), ValueError),
    (lambda: attt.lora_workspace_size([dict(FULL, x=3)], attt.BF16), TypeError),
    (lambda: attt.lora_workspace_size([dict(FULL, x=X[0])], attt.BF16), IndexError),
    (lambda: attt.lora_workspace_size([dict(FULL, scale="s")], attt.BF16), TypeError),
    (lambda: attt.lora_workspace_size([FULL], 7), attt.AtttError),
    (lambda: attt.lora_workspace_size(None, attt.BF16), TypeError)])
def test_refused(call, error):
    with pytest.raises(error):
        call()


def test_any_mapping_and_no_problems():
    want = attt.lora_workspace_size([FULL], attt.BF16)
    assert attt.lora_workspace_size((Mapping(FULL),), attt.BF16) == want > 256
    assert attt.lora_workspace_size([], attt.BF16) == 256
    assert attt.lora_grad([]) is None
