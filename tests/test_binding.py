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


class OnAccess:
    """A sequence that makes its problems when they are read and keeps none of them."""

    def __init__(self, n, make):
        self.n, self.make = n, make

    def __len__(self):
        return self.n

    def __getitem__(self, i):
        if i >= self.n:
            raise IndexError
        return self.make(i)


def test_problems_live_until_the_call_returns():
    """A problem that only the call refers to is released when the library is done with its pointers, not
    before: the last of 8000 problems (whose grouping takes the library most of the call) goes at the end."""
    import time
    import weakref
    big = dict(FULL, A=torch.zeros(64, 8), B=torch.zeros(8, 64), x=torch.zeros(4, 8))
    seen = {}

    class Problem(dict):
        pass

    def make(i):
        p = Problem(big)
        if i == 7999:
            seen["read"] = time.perf_counter()
            weakref.finalize(p, lambda: seen.setdefault("released", time.perf_counter()))
        return p

    attt.lora_workspace_size(OnAccess(8000, make), attt.BF16)
    done = time.perf_counter()
    assert done - seen["released"] < 0.5 * (done - seen["read"])


@pytest.mark.parametrize("call", [lambda p: attt.lora_workspace_size(p, attt.BF16), attt.lora_grad, attt.lora_forward,
                                  lambda p: attt.lora_sgd_step(p, 0.1), attt.lora_hot_swap])
def test_a_generator_has_no_length(call):
    with pytest.raises(TypeError):
        call(FULL for _ in range(1))


def test_other_threads_run_during_a_call():
    """8000 problems of their own: the library plans them for longer than the marshalling takes, and a
    second Python thread gets to run meanwhile."""
    import threading
    import time
    big = dict(FULL, A=torch.zeros(64, 8), B=torch.zeros(8, 64))
    problems, ticks, stop = [big] * 8000, [], threading.Event()

    def tick():
        while not stop.is_set():
            ticks.append(time.perf_counter())
            time.sleep(0.001)

    t = threading.Thread(target=tick)
    t.start()
    while len(ticks) < 5:
        time.sleep(0.001)
    begin = time.perf_counter()
    attt.lora_workspace_size(problems, attt.BF16)
    end = time.perf_counter()
    stop.set()
    t.join()
    at = [begin] + [x for x in ticks if begin < x < end] + [end]
    assert max(b - a for a, b in zip(at, at[1:])) < 0.5 * (end - begin)


def test_numbers_as_float_takes_them():
    """scale is what float() makes of it, and nothing but problems is nothing to do."""
    import numpy as np
    want = attt.lora_workspace_size([FULL], attt.BF16)
    for scale in ("2.0", " 1e-3 ", np.float32(2), np.array(0.5), torch.tensor(2.0), True):
        assert attt.lora_workspace_size([dict(FULL, scale=scale)], attt.BF16) == want
    for bad in ("two", None, [1.0]):
        with pytest.raises(TypeError):
            attt.lora_workspace_size([dict(FULL, scale=bad)], attt.BF16)
    with pytest.raises(attt.AtttError):
        attt.lora_workspace_size([dict(FULL, scale="inf")], attt.BF16)
    with pytest.raises(ValueError):                                       # the device, not the number
        attt.lora_sgd_step([dict(param=X, grad=X)], "0.1")
    for nothing in (None, (), []):
        assert attt.lora_grad(nothing) is None
