"""Addresses that the binding passes on (no GPU): tensors, arrays and raw addresses, none of them through a raised exception."""
import sys

import numpy as np
import pytest
import torch

from paper_2007_12216_amd import binding

TENSOR, ARRAY = torch.zeros(4, dtype=torch.int8), np.zeros(4, dtype=np.int8)


@pytest.mark.parametrize("obj,address", [(TENSOR, TENSOR.data_ptr()), (ARRAY, ARRAY.ctypes.data), (0, 0), (1 << 46, 1 << 46)],
                         ids=["tensor", "array", "null", "raw"])
def test_addresses_are_found_without_an_exception(obj, address):
    raised = []

    def trace(frame, event, arg):
        if event == "exception":
            raised.append(arg)
        return trace

    before = sys.gettrace()
    sys.settrace(trace)
    try:
        got = binding._ptr(obj)
    finally:
        sys.settrace(before)
    assert got == address and not raised


def test_subclasses_are_taken_too():
    class Address(int):
        pass

    class Array(np.ndarray):
        pass

    assert binding._ptr(Address(12)) == 12 and binding._ptr(True) == 1
    assert binding._ptr(ARRAY.view(Array)) == ARRAY.ctypes.data
    assert binding._ptr(torch.nn.Parameter(TENSOR, requires_grad=False)) == TENSOR.data_ptr()


@pytest.mark.parametrize("kinds", ["tttt", "aaaa", "iiii", "tiii", "ittt", "taia"])
def test_the_calls_take_any_mixture_of_addresses(kinds, monkeypatch):
    make = {"t": lambda k: (t := torch.zeros(4 + k), t.data_ptr()), "a": lambda k: (a := np.zeros(4 + k), a.ctypes.data), "i": lambda k: (4096 + k, 4096 + k)}
    given, want = zip(*(make[kind](k) for k, kind in enumerate(kinds)))
    seen = []

    class Library:
        def rnswino_conv2d(self, *args):
            seen.append(args)
            return 0

        rnswino_conv2d_requant = rnswino_conv2d

    monkeypatch.setattr(binding, "_lib", Library())
    plan = type("Plan", (), {"handle": 7})()
    binding.rnswino_conv2d(plan, *given, 9)
    binding.rnswino_conv2d_requant(plan, *given[:3], 5, True, given[3], 9)
    assert seen == [(7, *want, 9), (7, *want[:3], 5, 1, want[3], 9)]
