"""Precision and form arguments: every value that equals an accepted one is
accepted, hashable alike or not."""
import enum

import numpy as np
import pytest
import torch

import paper_1808_01517_amd as dl
from paper_1808_01517_amd import _lib


class Unhashable:
    __hash__ = None

    def __init__(self, value):
        self.value = value

    def __eq__(self, other):
        return other == self.value


class Mode(str, enum.Enum):
    HALF = "bf16"


@pytest.mark.parametrize("value,code", [
    (None, _lib.DLM_FP32), ("fp32", _lib.DLM_FP32), ("f32", _lib.DLM_FP32), (torch.float32, _lib.DLM_FP32),
    ("bf16", _lib.DLM_BF16), (torch.bfloat16, _lib.DLM_BF16), (np.int64(_lib.DLM_BF16), _lib.DLM_BF16),
    (torch.tensor(_lib.DLM_FP32), _lib.DLM_FP32), (torch.tensor(_lib.DLM_BF16), _lib.DLM_BF16),
    (np.array([_lib.DLM_BF16]), _lib.DLM_BF16), (Unhashable("bf16"), _lib.DLM_BF16), (Mode.HALF, _lib.DLM_BF16),
])
def test_precisions(value, code):
    assert dl.precision_code(value) == code


@pytest.mark.parametrize("value,code", [
    (None, _lib.DLM_LSC_FOLDED), ("folded", _lib.DLM_LSC_FOLDED), ("resample", _lib.DLM_LSC_RESAMPLE),
    (torch.tensor(_lib.DLM_LSC_FOLDED), _lib.DLM_LSC_FOLDED), (Unhashable("resample"), _lib.DLM_LSC_RESAMPLE),
])
def test_forms(value, code):
    assert dl.form_code(value) == code


@pytest.mark.parametrize("value", ["fp16", 7, [], {}, (), torch.float16, torch.tensor(9)])
def test_others_are_refused(value):
    with pytest.raises(ValueError):
        dl.precision_code(value)
    with pytest.raises(ValueError):
        dl.form_code(value)
