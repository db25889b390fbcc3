"""Without the _binding module every operator runs its Python path."""

import sys

import pytest
import torch

import paper_2607_27744_amd as pkg
from paper_2607_27744_amd import ops

BF = torch.bfloat16


@pytest.fixture
def absent(monkeypatch):
    monkeypatch.setattr(ops, "_binding", None)
    monkeypatch.delattr(pkg, "_binding", raising=False)
    monkeypatch.setitem(sys.modules, pkg.__name__ + "._binding", None)   # import raises


def _linear(dev):
    x, w = (torch.linspace(-1, 1, 512).view(8, 64).to(dev, BF) for _ in range(2))
    return ops.ikbo_linear(x, w)


def test_the_python_path_checks(absent):
    with pytest.warns(RuntimeWarning, match="native call path"):
        with pytest.raises(ValueError, match="on the GPU"):
            _linear("cpu")
    for call in (lambda t: ops.ikbo_mlp2(t, t, t), lambda t: ops.dca_attention(t, t, t, t, t),
                 lambda t: ops.glm_linear(t, t, t, t, t, t),
                 lambda t: ops.ikbo_lcb(t, t, t, t, t),
                 lambda t: ops.glm_fm_linear(t, t, t, t, t),
                 lambda t: ops.dca_attention_plan(t.int(), t.int(), num_cand=1, heads=1),
                 lambda t: ops.dca_attention_ex(t, t, t, t, t)):
        with pytest.raises((ValueError, TypeError)):
            call(torch.zeros(2, 2))


@pytest.mark.gpu
def test_the_python_path_runs(gpu_lib, monkeypatch, request):
    want = _linear("cuda")
    request.getfixturevalue("absent")
    with pytest.warns(RuntimeWarning, match="native call path"):
        got = _linear("cuda")
    assert torch.equal(got, want)
