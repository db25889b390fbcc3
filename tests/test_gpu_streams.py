"""GPU: calls on another stream than the current one. The memory that a call
takes by itself has to follow the order of the stream that uses it: a workspace
of the current stream's would be handed to that stream's next allocation while
the call's kernels still use it."""

import pytest
import torch

from paper_2607_27744_amd import ops
from test_gpu_binding import _calls

pytestmark = pytest.mark.gpu

NAMES = sorted(_calls()) if torch.cuda.is_available() else ["none"]


def _segments(stream):
    return [s for s in torch.cuda.memory_snapshot() if s["stream"] == stream.cuda_stream]


def _tensors(out):
    return list(out) if isinstance(out, tuple) else [out]


@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("given", [False, True], ids=["all new", "outputs given"])
def test_memory_of_the_calls_stream(gpu_lib, name, given):
    torch.manual_seed(0)
    fn, kw = _calls()[name]
    want = _tensors(fn(**kw))
    if given:
        keys = {"glm": ["y_req", "y_cand"], "lcb": ["y_req", "y_cand"],
                "lcb mapped": [None, "y_cand"], "plan": ["plan"]}.get(name, ["out", "out_sum"])
        kw = dict(kw, **{k: torch.empty_like(t) for k, t in zip(keys, want) if t is not None})
    side, cur = torch.cuda.Stream(), torch.cuda.current_stream()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    assert not _segments(side)
    scratch = name in ("linear", "linear add", "mapped", "glm", "mlp2", "fm", "lcb", "lcb mapped",
                       "attention mapped")
    side.wait_stream(cur)
    got = _tensors(fn(**kw, stream=side))
    assert bool(_segments(side)) == (scratch or not given)
    cur.wait_stream(side)
    if name == "plan":                          # past its last word nothing is written
        got, want = ([t[:4 * (8 + 2 * 3 + 1)] for t in ts] for ts in (got, want))
    for a, b in zip(got, want):
        assert a is None and b is None or torch.equal(a, b)


def test_output_freed_on_the_current_stream(gpu_lib):
    # An output that work on the current stream still reads is not handed to
    # the call's stream again.
    x, w = (torch.randn(512, 64, device="cuda").bfloat16() for _ in range(2))
    side, cur = torch.cuda.Stream(), torch.cuda.current_stream()
    side.wait_stream(cur)
    y = ops.ikbo_linear(x, w, stream=side)
    cur.wait_stream(side)
    torch.cuda._sleep(200_000_000)              # about 0.1 s of work that could read y
    at = y.data_ptr()
    del y
    with torch.cuda.stream(side):
        again = torch.empty(512, 512, dtype=torch.bfloat16, device="cuda")
    assert not cur.query() and again.data_ptr() != at
    torch.cuda.synchronize()


def test_identity_offsets_first_needed_under_capture(gpu_lib, monkeypatch):
    # Request-side attention builds its offsets on first use. A graph's own
    # memory, unwritten before its first replay, must not serve eager calls.
    monkeypatch.setattr(ops, "_IDENTITY", {})
    monkeypatch.setattr(ops, "_IDENTITY_VIEWS", {})
    kw = _calls()["attention request"][1]
    n = kw["q_req"].shape[0]
    offsets = dict(cand_offsets=torch.arange(n + 1, dtype=torch.int32, device="cuda"))
    want = ops.dca_attention(kw["q_req"], kw["k"], kw["v"], **offsets, kv_offsets=kw["kv_offsets"])
    out = torch.empty_like(want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ops.dca_request_attention(**kw, out=out)
    assert not ops._IDENTITY and not ops._IDENTITY_VIEWS
    for _ in range(3):
        assert torch.equal(ops.dca_request_attention(**kw), want)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
