"""GPU: the native call path and the Python one take the same calls, give the
same values and raise the same errors."""

from types import SimpleNamespace

import pytest
import torch

from paper_2607_27744_amd import ops

pytestmark = pytest.mark.gpu

BF = torch.bfloat16
PYTHON = SimpleNamespace(**{n: (lambda *a: None) for n in (
    "linear", "glm_linear", "mlp2", "fm_linear", "lcb", "plan", "attention")})


def _r(*shape, dtype=BF):
    return torch.randn(shape, device="cuda").to(dtype)


def _off(*counts):
    return torch.tensor([sum(counts[:i]) for i in range(len(counts) + 1)], dtype=torch.int32,
                        device="cuda")


def _ids(n, r):
    return (torch.arange(n, device="cuda") % r).to(torch.int32)


def _kv(h, d, n=40):
    kv = _r(n, 2 * h * d)
    return kv[:, :h * d].view(n, h, d), kv[:, h * d:].view(n, h, d)


def _calls():
    co, ko = _off(20, 0, 17), _off(10, 5, 25)
    k, v = _kv(2, 64)
    k2, v2 = _kv(4, 64)
    q = _r(37, 2, 2, 64)
    lin = dict(x_cand=_r(37, 64), w_cand=_r(48, 64), x_req=_r(3, 40), w_req=_r(48, 40),
               bias=_r(48, dtype=torch.float32), activation="relu")
    return {
        "linear": (ops.ikbo_linear, dict(lin, cand_offsets=co)),
        "linear plain": (ops.ikbo_linear, dict(x_cand=_r(5, 64), w_cand=_r(48, 64))),
        "linear f32": (ops.ikbo_linear, dict(x_cand=_r(5, 3, dtype=torch.float32),
                                             w_cand=_r(7, 3, dtype=torch.float32))),
        "linear add": (ops.ikbo_linear, dict(lin, cand_offsets=co, x_cand_add=_r(37, 64))),
        "mapped": (ops.ikbo_linear_mapped, dict(lin, cand_request_ids=_ids(37, 3))),
        "glm": (ops.glm_linear, dict(x_req=_r(3, 40), x_cand=_r(37, 64), w_rr=_r(24, 40),
                                     w_cr=_r(48, 40), w_cc=_r(48, 64), cand_offsets=co,
                                     b_req=_r(24, dtype=torch.float32))),
        "mlp2": (ops.ikbo_mlp2, dict(x_cand=_r(37, 128), w1_cand=_r(64, 128), w2=_r(128, 64),
                                     x_req=_r(3, 40), w1_req=_r(64, 40), cand_offsets=co,
                                     b2=_r(128, dtype=torch.float32))),
        "fm": (ops.glm_fm_linear, dict(x_req=_r(3, 32, 128), x_cand=_r(37, 8, 128),
                                       cand_offsets=co, w_req=_r(64, 1024), w_cand=_r(64, 320))),
        "lcb": (ops.ikbo_lcb, dict(x_req=_r(3, 20, 64), x_cand=_r(37, 16, 64), w_cr=_r(32, 20),
                                   w_cc=_r(32, 16), cand_offsets=co, w_rr=_r(8, 20))),
        "lcb mapped": (ops.ikbo_lcb_mapped, dict(x_req=_r(3, 20, 64), x_cand=_r(37, 16, 64),
                                                 w_cr=_r(32, 20), w_cc=_r(32, 16),
                                                 cand_request_ids=_ids(37, 3))),
        "plan": (ops.dca_attention_plan, dict(cand_offsets=co, kv_offsets=ko, num_cand=37,
                                              heads=2)),
        "attention": (ops.dca_attention, dict(q=q, k=k, v=v, cand_offsets=co, kv_offsets=ko)),
        "attention scale": (ops.dca_attention, dict(q=q, k=k, v=v, cand_offsets=co, kv_offsets=ko,
                                                    scale=1)),
        "attention residual": (ops.dca_attention_residual,
                               dict(q=q, k=k, v=v, cand_offsets=co, kv_offsets=ko, residual=q)),
        "attention mapped": (ops.dca_attention_mapped,
                             dict(q=q, k=k, v=v, cand_request_ids=_ids(37, 3), kv_offsets=ko)),
        "attention request": (ops.dca_request_attention, dict(q_req=_r(3, 2, 2, 64), k=k, v=v,
                                                              kv_offsets=ko)),
        "attention ex": (ops.dca_attention_ex, dict(q=q, k=k, v=v, cand_offsets=co,
                                                    kv_offsets=ko)),
        "proj": (ops.dca_attention_proj, dict(x=_r(37, 1, 256), w_q=_r(256, 256), k=k2, v=v2,
                                              cand_offsets=co, kv_offsets=ko, heads=4,
                                              residual=_r(37, 1, 4, 64))),
    }


def _outcome(fn, kw):
    try:
        out = fn(**kw)
    except Exception as e:
        return type(e), str(e)
    torch.cuda.synchronize()
    out = out if isinstance(out, tuple) else (out,)
    return [None if t is None else t.cpu() for t in out]


def _same(a, b):
    if isinstance(a, tuple) or isinstance(b, tuple):
        return a == b
    return len(a) == len(b) and all(
        (x is None and y is None) or (x.dtype == y.dtype and torch.equal(x, y))
        for x, y in zip(a, b))


def _spoiled(value, name=""):
    """Wrong, or merely unusual, forms of one argument. Never another number of
    candidates: the offsets, trusted device data, would not fit it."""
    if value is None:
        return
    yield None
    if torch.is_tensor(value):
        yield value.cpu()
        yield value.float() if value.dtype == BF else value.to(torch.float64)
        if name not in ("x_cand", "x", "q"):
            if value.dim() > 1:
                yield value[:-1]
            yield torch.cat([value, value])
        if value.dim() == 2:
            yield value.t().contiguous().t()
        yield torch.stack([value, value], -1)[..., 0]           # strided
        yield torch.nn.Parameter(value) if value.is_floating_point() else value.clone()
        yield "text"
    elif isinstance(value, str):
        yield "gelu"
    else:
        yield "text"


class _Spy:
    """The native module, noting whether the last call was taken there."""

    def __init__(self, module):
        self.module, self.taken = module, None

    def __getattr__(self, name):
        def call(*args):
            done = getattr(self.module, name)(*args)
            self.taken = done is not None
            return done
        return call


# Valid calls that the native path leaves to ops.py: weights or offsets of a
# request term that is not there.
LEFT = {("linear", "x_req"), ("linear add", "x_req"), ("mapped", "x_req"), ("mlp2", "x_req")}


@pytest.mark.parametrize("name", sorted(_calls() if torch.cuda.is_available() else ["none"]))
def test_same_as_the_python_path(gpu_lib, name, monkeypatch):
    torch.manual_seed(0)
    fn, kw = _calls()[name]
    native = _Spy(ops._native())
    cases = [("", kw)]
    for key, value in kw.items():
        cases += [(key, dict(kw, **{key: v})) for v in _spoiled(value, key)]
    if name != "plan":
        first = fn(**kw)
        outs = first if isinstance(first, tuple) else (first,)
        key = {"glm": "y_cand", "lcb": "y_cand", "lcb mapped": "y_cand"}.get(name, "out")
        given = outs[1] if key == "y_cand" else outs[0]
        cases += [(key, dict(kw, **{key: v})) for v in [torch.empty_like(given), *_spoiled(given)]]
    cases.append(("stream", dict(kw, stream=torch.cuda.current_stream())))
    valid = 0
    for key, case in cases:
        monkeypatch.setattr(ops, "_binding", native)
        native.taken = None
        a = _outcome(fn, case)
        monkeypatch.setattr(ops, "_binding", PYTHON)
        b = _outcome(fn, case)
        assert _same(a, b), (name, {k: (tuple(v.shape), v.dtype, str(v.device)) if torch.is_tensor(v)
                                    else v for k, v in case.items()}, a, b)
        if isinstance(a, tuple):                # an error, the same on both paths
            assert key and not native.taken
            continue
        valid += 1
        assert bool(native.taken) != ((name, key) in LEFT and case[key] is None), (name, key)
    assert valid > 2
    monkeypatch.setattr(ops, "_binding", native)
    if "out" in kw or name in ("linear", "attention"):
        out = torch.empty_like(fn(**kw))
        assert fn(**dict(kw, out=out)) is out
