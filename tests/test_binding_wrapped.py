"""The native call path and tensors whose memory cannot be taken: inside
torch.vmap and torch.func.grad an argument is an exact torch.Tensor on the
device, but without storage. The call has to raise, as the Python path does.

Fake device tensors stand in for the GPU's, so that no kernel can run."""

import types

import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

from paper_2607_27744_amd import ops

BF, I32 = torch.bfloat16, torch.int32
STREAM = types.SimpleNamespace(cuda_stream=0)
WS = ((1 << 20,), torch.uint8)
REQ = dict(x_req=((2, 40), BF), w_req=((48, 40), BF), out=((20, 48), BF), workspace=WS)
LINEAR = dict(x_cand=((20, 64), BF), w_cand=((48, 64), BF), **REQ)
LCB = dict(x_req=((2, 20, 64), BF), x_cand=((20, 16, 64), BF), w_cr=((32, 20), BF),
           w_cc=((32, 16), BF), y_cand=((20, 32, 64), BF), workspace=WS)
QKV = dict(q=((20, 1, 2, 64), BF), k=((40, 2, 64), BF), v=((40, 2, 64), BF),
           kv_offsets=((3,), I32), out=((20, 1, 2, 64), BF))
OFF, IDS = dict(cand_offsets=((3,), I32)), dict(cand_request_ids=((20,), I32))

# operator, its tensors (every buffer given), its other arguments
CALLS = {
    "linear": (ops.ikbo_linear, {**LINEAR, **OFF}, {}),
    "linear mapped": (ops.ikbo_linear_mapped, {**LINEAR, **IDS}, {}),
    "glm": (ops.glm_linear, dict(x_req=((2, 40), BF), x_cand=((20, 64), BF), w_rr=((24, 40), BF),
                                 w_cr=((48, 40), BF), w_cc=((48, 64), BF), y_req=((2, 24), BF),
                                 y_cand=((20, 48), BF), workspace=WS, **OFF), {}),
    "mlp2": (ops.ikbo_mlp2, dict(x_cand=((20, 128), BF), w1_cand=((64, 128), BF),
                                 w2=((128, 64), BF), x_req=((2, 40), BF), w1_req=((64, 40), BF),
                                 out=((20, 128), BF), workspace=WS, **OFF), {}),
    "fm": (ops.glm_fm_linear, dict(x_req=((2, 32, 128), BF), x_cand=((20, 8, 128), BF),
                                   w_req=((64, 1024), BF), w_cand=((64, 320), BF),
                                   out=((20, 64), BF), workspace=WS, **OFF), {}),
    "lcb": (ops.ikbo_lcb, {**LCB, **OFF}, {}),
    "lcb mapped": (ops.ikbo_lcb_mapped, {**LCB, **IDS}, {}),
    "plan": (ops.dca_attention_plan, dict(kv_offsets=((3,), I32), plan=WS, **OFF),
             dict(num_cand=20, heads=2)),
    "attention": (ops.dca_attention, {**QKV, **OFF}, {}),
    "attention mapped": (ops.dca_attention_mapped, {**QKV, **IDS, "workspace": WS}, {}),
    "attention residual": (ops.dca_attention_residual,
                           {**QKV, **OFF, "residual": QKV["q"], "out_sum": QKV["q"]}, {}),
    "attention ex": (ops.dca_attention_ex, {**QKV, **OFF, "plan": WS}, {}),
}


@pytest.mark.parametrize("transform,name", [(t, n) for t in ("vmap", "grad") for n in sorted(CALLS)
                                            if (t, n) != ("grad", "plan")])   # offsets only
def test_raises(transform, name):
    fn, tensors, other = CALLS[name]

    def call(*ts):
        return fn(**dict(zip(tensors, ts)), **other, stream=STREAM)

    with FakeTensorMode():
        ts = [torch.empty(s, dtype=d, device="cuda") for s, d in tensors.values()]
        with pytest.raises(RuntimeError, match="data pointer"):
            if transform == "vmap":
                torch.vmap(call)(*[torch.stack([t, t]) for t in ts])
            else:
                first = next(i for i, t in enumerate(ts) if t.is_floating_point())
                torch.func.grad(call, argnums=first)(*ts)
