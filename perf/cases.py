"""The work that a serving program has librocs do, as measurable cases.

A case names one of eight kinds of call (`kind`) and its sizes. Every kind runs
through the public entry points of `paper_2607_27744_amd` with the buffers that
a serving loop keeps (outputs, workspaces, the per-batch tile plan's memory),
on seeded inputs of the shapes and distributions of `workloads.py`: N(0, 1)
activations, weights of standard deviation 1/sqrt(fan-in), ragged candidate
counts and histories. `total` sizes (candidates, history rows) belong to the
case; how they fall on the requests comes from the seed.

  block      a small fp32 ROCS block: IKBO linear and one DCA attention
  rank       ranking: two stacked DCA layers with fused query projections over
             one stacked K/V projection of the shared history
  mlp        retrieval: the two-layer IKBO MLP
  fm         GLM FM interaction feeding an IKBO linear
  lcb        IKBO linear compression block, both groups' outputs
  linear     one IKBO linear layer (CSR offsets or a per-candidate map, with or
             without a pointwise residual input)
  attention  one DCA attention over given queries and K/V
  layer      one full DCA layer: query generator, K/V projections, request- and
             candidate-side attention
"""

import math

import numpy as np
import torch

from paper_2607_27744_amd import ops, pipelines, workloads

DEV = "cuda"
BF16 = torch.bfloat16


def listed():
    return [
        # One small fp32 batch, the smallest block of the framework: latency.
        {"name": "block_fp32_small", "kind": "block", "requests": 4, "cands": 256, "k_req": 256,
         "k_cand": 128, "d_out": 256, "history": 128, "heads": 2, "dim": 32},
        # A single online ranking request: a few hundred candidates, one history.
        {"name": "rank_one_request", "kind": "rank", "requests": 1, "cands": 203, "history": 613},
        # A ranking batch: 256 ragged requests of about 200 candidates each.
        {"name": "rank_batch", "kind": "rank", "requests": 256, "cands": 51203,
         "history": 163840},
        # The retrieval tower over a batch of ragged requests.
        {"name": "mlp_retrieval", "kind": "mlp", "requests": 64, "cands": 64324, "k_req": 1024,
         "k_cand": 256, "hidden": 512, "d_out": 256},
        # Feature interaction: 32 request fields, 8 candidate fields of width 128.
        {"name": "fm_interaction", "kind": "fm", "requests": 128, "cands": 65536, "d_out": 512},
        # Field compression of a retrieval batch.
        {"name": "lcb_batch", "kind": "lcb", "requests": 16, "cands": 65536, "f_req": 128,
         "f_cand": 32, "o_req": 64, "o_cand": 32, "emb": 128},
        # The production retrieval layer: a million candidates.
        {"name": "linear_production", "kind": "linear", "requests": 16, "cands": 1048576,
         "k_req": 2048, "k_cand": 512, "d_out": 1024, "relu": True, "bias": False,
         "residual": False, "mapped": False},
        # The same tower's first layer on candidates in arbitrary order.
        {"name": "linear_shuffled", "kind": "linear", "requests": 64, "cands": 64324,
         "k_req": 1024, "k_cand": 256, "d_out": 512, "relu": True, "bias": False,
         "residual": False, "mapped": True},
        # A ranking layer of widths off the tiles, with bias and residual input.
        {"name": "linear_odd_widths", "kind": "linear", "requests": 100, "cands": 20011,
         "k_req": 200, "k_cand": 360, "d_out": 300, "relu": True, "bias": True,
         "residual": True, "mapped": False},
        # Production retrieval attention: one query per candidate, history 2048.
        {"name": "attention_production", "kind": "attention", "requests": 16, "cands": 1048576,
         "tokens": 1, "history": 32768, "heads": 8, "dim": 128, "mapped": False},
        # Multi-token queries of candidates in arbitrary order.
        {"name": "attention_tokens_shuffled", "kind": "attention", "requests": 16, "cands": 8192,
         "tokens": 32, "history": 32768, "heads": 8, "dim": 128, "mapped": True},
        # A whole DCA layer, both groups.
        {"name": "dca_layer", "kind": "layer", "requests": 16, "cands": 8192, "tokens": 32,
         "history": 16384, "heads": 4, "dim": 64},
    ]


def _log(rng, lo, hi, step=1):
    """A whole number in [lo, hi], spread over its logarithm, a multiple of `step`."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step
    return min(max(v, lo), hi)


def draw(rng):
    kind = rng.choice(["block", "rank", "mlp", "fm", "lcb", "linear", "linear", "attention",
                       "attention", "layer"])
    if kind == "block":
        r = _log(rng, 1, 16)
        return {"kind": kind, "requests": r, "cands": r * _log(rng, 16, 128) + rng.randrange(16),
                "k_req": _log(rng, 64, 512), "k_cand": _log(rng, 32, 256),
                "d_out": _log(rng, 64, 512), "history": r * _log(rng, 8, 128),
                "heads": rng.choice([1, 2, 4]), "dim": rng.choice([16, 32, 64])}
    if kind == "rank":
        r = _log(rng, 1, 256)
        return {"kind": kind, "requests": r, "cands": r * _log(rng, 32, 512) + rng.randrange(64),
                "history": r * _log(rng, 64, 1024)}
    if kind == "mlp":
        return {"kind": kind, "requests": _log(rng, 1, 128), "cands": _log(rng, 256, 131072),
                "k_req": _log(rng, 64, 1024, 8), "k_cand": rng.choice([128, 256]),
                "hidden": _log(rng, 128, 1024, 64), "d_out": rng.choice([128, 256])}
    if kind == "fm":
        return {"kind": kind, "requests": _log(rng, 1, 128), "cands": _log(rng, 256, 131072),
                "d_out": _log(rng, 64, 1024, 64)}
    if kind == "lcb":
        emb, o_cand = rng.choice([(128, 32), (64, 32), (64, 64)])
        return {"kind": kind, "requests": _log(rng, 1, 64), "cands": _log(rng, 256, 65536),
                "f_req": _log(rng, 16, 128), "f_cand": rng.choice([16, 32, 64]),
                "o_req": rng.choice([32, 64]), "o_cand": o_cand, "emb": emb}
    if kind == "linear":
        return {"kind": kind, "requests": _log(rng, 1, 256), "cands": _log(rng, 128, 524288),
                "k_req": _log(rng, 64, 2048, 8),
                "k_cand": rng.choice([64, 128, 256, 512, _log(rng, 64, 512, 8)]),
                "d_out": rng.choice([128, 256, 512, 1024, _log(rng, 64, 1024, 4)]),
                "relu": rng.random() < 0.7, "bias": rng.random() < 0.5,
                "residual": rng.random() < 0.25, "mapped": rng.random() < 0.25}
    if kind == "attention":
        r, tokens = _log(rng, 1, 48), rng.choice([1, 1, 4, 32])
        return {"kind": kind, "requests": r,
                "cands": r * max(1, _log(rng, 16, 16384) // tokens) + rng.randrange(8),
                "tokens": tokens, "history": r * _log(rng, 64, 2048),
                "heads": rng.choice([2, 4, 8]), "dim": rng.choice([64, 128]),
                "mapped": rng.random() < 0.25}
    r = _log(rng, 1, 32)
    return {"kind": kind, "requests": r, "cands": r * _log(rng, 16, 256) + rng.randrange(8),
            "tokens": rng.choice([8, 16, 32]), "history": r * _log(rng, 64, 1024),
            "heads": rng.choice([2, 4]), "dim": 64}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

class _Draws:
    """Seeded inputs: numpy for the ragged splits, the GPU for the tensors."""

    def __init__(self, seed):
        self.np = np.random.default_rng(seed)
        self.gen = torch.Generator(device=DEV).manual_seed(seed)

    def normal(self, shape, std=1.0, dtype=BF16):
        t = torch.randn(shape, generator=self.gen, device=DEV, dtype=dtype)
        return t if std == 1.0 else t * std

    def weight(self, d_out, d_in, fan_in=None, dtype=BF16):
        return self.normal((d_out, d_in), 1.0 / math.sqrt(fan_in or d_in), dtype)

    def split(self, total, parts):
        """`total` rows on `parts` requests, from about 0.4 to 1.6 of the mean."""
        share = self.np.uniform(0.4, 1.6, size=parts)
        edges = np.floor(np.cumsum(share) / share.sum() * total + 0.5).astype(np.int64)
        edges[-1] = total
        return np.diff(edges, prepend=0)

    def offsets(self, total, parts):
        return torch.from_numpy(workloads.offsets_from_counts(self.split(total, parts))).to(DEV)


def _empty(*shape, dtype=BF16):
    return torch.empty(shape, dtype=dtype, device=DEV)


def _bytes(n):
    return torch.empty(max(int(n), 1), dtype=torch.uint8, device=DEV)


def _owners(offsets, n):
    counts = (offsets[1:] - offsets[:-1]).long()
    return torch.repeat_interleave(torch.arange(counts.numel(), device=DEV), counts,
                                   output_size=n)


def _layer_inputs(c, seed):
    d = _Draws(seed)
    return workloads.dca_layer_case(
        d.split(c["cands"], c["requests"]), d.split(c["history"], c["requests"]), f_req=64,
        f_cand=32, o_req=64, o_cand=32, emb=64, d_hidden=512, q_len=c["tokens"],
        heads=c["heads"], head_dim=c["dim"], d_seq=256, seed=seed)


def _inputs(c, seed):
    """The tensors of a case, by name; shared by prepare() and exact()."""
    d, kind = _Draws(seed), c["kind"]
    r, n = c["requests"], c["cands"]
    s = {"co": d.offsets(n, r)}
    if kind == "block":
        fan, f32 = c["k_req"] + c["k_cand"], torch.float32
        hd = (c["heads"], c["dim"])
        s.update(x_req=d.normal((r, c["k_req"]), dtype=f32),
                 x_cand=d.normal((n, c["k_cand"]), dtype=f32),
                 w_req=d.weight(c["d_out"], c["k_req"], fan, f32),
                 w_cand=d.weight(c["d_out"], c["k_cand"], fan, f32),
                 q=d.normal((n, 1) + hd, dtype=f32), ko=d.offsets(c["history"], r),
                 k=d.normal((c["history"],) + hd, dtype=f32),
                 v=d.normal((c["history"],) + hd, dtype=f32))
    elif kind == "rank":
        s.update(ko=d.offsets(c["history"], r), e_c=d.normal((n, 256)),
                 s=d.normal((c["history"], 256)), wkv=d.weight(1024, 256),
                 wq1=d.weight(256, 256), wq2=d.weight(256, 256))
    elif kind == "mlp":
        fan = c["k_req"] + c["k_cand"]
        s.update(x_req=d.normal((r, c["k_req"])), x_cand=d.normal((n, c["k_cand"])),
                 w1_req=d.weight(c["hidden"], c["k_req"], fan),
                 w1_cand=d.weight(c["hidden"], c["k_cand"], fan),
                 w2=d.weight(c["d_out"], c["hidden"]),
                 b1=d.normal((c["hidden"],), 0.1, torch.float32),
                 b2=d.normal((c["d_out"],), 0.1, torch.float32))
    elif kind == "fm":
        s.update(x_req=d.normal((r, 32, 128), 128 ** -0.5),
                 x_cand=d.normal((n, 8, 128), 128 ** -0.5),
                 w_req=d.weight(c["d_out"], 1024, 1344), w_cand=d.weight(c["d_out"], 320, 1344),
                 bias=d.normal((c["d_out"],), 0.1, torch.float32))
    elif kind == "lcb":
        fan = c["f_req"] + c["f_cand"]
        s.update(x_req=d.normal((r, c["f_req"], c["emb"])),
                 x_cand=d.normal((n, c["f_cand"], c["emb"])),
                 w_rr=d.weight(c["o_req"], c["f_req"]), w_cr=d.weight(c["o_cand"], c["f_req"], fan),
                 w_cc=d.weight(c["o_cand"], c["f_cand"], fan))
    elif kind == "linear":
        fan = c["k_req"] + c["k_cand"]
        s.update(x_req=d.normal((r, c["k_req"])), x_cand=d.normal((n, c["k_cand"])),
                 w_req=d.weight(c["d_out"], c["k_req"], fan),
                 w_cand=d.weight(c["d_out"], c["k_cand"], fan),
                 bias=d.normal((c["d_out"],), 0.1, torch.float32) if c["bias"] else None,
                 add=d.normal((n, c["k_cand"])) if c["residual"] else None)
    elif kind == "attention":
        width = c["heads"] * c["dim"]
        # K and V are the two halves of one projection's rows.
        s.update(ko=d.offsets(c["history"], r),
                 q=d.normal((n, c["tokens"], c["heads"], c["dim"])),
                 kv=d.normal((c["history"], 2 * width)))
    if c.get("mapped"):
        perm = torch.from_numpy(d.np.permutation(n)).to(DEV)
        s["ids"] = _owners(s["co"], n)[perm].to(torch.int32)
    return s


def _halves(kv, heads, dim):
    w = heads * dim
    return kv[:, :w].view(-1, heads, dim), kv[:, w:].view(-1, heads, dim)


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "layer":
        return {"case": c, "layer": pipelines.prepare_dca_layer(_layer_inputs(c, seed))}
    s = _inputs(c, seed)
    s["case"] = c
    r, n = c["requests"], c["cands"]
    if kind == "block":
        s.update(out=_empty(n, c["d_out"], dtype=torch.float32), att=torch.empty_like(s["q"]),
                 ws=_bytes(ops.linear_workspace_size(r, n, c["d_out"], c["k_req"])))
    elif kind == "rank":
        s.update(kv=_empty(c["history"], 1024), plan=_bytes(ops.dca_attention_plan_size(r)),
                 a1=_empty(n, 1, 4, 64), a2=_empty(n, 1, 4, 64), u=_empty(n, 1, 4, 64))
    elif kind == "mlp":
        s.update(out=_empty(n, c["d_out"]), ws=_bytes(ops.mlp2_workspace_size(
            r, n, c["k_req"], c["k_cand"], c["hidden"], c["d_out"], BF16)))
    elif kind == "fm":
        s.update(out=_empty(n, c["d_out"]), ws=_bytes(ops.fm_linear_workspace_size(
            r, n, 32, 8, 128, c["d_out"], BF16)))
    elif kind == "lcb":
        s.update(y_req=_empty(r, c["o_req"], c["emb"]), y_cand=_empty(n, c["o_cand"], c["emb"]),
                 ws=_bytes(ops._lib.load().rocs_ikbo_lcb_workspace_size(r, c["o_cand"], c["emb"])))
    elif kind == "linear":
        s.update(out=_empty(n, c["d_out"]),
                 ws=_bytes(ops.linear_workspace_size(r, n, c["d_out"], c["k_req"])))
    elif kind == "attention":
        s.update(out=torch.empty_like(s["q"]))
        if c["mapped"]:
            s["ws"] = _bytes(ops.dca_attention_mapped_workspace_size(r, n))
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "block":
        ops.ikbo_linear(s["x_cand"], s["w_cand"], x_req=s["x_req"], w_req=s["w_req"],
                        cand_offsets=s["co"], activation="relu", out=s["out"], workspace=s["ws"])
        ops.dca_attention(s["q"], s["k"], s["v"], s["co"], s["ko"], out=s["att"])
        return {"linear": s["out"], "attention": s["att"]}
    if kind == "rank":
        n, kv = c["cands"], s["kv"]
        k1, v1 = _halves(kv[:, :512], 4, 64)
        k2, v2 = _halves(kv[:, 512:], 4, 64)
        ops.ikbo_linear(s["s"], s["wkv"], out=kv)
        plan = ops.dca_attention_plan(s["co"], s["ko"], num_cand=n, heads=4, plan=s["plan"])
        ops.dca_attention_proj(s["e_c"].view(n, 1, 256), s["wq1"], k1, v1, s["co"], s["ko"],
                               heads=4, plan=plan, residual=s["e_c"].view(n, 1, 4, 64),
                               out=s["a1"], out_sum=s["u"])
        ops.dca_attention_proj(s["u"].view(n, 1, 256), s["wq2"], k2, v2, s["co"], s["ko"],
                               heads=4, plan=plan, out=s["a2"])
        return {"kv": kv, "a1": s["a1"], "u": s["u"], "a2": s["a2"]}
    if kind == "mlp":
        return ops.ikbo_mlp2(s["x_cand"], s["w1_cand"], s["w2"], x_req=s["x_req"],
                             w1_req=s["w1_req"], cand_offsets=s["co"], b1=s["b1"], b2=s["b2"],
                             out=s["out"], workspace=s["ws"])
    if kind == "fm":
        return ops.glm_fm_linear(s["x_req"], s["x_cand"], s["co"], s["w_req"], s["w_cand"],
                                 bias=s["bias"], out=s["out"], workspace=s["ws"])
    if kind == "lcb":
        return ops.ikbo_lcb(s["x_req"], s["x_cand"], s["w_cr"], s["w_cc"], s["co"],
                            w_rr=s["w_rr"], y_req=s["y_req"], y_cand=s["y_cand"],
                            workspace=s["ws"])
    if kind == "linear":
        call, index = ((ops.ikbo_linear_mapped, {"cand_request_ids": s["ids"]}) if c["mapped"]
                       else (ops.ikbo_linear, {"cand_offsets": s["co"]}))
        return call(s["x_cand"], s["w_cand"], x_req=s["x_req"], w_req=s["w_req"],
                    bias=s["bias"], activation="relu" if c["relu"] else "none",
                    x_cand_add=s["add"], out=s["out"], workspace=s["ws"], **index)
    if kind == "attention":
        k, v = _halves(s["kv"], c["heads"], c["dim"])
        if c["mapped"]:
            return ops.dca_attention_mapped(s["q"], k, v, s["ids"], s["ko"], out=s["out"],
                                            workspace=s["ws"])
        return ops.dca_attention(s["q"], k, v, s["co"], s["ko"], out=s["out"])
    return pipelines.dca_layer_step(s["layer"])


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how far a correct one may be off
# ---------------------------------------------------------------------------

def work(case):
    c, kind = case, case["kind"]
    r, n = c["requests"], c["cands"]
    mean_l = c.get("history", 0) / r
    if kind == "block":
        hd = c["heads"] * c["dim"]
        fan = c["k_req"] + c["k_cand"]
        return {"bytes": 4.0 * (r * c["k_req"] + n * c["k_cand"] + fan * c["d_out"]
                                + n * c["d_out"] + 2 * n * hd + 2 * c["history"] * hd),
                "flops": 2.0 * c["d_out"] * (n * c["k_cand"] + r * c["k_req"])
                + 4.0 * n * mean_l * hd}
    if kind == "rank":
        # History in, K and V of two layers out; candidates in, three outputs.
        return {"bytes": 2.0 * (c["history"] * (256 + 1024) + n * 256 * 4 + 6 * 256 * 256),
                "flops": 2.0 * c["history"] * 256 * 1024 + 4.0 * n * 256 * 256
                + 2 * 4.0 * n * mean_l * 256}
    if kind == "mlp":
        fan = c["k_req"] + c["k_cand"]
        return {"bytes": 2.0 * (r * c["k_req"] + n * (c["k_cand"] + c["d_out"])
                                + c["hidden"] * (fan + c["d_out"])),
                "flops": 2.0 * c["hidden"] * (n * (c["k_cand"] + c["d_out"]) + r * c["k_req"])}
    if kind == "fm":
        return {"bytes": 2.0 * (r * 32 * 128 + n * (8 * 128 + c["d_out"]) + c["d_out"] * 1344),
                "flops": 2.0 * (r * 1024 * 128 + n * 320 * 128
                                + c["d_out"] * (r * 1024 + n * 320))}
    if kind == "lcb":
        o = c["o_req"] + c["o_cand"]
        return {"bytes": 2.0 * (c["emb"] * (r * (c["f_req"] + c["o_req"])
                                            + n * (c["f_cand"] + c["o_cand"]))
                                + o * c["f_req"] + c["o_cand"] * c["f_cand"]),
                "flops": 2.0 * c["emb"] * (r * o * c["f_req"] + n * c["o_cand"] * c["f_cand"])}
    if kind == "linear":
        x = c["k_cand"] * (2 if c["residual"] else 1)
        return {"bytes": 2.0 * (r * c["k_req"] + n * (x + c["d_out"])
                                + c["d_out"] * (c["k_req"] + c["k_cand"]))
                + (4.0 * n if c["mapped"] else 0.0),
                "flops": 2.0 * c["d_out"] * (n * c["k_cand"] + r * c["k_req"])}
    rows, hd = n * c["tokens"], c["heads"] * c["dim"]
    if kind == "attention":
        return {"bytes": 4.0 * hd * (rows + c["history"]) + (4.0 * n if c["mapped"] else 0.0),
                "flops": 4.0 * rows * mean_l * hd}
    d_q = c["tokens"] * hd
    return {"bytes": 2.0 * (r * 64 * 64 + n * 32 * 64 + c["history"] * 256 + 2 * (r + n) * d_q),
            "flops": 2.0 * n * 32 * 64 * (32 + 512) + 2.0 * n * 512 * d_q
            + 2.0 * r * (96 * 64 * 64 + 2 * 4096 * 512 + 2 * 512 * d_q)
            + 8.0 * c["history"] * 256 * hd + 4.0 * (rows + r * c["tokens"]) * mean_l * hd}


def tolerance(case):
    # About four times the distance to exact() measured for each kind.
    kind = case["kind"]
    if kind == "block":
        return {"rel": 1e-6, "max": 1e-5}      # fp32 sums (2.6e-7 measured)
    if kind in ("rank", "layer"):
        return {"rel": 1.5e-2, "max": 0.1}     # bf16 through several operators (3.8e-3)
    if kind in ("attention", "mlp", "fm"):
        return {"rel": 9e-3, "max": 0.05}      # bf16 intermediate and output (2.3e-3)
    return {"rel": 7e-3, "max": 0.05}          # bf16 outputs of fp32 sums (1.7e-3)


# ---------------------------------------------------------------------------
# The same in float64, in plain torch
# ---------------------------------------------------------------------------

def _d(t):
    return None if t is None else t.double()


def _bounds(offsets):
    off = offsets.tolist()
    return list(zip(off[:-1], off[1:]))


def _linear64(x_cand, w_cand, x_req=None, w_req=None, owners=None, bias=None, relu=False):
    y = _d(x_cand) @ _d(w_cand).t()
    if x_req is not None:
        y += (_d(x_req) @ _d(w_req).t())[owners]
    if bias is not None:
        y += _d(bias)
    return y.clamp_(min=0.0) if relu else y


def _attention64(q, k, v, co, ko, rows=8192):
    """q [N, T, H, d] of request-contiguous candidates; k, v [L, H, d]."""
    out = torch.zeros(q.shape, dtype=torch.float64, device=q.device)
    t, h, d = q.shape[1:]
    for (a, b), (ka, kb) in zip(_bounds(co), _bounds(ko)):
        if a == b or ka == kb:
            continue
        kk = [_d(k[ka:kb, i]).contiguous() for i in range(h)]
        vv = [_d(v[ka:kb, i]).contiguous() for i in range(h)]
        step = max(1, rows // t)
        for lo in range(a, b, step):
            hi = min(lo + step, b)
            for i in range(h):
                qq = _d(q[lo:hi, :, i]).reshape(-1, d)
                p = torch.softmax(qq @ kk[i].t() / math.sqrt(d), dim=1)
                out[lo:hi, :, i] = (p @ vv[i]).view(hi - lo, t, d)
    return out


def _layer64(c, seed):
    w = _layer_inputs(c, seed)
    g = {k: torch.from_numpy(np.ascontiguousarray(v)).to(DEV) for k, v in vars(w).items()
         if isinstance(v, np.ndarray)}
    r, n, t, h, d = c["requests"], c["cands"], c["tokens"], c["heads"], c["dim"]
    co, ko = g["cand_offsets"], g["kv_offsets"]
    own = _owners(co, n)
    x_r, x_c = _d(g["y_req"]), _d(g["y_cand"])
    z_r = torch.matmul(_d(g["lcb_rr"]), x_r).reshape(r, -1)
    z_c = (torch.matmul(_d(g["lcb_cc"]), x_c)
           + torch.matmul(_d(g["lcb_cr"]), x_r)[own]).reshape(n, -1)
    h_r = _linear64(z_r, g["w1_rr"], bias=g["b1_r"], relu=True)
    h_c = _linear64(z_c, g["w1_cc"], z_r, g["w1_cr"], own, g["b1_c"], True)
    q_r = _linear64(h_r, g["w2_rr"]).view(r, t, h, d)
    q_c = _linear64(h_c, g["w2_cc"], h_r, g["w2_cr"], own).view(n, t, h, d)
    k_r, v_r, k_c, v_c = (_linear64(g["s"], g[name]).view(-1, h, d)
                          for name in ("wk_r", "wv_r", "wk_c", "wv_c"))
    return {"q_req": q_r, "q_cand": q_c,
            "a_req": _attention64(q_r, k_r, v_r, torch.arange(r + 1), ko),
            "a_cand": _attention64(q_c, k_c, v_c, co, ko)}


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "layer":
        return _layer64(c, seed)
    s = _inputs(c, seed)
    r, n = c["requests"], c["cands"]
    own = _owners(s["co"], n)
    if kind == "block":
        return {"linear": _linear64(s["x_cand"], s["w_cand"], s["x_req"], s["w_req"], own,
                                    relu=True),
                "attention": _attention64(s["q"], s["k"], s["v"], s["co"], s["ko"])}
    if kind == "rank":
        kv = _linear64(s["s"], s["wkv"])
        e = _d(s["e_c"])
        k1, v1 = _halves(kv[:, :512], 4, 64)
        k2, v2 = _halves(kv[:, 512:], 4, 64)
        a1 = _attention64((e @ _d(s["wq1"]).t()).view(n, 1, 4, 64), k1, v1, s["co"], s["ko"])
        u = a1 + e.view(n, 1, 4, 64)
        a2 = _attention64((u.view(n, 256) @ _d(s["wq2"]).t()).view(n, 1, 4, 64), k2, v2,
                          s["co"], s["ko"])
        return {"kv": kv, "a1": a1, "u": u, "a2": a2}
    if kind == "mlp":
        h = _linear64(s["x_cand"], s["w1_cand"], s["x_req"], s["w1_req"], own, s["b1"], True)
        return _linear64(h, s["w2"], bias=s["b2"])
    if kind == "fm":
        x_r, out = _d(s["x_req"]), []
        y_r = torch.matmul(x_r, x_r.transpose(1, 2).contiguous()).reshape(r, -1)
        z = y_r @ _d(s["w_req"]).t() + _d(s["bias"])
        for lo in range(0, n, 8192):
            o, x_c = own[lo:lo + 8192], _d(s["x_cand"][lo:lo + 8192])
            fields = torch.cat([x_r[o], x_c], dim=1).transpose(1, 2).contiguous()
            y_c = torch.matmul(x_c, fields).reshape(o.numel(), -1)
            out.append((y_c @ _d(s["w_cand"]).t() + z[o]).clamp_(min=0.0))
        return torch.cat(out)
    if kind == "lcb":
        x_r = _d(s["x_req"])
        y_c = torch.matmul(_d(s["w_cc"]), _d(s["x_cand"]))
        y_c += torch.matmul(_d(s["w_cr"]), x_r)[own]
        return torch.matmul(_d(s["w_rr"]), x_r), y_c
    if kind == "linear":
        x = s["x_cand"] if s["add"] is None else s["x_cand"] + s["add"]
        return _linear64(x, s["w_cand"], s["x_req"], s["w_req"],
                         s["ids"].long() if c["mapped"] else own, s["bias"], c["relu"])
    k, v = _halves(s["kv"], c["heads"], c["dim"])
    if not c["mapped"]:
        return _attention64(s["q"], k, v, s["co"], s["ko"])
    order = torch.argsort(s["ids"], stable=True)
    out = torch.empty(s["q"].shape, dtype=torch.float64, device=DEV)
    out[order] = _attention64(s["q"][order], k, v, s["co"], s["ko"])
    return out
