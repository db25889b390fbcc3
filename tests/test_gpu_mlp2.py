"""GPU parity: rocs_ikbo_mlp2 (two stacked linear layers, the first with the
request broadcast, the hidden layer on chip) against the oracle's
composition of two explicit-broadcast layers with H rounded to bf16."""

import numpy as np
import pytest
import torch

from gpu_util import assert_close, dev_bf16, dev_f32, dev_i32, host
from oracle import pipelines
from paper_2607_27744_amd import ops
from paper_2607_27744_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (counts, K_r, K_c, D_h, D_o, act1, act2, biases): every fused (K_c, D_o)
# pair; requests whose candidates end inside a 128-row tile, an empty
# request, a single candidate, one and several hidden chunks.
FUSED = [
    ([300, 0, 130, 1, 257], 64, 256, 192, 256, "relu", "none", True),
    ([129, 64, 7], 32, 128, 64, 128, "relu", "relu", False),
    ([1], 16, 256, 512, 128, "none", "none", True),
    ([700, 513], 1024, 128, 256, 256, "relu", "none", True),
    # Many requests per 128-candidate tile: the tile runs once per pair.
    ([3, 1, 0, 2, 5, 1, 1, 4, 0, 7] * 6 + [150], 16, 128, 1024, 128, "relu", "relu", True),
]


def _run(c, request=True, dtype=torch.bfloat16, **kw):
    dev = dev_bf16 if dtype == torch.bfloat16 else dev_f32
    b1 = None if c.b1 is None else dev_f32(c.b1)
    b2 = None if c.b2 is None else dev_f32(c.b2)
    if request:
        return host(ops.ikbo_mlp2(dev(c.x_cand), dev(c.w1_cand), dev(c.w2), x_req=dev(c.x_req),
                                  w1_req=dev(c.w1_req), cand_offsets=dev_i32(c.cand_offsets),
                                  b1=b1, b2=b2, **kw))
    return host(ops.ikbo_mlp2(dev(c.x_cand), dev(c.w1_cand), dev(c.w2), b1=b1, b2=b2, **kw))


def _want(c, request=True, act1="relu", act2="none", rows=None):
    if request:
        return pipelines.ikbo_mlp2(c.x_req, c.x_cand, c.w1_req, c.w1_cand, c.b1, c.w2, c.b2,
                                   c.cand_offsets, act1, act2, rows=rows)
    return pipelines.ikbo_mlp2(None, c.x_cand, None, c.w1_cand, c.b1, c.w2, c.b2, None, act1,
                               act2, rows=rows)


@pytest.mark.parametrize("case", FUSED, ids=lambda c: f"kc{c[2]}-dh{c[3]}-do{c[4]}")
def test_fused_matches_oracle(gpu_lib, case):
    counts, k_req, k_cand, d_h, d_o, a1, a2, biases = case
    c = wl.mlp2_case(counts, k_req, k_cand, d_h, d_o, seed=3, biases=biases)
    got = _run(c, activation1=a1, activation2=a2)
    assert_close(got, _want(c, act1=a1, act2=a2), f"mlp2 {case}")


def test_no_request_term(gpu_lib):
    # Without x_req the tiles run over the candidates contiguously and the
    # first layer's additive row is b1 (or nothing).
    c = wl.mlp2_case([200, 77], 8, 256, 128, 256, seed=4)
    assert_close(_run(c, request=False), _want(c, request=False), "b1 only")
    c.b1 = None
    assert_close(_run(c, request=False), _want(c, request=False), "no additive term")


def test_two_launch_form(gpu_lib):
    # Shapes without the fused kernel (K_c = 96) and fp32 run two launches of
    # the linear kernels with H in the workspace; same results.
    c = wl.mlp2_case([90, 0, 33], 40, 96, 80, 48, seed=5)
    assert_close(_run(c), _want(c), "bf16 two launches")
    c = wl.mlp2_case([20, 13], 24, 32, 40, 16, seed=6, bf16=False)
    got = _run(c, dtype=torch.float32)
    want = pipelines.ikbo_mlp2(c.x_req, c.x_cand, c.w1_req, c.w1_cand, c.b1, c.w2, c.b2,
                               c.cand_offsets, hidden="f32")
    assert_close(got, want, "fp32")


def test_index_probe_is_bit_exact(gpu_lib):
    # x_req[r] = r in feature 0, W1_CR picks it into hidden unit 0, W2 copies
    # hidden unit 0 into every output: out[n, :] == m_n exactly.
    counts = np.array([3, 0, 200, 1, 0, 140])
    c = wl.mlp2_case(counts, 8, 128, 64, 128, seed=7, biases=False)
    c.x_req = np.zeros_like(c.x_req)
    c.x_req[:, 0] = np.arange(6)
    c.w1_req = np.zeros_like(c.w1_req)
    c.w1_req[0, 0] = 1.0
    c.w1_cand = np.zeros_like(c.w1_cand)
    c.w2 = np.zeros_like(c.w2)
    c.w2[:, 0] = 1.0
    got = _run(c)
    want = np.repeat(np.arange(6), counts)[:, None] * np.ones((1, 128))
    np.testing.assert_array_equal(got, want)


def test_workload2_shape_sampled(gpu_lib):
    # The retrieval workload's two layers (64 requests, 512..1536 candidates
    # each, 1024 + 256 -> 512 ReLU -> 256) as one fused call, checked on a
    # sample of rows that covers every request's first and last candidate.
    w = wl.make_workload(2, seed=0)
    got = ops.ikbo_mlp2(dev_bf16(w.x_cand), dev_bf16(w.w1_cand), dev_bf16(w.w2),
                        x_req=dev_bf16(w.x_req), w1_req=dev_bf16(w.w1_req),
                        cand_offsets=dev_i32(w.cand_offsets))
    off = w.cand_offsets
    rows = np.unique(np.concatenate([off[:-1], off[1:] - 1,
                                     np.random.default_rng(0).integers(0, w.n_cand, 512)]))
    want = pipelines.ikbo_mlp2(w.x_req, w.x_cand, w.w1_req, w.w1_cand, None, w.w2, None, off,
                               rows=rows)
    assert_close(host(got)[rows], want, "workload 2")
    # Matches the two-launch pipeline's output (bf16 output rounding aside).
    ref = pipelines.retrieval_mlp(w, rows=rows)["out"]
    assert_close(host(got)[rows], ref, "workload 2 vs pipeline")


def test_repeated_calls_and_empty(gpu_lib):
    c = wl.mlp2_case([150, 40], 16, 256, 128, 128, seed=8)
    first = _run(c)
    np.testing.assert_array_equal(_run(c), first)                 # deterministic
    out = ops.ikbo_mlp2(dev_bf16(c.x_cand[:0]), dev_bf16(c.w1_cand), dev_bf16(c.w2),
                        x_req=dev_bf16(c.x_req), w1_req=dev_bf16(c.w1_req),
                        cand_offsets=dev_i32(np.zeros(3, dtype=np.int32)))
    assert out.shape == (0, 128)


@pytest.mark.parametrize("k_cand,d_h,d_o", [(128, 64, 128), (256, 64, 256), (128, 192, 256),
                                            (256, 320, 128), (128, 960, 128), (256, 1024, 256)])
@pytest.mark.parametrize("counts", [[1], [31, 0, 2], [32, 1] * 20 + [7], [5000, 0, 3193], [16384], [16380, 5]],
                         ids=lambda c: f"N{sum(c)}-R{len(c)}")
def test_few_candidates(gpu_lib, counts, k_cand, d_h, d_o):
    # 32-candidate workgroups, two for each CU at most (16,384 candidates on 256
    # CUs), and one candidate past one and two rounds: hidden layers of two blocks to the largest, rows
    # past the end, requests that end inside a workgroup.
    c = wl.mlp2_case(counts, 16, k_cand, d_h, d_o, seed=sum(counts) + d_h)
    got = _run(c, activation2="relu")
    np.testing.assert_array_equal(_run(c, activation2="relu"), got)
    rows = np.unique(np.concatenate([np.arange(min(c.n_cand, 96)), [c.n_cand - 1],
                                     np.random.default_rng(1).integers(0, c.n_cand, 200)]))
    assert_close(got[rows], _want(c, act2="relu", rows=rows), f"{counts} {k_cand} {d_h} {d_o}")


@pytest.mark.parametrize("n,k_cand", [(200, 128), (17000, 128), (200, 136)],
                         ids=["small", "persistent", "two launches"])
@pytest.mark.parametrize("acts", [("none", "none"), ("relu", "none"), ("relu", "relu")],
                         ids="-".join)
def test_nan_stays_in_its_row_and_is_no_infinity(gpu_lib, n, k_cand, acts):
    # Every form of the operator: NaN of either sign stays NaN where there is no
    # activation and becomes nothing but 0 under ReLU.
    c = wl.mlp2_case([n - 60, 60], 16, k_cand, 64, 128, seed=5)
    x, b2 = c.x_cand.copy(), c.b2.copy()
    x[3, 0], x[n - 1, 5] = np.nan, np.copysign(np.nan, -1)
    b2[7], b2[9] = np.nan, np.copysign(np.nan, -1)
    args = dict(x_req=dev_bf16(c.x_req), w1_req=dev_bf16(c.w1_req), b1=dev_f32(c.b1),
                cand_offsets=dev_i32(c.cand_offsets), activation1=acts[0], activation2=acts[1])
    want = host(ops.ikbo_mlp2(dev_bf16(c.x_cand), dev_bf16(c.w1_cand), dev_bf16(c.w2),
                              b2=dev_f32(c.b2), **args))
    got = host(ops.ikbo_mlp2(dev_bf16(x), dev_bf16(c.w1_cand), dev_bf16(c.w2), b2=dev_f32(b2),
                             **args))
    rows, cols = np.setdiff1d(np.arange(n), [3, n - 1]), np.setdiff1d(np.arange(128), [7, 9])
    assert np.array_equal(got[np.ix_(rows, cols)], want[np.ix_(rows, cols)])
    spoiled = [got[rows][:, [7, 9]]]
    if acts[0] == "none":                        # else the hidden layer's ReLU comes between
        spoiled.append(got[[3, n - 1]])
    assert not np.any(np.isinf(got))
    for part in spoiled:
        assert np.all(np.isnan(part) | (part == 0) if acts[1] == "relu" else np.isnan(part))
