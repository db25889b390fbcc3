"""GPU parity: rocs_glm_fm_linear (GLM FM interaction fused into the operand
of the linear that consumes it) against the oracle's composition of the
explicit-broadcast interaction and linear, Y^R and Y^C rounded to bf16."""

import numpy as np
import pytest
import torch

from gpu_util import assert_close, dev_bf16, dev_f32, dev_i32, host
from oracle import pipelines
from oracle.bf16 import round_bf16
from paper_2607_27744_amd import ops
from paper_2607_27744_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _run(c, act="relu", dtype=torch.bfloat16):
    dev = dev_bf16 if dtype == torch.bfloat16 else dev_f32
    bias = None if c.bias is None else dev_f32(c.bias)
    need = ops.fm_linear_workspace_size(c.n_req, c.n_cand, c.f_req, c.f_cand, c.emb_dim,
                                        c.d_out, dtype)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    out = ops.glm_fm_linear(dev(c.x_req), dev(c.x_cand), dev_i32(c.cand_offsets), dev(c.w_req),
                            dev(c.w_cand), bias=bias, activation=act, workspace=ws)
    k_r = c.f_req * c.f_req
    y_req = ws[:c.n_req * k_r * (2 if dtype == torch.bfloat16 else 4)]
    y_req = y_req.view(dtype).view(c.n_req, k_r)
    return host(out), host(y_req)


def _want(c, act="relu", rows=None):
    y_req, _, out = pipelines.glm_fm_linear(c.x_req, c.x_cand, c.w_req, c.w_cand, c.bias,
                                            c.cand_offsets, act, rows=rows)
    return out, y_req


# (counts, D, act, bias): the fused shape (F_r 32, F_c 8, E 128) with
# request-aligned tiles that end inside a request, an empty request, a single
# candidate, one and several output chunks.
FUSED = [
    ([300, 0, 130, 1, 257], 512, "relu", True),
    ([129, 64, 7], 64, "none", False),
    ([1], 128, "relu", True),
]


@pytest.mark.parametrize("case", FUSED, ids=lambda c: f"d{c[1]}-{c[2]}")
def test_fused_matches_oracle(gpu_lib, case):
    counts, d, act, bias = case
    c = wl.fm_linear_case(counts, 32, 8, 128, d, seed=2, bias=bias)
    got, y_req = _run(c, act)
    want, want_yr = _want(c, act)
    assert_close(y_req, want_yr, "Y^R")
    assert_close(got, want, f"fm_linear {case}")


def test_two_operator_form(gpu_lib):
    # Shapes without the fused kernel, and fp32, run the interaction and the
    # linear kernels one after the other; same results.
    c = wl.fm_linear_case([70, 0, 33], 16, 4, 64, 48, seed=3)
    got, _ = _run(c)
    assert_close(got, _want(c)[0], "bf16 two operators")
    c = wl.fm_linear_case([20, 9], 8, 4, 32, 24, seed=4, bf16=False)
    got, _ = _run(c, dtype=torch.float32)
    y_req, y_cand, out = pipelines.glm_fm_linear(c.x_req, c.x_cand, c.w_req, c.w_cand, c.bias,
                                                 c.cand_offsets)
    # fp32 storage of Y^R and Y^C: recompute without the bf16 rounding.
    from oracle import ikbo
    yr, yc = ikbo.glm_fm(c.x_req, c.x_cand, c.cand_offsets)
    m = ikbo.request_ids(c.cand_offsets)
    want = ikbo.ikbo_linear(yr[m], yc, c.w_req, c.w_cand, c.bias, np.arange(m.size + 1), "relu")
    assert_close(got, want, "fp32 two operators")


def test_index_probe_is_bit_exact(gpu_lib):
    # One-hot embeddings: request r's fields are r e_j, candidate field i is
    # e_i. W_CR sums the trace of Y^R (32 r^2), W_CC picks Y^C[n][0][0] (= r):
    # out[n] = 32 r^2 + r exactly (r <= 5 keeps every value a small integer).
    counts = np.array([3, 0, 140, 1, 0, 129])
    c = wl.fm_linear_case(counts, 32, 8, 128, 64, seed=5, bias=False)
    c.x_req = np.zeros_like(c.x_req)
    for r in range(6):
        c.x_req[r, :, :32] = r * np.eye(32)
    c.x_cand = np.zeros_like(c.x_cand)
    for i in range(8):
        c.x_cand[:, i, i] = 1.0
    c.w_req = np.zeros_like(c.w_req)
    c.w_req[0, np.arange(32) * 33] = 1.0
    c.w_cand = np.zeros_like(c.w_cand)
    c.w_cand[1, 0] = 1.0
    got, _ = _run(c, act="none")
    m = np.repeat(np.arange(6), counts)
    np.testing.assert_array_equal(got[:, 0], 32.0 * m ** 2)
    np.testing.assert_array_equal(got[:, 1], m)
    np.testing.assert_array_equal(got[:, 2:], 0.0)


def test_candidate_block_probe_is_bit_exact(gpu_lib):
    # The candidate-candidate features alone: W_CC picks Y^C[n][i][32 + j] =
    # <x_i, x_j> for a few (i, j) pairs; integer embeddings make the dot
    # products exact, and the output is their bf16 rounding (the interaction
    # is handed to the linear in bf16).
    counts = np.array([130, 70])
    c = wl.fm_linear_case(counts, 32, 8, 128, 64, seed=6, bias=False)
    rng = np.random.default_rng(6)
    c.x_req = np.zeros_like(c.x_req)
    c.x_cand = rng.integers(-2, 3, size=c.x_cand.shape).astype(np.float64)
    c.w_req = np.zeros_like(c.w_req)
    c.w_cand = np.zeros_like(c.w_cand)
    pairs = [(0, 0), (1, 0), (7, 3), (6, 7), (2, 5), (5, 2), (3, 3), (4, 1)]
    for o, (i, j) in enumerate(pairs):
        c.w_cand[o, 40 * i + 32 + j] = 1.0
    got, _ = _run(c, act="none")
    for o, (i, j) in enumerate(pairs):
        want = round_bf16(np.einsum("nd,nd->n", c.x_cand[:, i], c.x_cand[:, j]))
        np.testing.assert_array_equal(got[:, o], want, err_msg=f"pair {(i, j)}")


def test_workload4_shape_sampled(gpu_lib):
    w = wl.make_workload(4, seed=0)
    c = wl.fm_linear_case([1], 32, 8, 128, 512)      # only for the field names
    c.__dict__.update(x_req=w.x_req, x_cand=w.x_cand, cand_offsets=w.cand_offsets,
                      w_req=w.w_req, w_cand=w.w_cand, bias=None, n_req=w.n_req,
                      n_cand=w.n_cand, d_out=512)
    got, y_req = _run(c)
    off = w.cand_offsets
    rows = np.unique(np.concatenate([off[:-1], off[1:] - 1,
                                     np.random.default_rng(0).integers(0, w.n_cand, 256)]))
    want = pipelines.fm_linear(w, rows=rows)
    assert_close(got[rows], want["out"], "workload 4")
    assert_close(y_req, want["y_req"], "workload 4 Y^R")


# The block walk and the feature slices: runs of one, two and several blocks
# per workgroup, blocks of one candidate, waves without features (320 of 512),
# slices of 64 (d 576), 512 (1024) and the largest d_out.
@pytest.mark.parametrize("counts,d", [([1, 31, 32, 33, 0, 64], 320), ([9000, 1, 0, 7003], 192),
                                      ([3] * 300, 576), ([8300, 9100, 17], 1024), ([40, 7], 4096)],
                         ids=lambda v: f"N{sum(v)}" if isinstance(v, list) else f"d{v}")
def test_fused_block_walk_and_slices(gpu_lib, counts, d):
    c = wl.fm_linear_case(counts, 32, 8, 128, d, seed=d)
    got, _ = _run(c)
    n = c.n_cand
    rows = np.unique(np.concatenate([np.arange(0, n, max(1, n // 400)), c.cand_offsets[1:] - 1]))
    assert_close(got[rows], _want(c, rows=rows)[0], f"fm_linear N{n} d{d}")


@pytest.mark.parametrize("shape", [(32, 8, 128, 64), (16, 4, 64, 48)], ids=["fused", "two operators"])
@pytest.mark.parametrize("act", ["none", "relu"])
def test_nan_stays_in_its_row_and_is_no_infinity(gpu_lib, shape, act):
    f_req, f_cand, emb, d = shape
    c = wl.fm_linear_case([70, 0, 33], f_req, f_cand, emb, d, seed=6)
    want, _ = _run(c, act)
    c.x_cand = c.x_cand.copy()
    c.x_cand[4, 0, 0], c.x_cand[80, 1, 3] = np.nan, np.copysign(np.nan, -1)
    got, _ = _run(c, act)
    rows = np.setdiff1d(np.arange(103), [4, 80])
    assert np.array_equal(got[rows], want[rows])
    part = got[[4, 80]]
    assert np.all(np.isnan(part) | (part == 0) if act == "relu" else np.isnan(part))
