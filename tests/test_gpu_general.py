"""GPU parity of the general (any dtype, any size) kernels at their edges: the
16 / 32 tile switch, k remainders, aligned and unaligned rows, the request term
inside the product or through the table, rows of several requests in one tile."""

import numpy as np
import pytest
import torch

from gpu_util import assert_close, dev_bf16, dev_f32, dev_i32, host
from oracle import ikbo
from oracle.bf16 import round_bf16
from paper_2607_27744_amd import ops
from paper_2607_27744_amd import workloads as wl

pytestmark = pytest.mark.gpu

# fp32 sums of up to 1200 products of unit-variance terms scaled to O(1)
# outputs: error below 1200 * 2^-24 of the largest partial sum.
F32 = dict(atol=1e-4, rtol=1e-4, normwise=1e-5)

LINEAR = [  # counts, k_req, k_cand, d_out
    ([1], 1, 1, 1),
    ([3, 0, 14], 15, 17, 16),
    ([16, 1, 30, 0, 2], 64, 33, 31),        # 16 x 16 tiles of several requests
    ([700, 340], 20, 36, 500),              # 32 x 32 tiles (1040 x 500)
    ([9000, 1, 0, 7001], 700, 5, 33),       # the request table (N d_out k_req > 2^27)
]


@pytest.mark.parametrize("shape", LINEAR, ids=lambda s: f"N{sum(s[0])}-k{s[1]}-{s[2]}-d{s[3]}")
@pytest.mark.parametrize("mapped", [False, True], ids=["csr", "mapped"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_linear_general(gpu_lib, shape, mapped, dtype):
    counts, kr, kc, d = shape
    bf = dtype == "bf16"
    kc = kc if kc % 8 else kc + 1            # odd k keeps bf16 off the fast path
    c = wl.linear_case(counts, kr, kc, d, seed=kr + d, bf16=bf, bias_std=0.3, add_residual=True)
    dev = dev_bf16 if bf else dev_f32
    m = np.random.default_rng(d).permutation(ikbo.request_ids(c.cand_offsets))
    kw = dict(x_req=dev(c.x_req), w_req=dev(c.w_req), bias=dev_f32(c.bias),
              x_cand_add=dev(c.x_cand_add), activation="relu")
    xc = np.asarray(c.x_cand, np.float64) + c.x_cand_add
    xc = round_bf16(xc) if bf else xc.astype(np.float32)
    if mapped:
        got = gpu_lib.ikbo_linear_mapped(dev(c.x_cand), dev(c.w_cand),
                                         cand_request_ids=dev_i32(m), **kw)
        want = ikbo.ikbo_linear(c.x_req, xc, c.w_req, c.w_cand, c.bias, None, "relu",
                                request_map=m)
    else:
        got = gpu_lib.ikbo_linear(dev(c.x_cand), dev(c.w_cand),
                                  cand_offsets=dev_i32(c.cand_offsets), **kw)
        want = ikbo.ikbo_linear(c.x_req, xc, c.w_req, c.w_cand, c.bias, c.cand_offsets, "relu")
    assert_close(host(got), want, str(shape), **({} if bf else F32))


def test_linear_general_unaligned_rows(gpu_lib):
    # The same widths from pointers that are not aligned to four elements.
    c = wl.linear_case([40, 3], 20, 24, 36, seed=3, bf16=False)

    def off1(a):
        t = torch.empty(a.size + 1, dtype=torch.float32, device="cuda")[1:].view(a.shape)
        return t.copy_(dev_f32(a))

    got = gpu_lib.ikbo_linear(off1(c.x_cand), off1(c.w_cand), x_req=off1(c.x_req),
                              w_req=off1(c.w_req), cand_offsets=dev_i32(c.cand_offsets))
    want = ikbo.ikbo_linear(c.x_req, c.x_cand, c.w_req, c.w_cand, None, c.cand_offsets, "none")
    assert_close(host(got), want, "unaligned", **F32)


@pytest.mark.parametrize("dim", [1, 30, 32, 48, 100, 128, 250, 256])
@pytest.mark.parametrize("q_len", [1, 3])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attention_general(gpu_lib, dim, q_len, dtype):
    # Histories at the 16-key block and the 64-key round of the four waves;
    # requests that start inside a 16-row tile, one larger than a tile.
    counts, lens = [1, 2, 0, 16, 5, 40, 3, 1], [1, 15, 9, 16, 17, 64, 0, 65]
    bf = dtype == "bf16"
    c = wl.attention_case(counts, lens, 2, dim, q_len=q_len, seed=dim, bf16=bf)
    dev = dev_bf16 if bf else dev_f32
    v = c.v.copy()
    at = int(c.kv_offsets[4])
    v[at] = np.inf                            # stays inside request 4's rows
    got = host(gpu_lib.dca_attention(dev(c.q), dev(c.k), dev(v), dev_i32(c.cand_offsets),
                                     dev_i32(c.kv_offsets)))
    want = ikbo.dca_attention(c.q, c.k, c.v, c.cand_offsets, c.kv_offsets, mode="explicit")
    a, b = int(c.cand_offsets[4]), int(c.cand_offsets[5])
    assert np.all(np.isinf(got[a:b]))
    keep = np.r_[0:a, b:got.shape[0]]
    assert_close(got[keep], want[keep], f"d{dim} T{q_len}", **({} if bf else F32))


@pytest.mark.parametrize("dims", [(2, 16, 20), (3, 40, 37), (1, 256, 96)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attention_general_projection_and_residual(gpu_lib, dims, dtype):
    heads, dim, d_in = dims
    bf = dtype == "bf16"
    dev = dev_bf16 if bf else dev_f32
    c = wl.attention_case([7, 0, 30], [33, 4, 70], heads, dim, seed=dim, bf16=bf)
    n = 37
    x = wl.normal(wl.tensor_rng(1, 9, 1), (n, 1, d_in), bf16=bf)
    w = wl.normal(wl.tensor_rng(1, 9, 2), (heads * dim, d_in), std=d_in ** -0.5, bf16=bf)
    res = wl.normal(wl.tensor_rng(1, 9, 3), (n, 1, heads, dim), bf16=bf)
    got, got_sum = gpu_lib.dca_attention_proj(
        dev(x), dev(w), dev(c.k), dev(c.v), dev_i32(c.cand_offsets), dev_i32(c.kv_offsets),
        heads=heads, residual=dev(res))
    q = (x.astype(np.float64).reshape(n, d_in) @ w.astype(np.float64).T)
    q = (round_bf16(q) if bf else q).reshape(n, 1, heads, dim)
    want = ikbo.dca_attention(q, c.k, c.v, c.cand_offsets, c.kv_offsets, mode="explicit")
    assert_close(host(got), want, "proj", **({} if bf else F32))
    assert_close(host(got_sum), host(got) + res, "sum", **({} if bf else F32))


def _lane_tree(q, k, v):
    """Attention of every row over all keys in fp32 steps: a score is summed over
    the dims pairwise, the keys are taken in order."""
    d = q.shape[-1]
    s = q[:, None, :] * k[None]
    while s.shape[-1] > 1:
        s = s[..., :s.shape[-1] // 2] + s[..., s.shape[-1] // 2:]
    s = s[..., 0] * np.float32(d ** -0.5)
    m = np.full(len(q), -np.inf, np.float32)
    total, o = np.zeros(len(q), np.float32), np.zeros(q.shape, np.float32)
    for j in range(len(k)):
        new = np.maximum(m, s[:, j])
        alpha, p = np.exp(m - new), np.exp(s[:, j] - new)
        total = total * alpha + p
        o = o * alpha[:, None] + p[:, None] * v[j]
        m = new
    return o * (np.float32(1) / total)[:, None]


@pytest.mark.parametrize("dim", [32, 64, 128, 256])
@pytest.mark.parametrize("length", [5, 32])
def test_attention_general_is_as_exact_as_a_lane_tree(gpu_lib, dim, length):
    # fp32 scores summed in one chain over the dims had up to 2.5 times this
    # error. 2% for the noise of the estimate over 2,048 rows.
    rng = np.random.default_rng(dim + length)
    q, k, v = (rng.standard_normal(s).astype(np.float32)
               for s in ((2048, dim), (length, dim), (length, dim)))
    dev = dev_f32
    got = host(gpu_lib.dca_attention(dev(q)[:, None, None], dev(k)[:, None], dev(v)[:, None],
                                     dev_i32([0, len(q)]), dev_i32([0, length])))[:, 0, 0]
    s = q.astype(np.float64) @ k.T.astype(np.float64) / dim ** 0.5
    p = np.exp(s - s.max(1, keepdims=True))
    want = p @ v.astype(np.float64) / p.sum(1, keepdims=True)

    def error(y):
        return np.linalg.norm(y - want) / np.linalg.norm(want)

    assert error(got) <= 1.02 * error(_lane_tree(q, k, v).astype(np.float64))


@pytest.mark.parametrize("n_req,n,heads,q_len,dim", [
    (8, 37, 2, 1, 32), (8, 35, 1, 3, 250),          # two rows a workgroup
    (7, 37, 2, 1, 48), (9, 700, 12, 1, 16),         # sixteen: few requests, many rows
    (3, 9, 1, 1, 256)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attention_general_mapped(gpu_lib, n_req, n, heads, q_len, dim, dtype):
    # A map in any order: every row of a workgroup may be of another request.
    bf = dtype == "bf16"
    rng = np.random.default_rng(n + dim)
    lens = rng.integers(0, 70, n_req)
    lens[0], lens[-1] = 0, 17
    c = wl.attention_case([n] + [0] * (n_req - 1), lens, heads, dim, q_len=q_len, seed=dim, bf16=bf)
    ids = rng.integers(0, n_req, n).astype(np.int32)
    dev = dev_bf16 if bf else dev_f32
    got = host(gpu_lib.dca_attention_mapped(dev(c.q), dev(c.k), dev(c.v), dev_i32(ids),
                                            dev_i32(c.kv_offsets)))
    order = np.argsort(ids, kind="stable")
    off = np.concatenate([[0], np.cumsum(np.bincount(ids, minlength=n_req))])
    want = np.empty(c.q.shape)
    want[order] = ikbo.dca_attention(c.q[order], c.k, c.v, off, c.kv_offsets, mode="explicit")
    assert_close(got, want, f"R{n_req} d{dim}", **({} if bf else F32))


def test_attention_general_few_rows_a_request(gpu_lib):
    # Four rows a workgroup, rows of up to four requests in each.
    c = wl.attention_case([1, 2, 0, 3, 1, 1, 1, 2], [5, 64, 3, 17, 0, 1, 70, 33], 2, 40, seed=4,
                          bf16=False)
    got = host(gpu_lib.dca_attention(dev_f32(c.q), dev_f32(c.k), dev_f32(c.v),
                                     dev_i32(c.cand_offsets), dev_i32(c.kv_offsets)))
    want = ikbo.dca_attention(c.q, c.k, c.v, c.cand_offsets, c.kv_offsets, mode="explicit")
    assert_close(got, want, "few rows", **F32)
