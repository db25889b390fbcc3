"""GPU parity of the tiled linear at its edges: 64 and 128 tiles, one to several
K slabs with a partial last one, rows of 8- and 16-byte alignment, maps in any
order, the residual; and the same values as the streaming kernel, bit for bit."""

import numpy as np
import pytest
import torch

from gpu_util import assert_close, dev_bf16, dev_f32, dev_i32, host
from oracle import ikbo
from oracle.bf16 import round_bf16
from paper_2607_27744_amd import ops
from paper_2607_27744_amd import workloads as wl

pytestmark = pytest.mark.gpu

# counts, k_req, k_cand, d_out: below / above 256 tiles of 128 x 128 (the tile
# switch on 256 CUs), N and D at and off tile edges, K of one slab, off the
# 32- and 64-wide slabs, the shortest, and both sides of 256 (the waves' places
# with a residual).
CASES = [
    ([1], 8, 8, 4),
    ([63, 1, 0, 64], 16, 64, 64),
    ([129, 127], 64, 72, 68),
    ([300, 0, 5], 40, 200, 132),
    ([5000, 11, 3181, 0], 64, 104, 516),
    ([2047, 6100, 45], 72, 320, 520),
    ([4001, 0, 4100], 16, 264, 644),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"N{sum(c[0])}-k{c[2]}-d{c[3]}")
@pytest.mark.parametrize("add", [False, True], ids=["plain", "residual"])
@pytest.mark.parametrize("mapped", [False, True], ids=["csr", "mapped"])
def test_tiles(gpu_lib, case, add, mapped):
    counts, kr, kc, d = case
    c = wl.linear_case(counts, kr, kc, d, seed=kc + d, bias_std=0.3, add_residual=add)
    xc = round_bf16(np.asarray(c.x_cand, np.float64) + c.x_cand_add) if add else c.x_cand
    kw = dict(x_req=dev_bf16(c.x_req), w_req=dev_bf16(c.w_req), bias=dev_f32(c.bias),
              x_cand_add=dev_bf16(c.x_cand_add) if add else None, activation="relu")
    X, W = dev_bf16(c.x_cand), dev_bf16(c.w_cand)
    m = ikbo.request_ids(c.cand_offsets)
    if mapped:
        m = np.random.default_rng(d).permutation(m)
        ids = m.astype(np.int32)
        ids[0] = len(counts) + 7                       # clamped to the last request
        m = np.minimum(ids, len(counts) - 1)
        got = gpu_lib.ikbo_linear_mapped(X, W, cand_request_ids=dev_i32(ids), **kw)
    else:
        got = gpu_lib.ikbo_linear(X, W, cand_offsets=dev_i32(c.cand_offsets), **kw)
    want = ikbo.ikbo_linear(c.x_req, xc, c.w_req, c.w_cand, c.bias, None, "relu", request_map=m)
    assert_close(host(got), round_bf16(want), str(case))


@pytest.mark.parametrize("counts,kc,d", [([300, 0, 211], 64, 256), ([5000, 3192], 128, 516),
                                         ([20000, 9000, 3768], 192, 512)],
                         ids=["64-tiles", "128-tiles", "streaming"])
@pytest.mark.parametrize("act", ["relu", "none"])
def test_same_values_as_the_streaming_kernel(gpu_lib, counts, kc, d, act):
    # The combined call always runs the streaming candidate kernel; the
    # separate call picks by size. Both sum k in order and add the request row
    # after the products. NaN and infinities travel alike.
    c = wl.linear_case(counts, 32, kc, d, seed=d, bias_std=0.2)
    X = dev_bf16(c.x_cand)
    X[1, 0], X[3, 1] = float("nan"), float("inf")
    args = (dev_bf16(c.x_req), X, dev_bf16(c.w_req), dev_bf16(c.w_cand), dev_i32(c.cand_offsets))
    _, stream = gpu_lib.ikbo_linear_combined(*args, b_cand=dev_f32(c.bias), activation=act)
    got = gpu_lib.ikbo_linear(X, args[3], x_req=args[0], w_req=args[2], cand_offsets=args[4],
                              bias=dev_f32(c.bias), activation=act)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), stream.view(torch.int16))


@pytest.mark.parametrize("kc", [448, 512])
@pytest.mark.parametrize("last", [1047, 1049], ids=["tiled", "streaming"])
def test_both_sides_of_half_a_round(gpu_lib, kc, last):
    # 2,048 and 2,050 x 4,096: half of one round of 256 x 256 tiles on 256 CUs
    # and just more. (tests/test_linear_rule.py: which kernel that takes.)
    c = wl.linear_case([1000, 0, last, 1], 24, kc, 4096, seed=kc, bias_std=0.2)
    args = (dev_bf16(c.x_req), dev_bf16(c.x_cand), dev_bf16(c.w_req), dev_bf16(c.w_cand),
            dev_i32(c.cand_offsets))
    _, stream = gpu_lib.ikbo_linear_combined(*args, b_cand=dev_f32(c.bias), activation="relu")
    got = gpu_lib.ikbo_linear(args[1], args[3], x_req=args[0], w_req=args[2],
                              cand_offsets=args[4], bias=dev_f32(c.bias), activation="relu")
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), stream.view(torch.int16))
    rows = np.array([0, 255, 256, 999, 1000, 2046, last + 999, last + 1000])
    want = ikbo.ikbo_linear(c.x_req, c.x_cand[rows], c.w_req, c.w_cand, c.bias, None, "relu",
                            request_map=ikbo.request_ids(c.cand_offsets)[rows])
    assert_close(host(got)[rows], round_bf16(want), f"k{kc}")
