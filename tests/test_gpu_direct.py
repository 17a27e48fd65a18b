"""Rings and trains whose slices are made on chip (kernels/krondirect.hpp), against the oracle: every instantiation and number of steps of the
bond inside a half, shapes that fill it and that do not, calls of one token and of several, a workspace of the layer's own and a shared one."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2602_01613_amd as tn
import workloads as wl
from gpu_util import TOL, dtype_code, make_layer, to_dev, to_host

pytestmark = pytest.mark.gpu

# format, out-modes, in-modes, ranks, instantiation, steps; each is held to it by test_create_host.py
DIRECT_LAYERS = [
    (wl.FORMAT_TR, (8, 16, 8, 8), (8, 10, 8, 8), (20,) * 5, 0, 1),
    (wl.FORMAT_TR, (8, 16, 8, 8), (8, 10, 8, 8), (64, 5, 33, 7, 64), 0, 2),
    (wl.FORMAT_TR, (8, 8, 8, 8), (8, 8, 8, 8), (96, 3, 90, 11, 96), 0, 3),
    (wl.FORMAT_TR, (4, 8, 4, 8), (8, 10, 8, 8), (32,) * 5, 1, 1),
    (wl.FORMAT_TR, (4, 8, 4, 8), (8, 10, 8, 8), (48, 9, 40, 6, 48), 1, 2),
    (wl.FORMAT_TR, (8, 10, 8, 8), (8, 16, 8, 8), (24,) * 5, 2, 1),
    (wl.FORMAT_TR, (8, 10, 8, 8), (8, 16, 8, 8), (72, 5, 72, 5, 72), 2, 3),
    (wl.FORMAT_TR, (10, 16, 10, 16), (8, 10, 8, 8), (20, 6, 20, 6, 20), 3, 1),
    (wl.FORMAT_TR, (8, 10, 8, 8), (10, 16, 10, 16), (20, 9, 20, 9, 20), 4, 1),
    (wl.FORMAT_TR, (8, 10, 8, 8), (10, 16, 10, 16), (66, 4, 66, 3, 66), 4, 3),
    (wl.FORMAT_TT, (8, 10, 8, 8), (8, 16, 8, 8), (1, 32, 32, 32, 1), 2, 1),
    (wl.FORMAT_TT, (4, 8, 4, 8), (8, 10, 8, 8), (1, 32, 32, 32, 1), 1, 1),
]


@pytest.mark.parametrize("n", range(len(DIRECT_LAYERS)))
def test_slices_made_on_chip(n):
    fmt, om, im, rk, _, _ = DIRECT_LAYERS[n]
    spec = wl.TNSpec(fmt, "bf16", om, im, rk)
    ts = wl.make_tensors(spec, 4, instance=700 + n)
    rows = np.unique(np.concatenate([np.random.default_rng(n).choice(spec.M, 46, replace=False), [0, spec.M - 1]]))
    w = O.tr_dense_rows(ts, rows) if fmt == wl.FORMAT_TR else O.dense_weight(fmt, ts, len(om))[rows]
    block = torch.full((1 << 30,), 0xFF, dtype=torch.uint8, device="cuda")        # NaN wherever nothing was written
    own = make_layer(spec, ts, 16)
    shared = tn.TNLinear(fmt, dtype_code("bf16"), om, im, rk, [to_dev(t, "bf16") for t in ts], 16, workspace=block)
    for tokens in (1, 2, 3, 7):
        print(f"layer {n} tokens {tokens}", flush=True)
        x = wl.make_x(spec, tokens, 4, instance=700 + n)
        xd = to_dev(x, "bf16")
        ref = O.apply_linear(w, x)
        for layer in (own, shared):
            y = layer(xd)
            assert O.rel_max_err(to_host(y)[:, rows], ref) <= TOL["bf16"]
            assert torch.equal(layer(xd), y)
    own.close()
    shared.close()


# layers of the above that one workgroup a token walks the whole bond of where K ranges are switched off, straight to the output: of each
# instantiation that is cheaper so than the slices in memory, and whether in a shared workspace; and those that 16 tokens, the most, take
ONE_RANGE = [(0, False), (1, False), (2, False), (4, True), (5, False), (6, True), (9, False), (10, False)]
MOST_TOKENS = [(0, True), (10, True), (11, True), (11, False)]


@pytest.mark.parametrize("n,in_block,tokens,flags", [(n, b, t, tn.TN_FLAG_NO_SPLIT_K) for n, b in ONE_RANGE for t in (2, 7)] + [(n, b, 16, 0) for n, b in MOST_TOKENS])
def test_one_range_and_most_tokens(n, in_block, tokens, flags):
    fmt, om, im, rk, _, _ = DIRECT_LAYERS[n]
    spec = wl.TNSpec(fmt, "bf16", om, im, rk)
    ts = wl.make_tensors(spec, 4, instance=720 + n)
    rows = np.unique(np.concatenate([np.random.default_rng(n).choice(spec.M, 46, replace=False), [0, spec.M - 1]]))
    w = O.tr_dense_rows(ts, rows) if fmt == wl.FORMAT_TR else O.dense_weight(fmt, ts, len(om))[rows]
    block = torch.full((1 << 30,), 0xFF, dtype=torch.uint8, device="cuda") if in_block else None
    layer = tn.TNLinear(fmt, dtype_code("bf16"), om, im, rk, [to_dev(t, "bf16") for t in ts], 16, flags=flags, workspace=block)
    x = wl.make_x(spec, tokens, 4, instance=720 + n)
    xd = to_dev(x, "bf16")
    y = layer(xd)
    assert O.rel_max_err(to_host(y)[:, rows], O.apply_linear(w, x)) <= TOL["bf16"]
    assert torch.equal(layer(xd), y)
    layer.close()
