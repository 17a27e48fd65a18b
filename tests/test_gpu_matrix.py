"""Calls of many tokens of trains and rings in the order that contracts the factors with each other first
(TN_QUERY_MATRIX_MIN_TOKENS) against the fp64 oracle. Tolerance as for every bf16 layer: 2e-2 of the largest value, where one
rounding of 2^-9 each for the halves, for W and for the result leave 3e-3."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as wl
import paper_2602_01613_amd as tn
from gpu_util import TOL, make_layer, to_dev, to_host

pytestmark = pytest.mark.gpu

CASES = [
    # (format, out modes, in modes, ranks, flags)
    (tn.TN_FORMAT_TR, (8, 10, 8, 8), (8, 10, 8, 8), (16,) * 5, 0),                          # halves of 256 values of the bonds
    (tn.TN_FORMAT_TR, (8, 10, 8, 8), (8, 10, 8, 8), (16, 24, 16, 8, 16), 0),                # bonds of different sizes
    (tn.TN_FORMAT_TR, (4, 8, 4, 8), (8, 10, 8, 8), (32,) * 5, tn.TN_FLAG_TRANSPOSE),
    (tn.TN_FORMAT_TR, (40, 8, 8), (8, 8, 40), (16, 32, 16, 16), 0),                         # three cores: a half of one, kept
    (tn.TN_FORMAT_TT, (8, 10, 8, 8), (8, 10, 8, 8), (1, 64, 96, 64, 1), tn.TN_FLAG_TRAINABLE),   # a bond of 96, laid out as 128
    (tn.TN_FORMAT_TT, (16, 8, 8), (8, 10, 16), (1, 128, 72, 1), tn.TN_FLAG_TRAINABLE),      # a bond of 72, a half of one core
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_factors_first(case):
    fmt, om, im, rk, flags = CASES[case]
    spec = wl.TNSpec(fmt, "bf16", om, im, rk)
    ts = wl.make_tensors(spec, 500 + case)
    w = O.dense_weight(fmt, ts, len(om))
    if flags & tn.TN_FLAG_TRANSPOSE:
        w = w.T
    layer = make_layer(spec, ts, 4200, flags=flags)
    first = layer.query(tn.TN_QUERY_MATRIX_MIN_TOKENS)
    assert 0 < first <= 4200, first
    rng = np.random.default_rng(case)
    again = None
    for tokens in (first, first + 1, 1, 4200, 4201, 4200):          # the largest a layer is made for, and beyond; a small call between
        x = wl.round_to_dtype(rng.standard_normal((tokens, w.shape[1])), "bf16") if tokens != 4200 or again is None else again[0]
        yd = layer(to_dev(x, "bf16"))
        assert O.rel_max_err(to_host(yd), O.apply_linear(w, x)) <= TOL["bf16"], (case, tokens)
        if tokens == 4200:
            if again is None:
                again = (x, yd.clone())
            else:
                assert torch.equal(yd, again[1])                    # fixed-order sums, nothing left over from the calls between
    layer.close()


def test_ranges_of_token_counts():
    """Where the other order's price is a staircase (train 25600 -> 5120, rank 64), the order of a call follows its token count:
    both sides of every change agree with the layer that never takes this order (two bf16 results, each within the
    tolerance of test_factors_first of the same numbers)."""
    spec = wl.stack_spec(wl.FORMAT_TT, 25600, 5120, 64)
    ts = wl.make_tensors(spec, 510)
    layer = make_layer(spec, ts, 4000)
    plain = make_layer(spec, ts, 4000, flags=tn.TN_FLAG_NO_LAZY_MERGE)
    taken = [layer.query(tn.TN_QUERY_MATRIX_TOKENS_BASE + t) for t in range(4001)]
    first = layer.query(tn.TN_QUERY_MATRIX_MIN_TOKENS)
    assert not any(taken[:first or 4001]) and (not first or taken[first])
    assert not any(plain.query(tn.TN_QUERY_MATRIX_TOKENS_BASE + t) for t in (1, 64, 4000))
    changes = [t for t in range(1, 4001) if taken[t] != taken[t - 1]]
    x = wl.make_x(spec, max(changes + [64]), 510)
    xd = to_dev(x, "bf16")
    for t in sorted({1, 64} | set(changes) | {c - 1 for c in changes}):
        a, b = to_host(layer(xd[:t].contiguous())), to_host(plain(xd[:t].contiguous()))
        assert O.rel_max_err(a, b) <= TOL["bf16"], t
    layer.close()
    plain.close()


def test_shared_block_and_graph():
    """W and the halves in a caller's block that another layer uses between the calls; the same calls as a HIP graph, replayed."""
    specs = [wl.TNSpec(wl.FORMAT_TR, "bf16", (8, 10, 8, 8), (8, 10, 8, 8), (16,) * 5),
             wl.TNSpec(wl.FORMAT_TT, "bf16", (8, 10, 8, 8), (8, 10, 8, 8), (1, 64, 96, 64, 1))]
    block = torch.empty(256 << 20, dtype=torch.uint8, device="cuda")
    layers, refs = [], []
    for n, spec in enumerate(specs):
        ts = wl.make_tensors(spec, 520 + n)
        refs.append(O.dense_weight(spec.format, ts, 4))
        layers.append(tn.TNLinear(spec.format, tn.TN_DTYPE_BF16, spec.out_modes, spec.in_modes, spec.ranks,
                                  [to_dev(t, "bf16") for t in ts], 3000, workspace=block))
        assert layers[-1].query(tn.TN_QUERY_WORKSPACE_BYTES) == 0
    assert 0 < layers[0].query(tn.TN_QUERY_MATRIX_MIN_TOKENS) <= 3000
    xd = torch.empty((3000, 5120), dtype=torch.bfloat16, device="cuda")
    ys = [torch.empty((3000, 5120), dtype=torch.bfloat16, device="cuda") for _ in specs]
    rng = np.random.default_rng(9)

    def run():
        for layer, y in zip(layers, ys):
            layer.forward(xd, out=y)

    run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for _ in range(3):
        x = wl.round_to_dtype(rng.standard_normal((3000, 5120)), "bf16")
        xd.copy_(to_dev(x, "bf16"))
        graph.replay()
        torch.cuda.synchronize()
        got = [y.clone() for y in ys]
        run()
        torch.cuda.synchronize()
        for g, y, w in zip(got, ys, refs):
            assert torch.equal(g, y)
            assert O.rel_max_err(to_host(y), O.apply_linear(w, x)) <= TOL["bf16"]
    for layer in layers:
        layer.close()


def test_no_room_for_w():
    """A workspace too small for W: such calls run as before."""
    spec = wl.TNSpec(wl.FORMAT_TR, "bf16", (8, 10, 8, 8), (8, 10, 8, 8), (16,) * 5)
    ts = wl.make_tensors(spec, 530)
    layer = make_layer(spec, ts, 300, workspace_limit_bytes=40 << 20)
    assert layer.query(tn.TN_QUERY_MATRIX_MIN_TOKENS) == 0
    x = wl.make_x(spec, 300, 530)
    assert O.rel_max_err(to_host(layer(to_dev(x, "bf16"))), O.apply_linear(O.dense_weight(spec.format, ts, 4), x)) <= TOL["bf16"]
    layer.close()


GRAD_CASES = [
    # (format, out modes, in modes, ranks, flags)
    (tn.TN_FORMAT_TT, (4, 8, 4, 8), (8, 10, 8, 8), (1, 64, 64, 64, 1), 0),
    (tn.TN_FORMAT_TT, (4, 8, 4, 8), (8, 8, 8, 8), (1, 64, 96, 64, 1), tn.TN_FLAG_TRANSPOSE),
    (tn.TN_FORMAT_TT, (16, 8, 8), (8, 8, 16), (1, 64, 72, 1), 0),                   # a half of one core: its gradient is the first product's
    (tn.TN_FORMAT_TR, (4, 8, 4, 8), (8, 8, 8, 8), (16, 16, 8, 16, 16), 0),
    (tn.TN_FORMAT_TR, (8, 8, 16), (8, 16, 8), (16, 16, 8, 16), 0),
    (tn.TN_FORMAT_DENSE, (1032,), (704,), (), 0),                                   # columns that end inside a tile
]


@pytest.mark.parametrize("case", range(len(GRAD_CASES)))
def test_gradients_through_dw(case):
    """Gradients of many tokens (a padded range, several ranges of tokens, one more than the layer is made for) against the
    oracle; a skipped tensor; the same bits twice. Tolerance as in test_gpu_gradients."""
    fmt, om, im, rk, flags = GRAD_CASES[case]
    spec = wl.TNSpec(fmt, "bf16", om, im, rk)
    rng = np.random.default_rng(540 + case)
    ts = [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(max(1, s[-1])), "bf16") for s in spec.tensor_shapes()]
    layer = make_layer(spec, ts, 1000, flags=tn.TN_FLAG_TRAINABLE | flags)
    assert layer.query(tn.TN_QUERY_BACKWARD_CHUNK_TOKENS) == 1024          # through dW: whole ranges of 64
    for tokens in (65, 1000, 1025):
        x = wl.round_to_dtype(rng.standard_normal((tokens, layer.N)), "bf16")
        dy = wl.round_to_dtype(rng.standard_normal((tokens, layer.M)), "bf16")
        xd, dyd = to_dev(x, "bf16"), to_dev(dy, "bf16")
        got = layer.param_gradients(xd, dyd)
        ref = O.param_gradients(fmt, ts, dy if flags else x, x if flags else dy, n_out_modes=len(om))
        for g, r in zip(got, ref):
            assert O.rel_max_err(to_host(g), r) <= 2e-2, (case, tokens)
        for g, a in zip(got, layer.param_gradients(xd, dyd)):
            assert torch.equal(g, a)
        # only the last tensor's
        last = torch.full_like(got[-1], float("nan"))
        tn.binding.tn_linear_param_gradients(layer._handle, xd.data_ptr(), dyd.data_ptr(), [None] * (len(ts) - 1) + [last.data_ptr()],
                                             tokens, torch.cuda.current_stream().cuda_stream)
        assert torch.equal(last, got[-1])
    layer.close()


@pytest.mark.parametrize("mean", [0.0, 1.0, 5.0])
@pytest.mark.parametrize("case", range(len(GRAD_CASES)))
def test_gradients_keep_what_averages_out_over_tokens(case, mean):
    """Activations and output gradients with a component common to all tokens, as in fine-tuning: the sum over tokens has to be
    held to more than bf16. Relative 2-norm error; every product of a sum leaves at most 2 * 2^-16 (the low part's rounding, and the
    product of two low parts) = 3e-5 of its terms, three products in a row 1e-4. (Rounded to bf16 the sum left 2.8e-3, and the
    steps that round per token leave 1e-4 to 3e-4 where there is such a component.)"""
    fmt, om, im, rk, flags = GRAD_CASES[case]
    spec = wl.TNSpec(fmt, "bf16", om, im, rk)
    rng = np.random.default_rng(560 + case)
    ts = [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(max(1, s[-1])), "bf16") for s in spec.tensor_shapes()]
    layer = make_layer(spec, ts, 1000, flags=tn.TN_FLAG_TRAINABLE | flags)
    assert layer.query(tn.TN_QUERY_BACKWARD_CHUNK_TOKENS) == 1024
    x = wl.round_to_dtype(rng.standard_normal((1025, layer.N)) + mean * rng.choice([-1.0, 1.0], layer.N), "bf16")
    dy = wl.round_to_dtype(rng.standard_normal((1025, layer.M)) + mean * rng.choice([-1.0, 1.0], layer.M), "bf16")
    for tokens in (1000, 1025):
        got = layer.param_gradients(to_dev(x[:tokens], "bf16"), to_dev(dy[:tokens], "bf16"))
        ref = O.param_gradients(fmt, ts, dy[:tokens] if flags else x[:tokens], x[:tokens] if flags else dy[:tokens], n_out_modes=len(om))
        for n, (g, r) in enumerate(zip(got, ref)):
            err = np.linalg.norm(to_host(g) - r) / np.linalg.norm(r)
            assert err <= 1e-4, (case, tokens, n, err)
    layer.close()
