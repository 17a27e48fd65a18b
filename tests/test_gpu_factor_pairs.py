"""Both factors on a side of a Tucker core in one launch with a workgroup to a token: against the oracle, and against one launch per step."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as wl
import paper_2602_01613_amd as tn
from gpu_util import TOL, make_layer, run_layer, to_dev, to_host

pytestmark = pytest.mark.gpu

# out-modes, in-modes, ranks
FACTOR_PAIRS = [((160, 160), (64, 80), (96, 96, 16, 16)),        # the largest; in-factors padded to a k-step
                ((16, 16), (16, 16), (16, 16, 16, 16)),          # the smallest
                ((64, 128), (160, 144), (64, 96, 32, 16)),       # the edge of the narrow form; in-factors on the wide one
                ((80, 64), (64, 128), (80, 48, 48, 16)),         # past it in the first mode
                ((80, 64), (128, 64), (80, 48, 16, 48)),         # the outer in-mode first: x is gathered
                ((64, 144), (48, 112), (32, 64, 32, 64)),        # so it is, and the inner out-factor comes first
                ((32, 176), (64, 128), (32, 32, 32, 32)),        # a mode too long
                ((160, 160), (64, 72), (112, 32, 16, 16)),       # a rank too large; no whole tiles
                ((4, 8, 16), (32, 48), (4, 8, 16, 32, 32))]      # three out-modes


def factor_pair(case):
    om, im, rk = FACTOR_PAIRS[case]
    return wl.TNSpec(wl.FORMAT_TUCKER, "bf16", om, im, rk)


def pair_layer(case, instance=0):
    spec = factor_pair(case)
    rng = np.random.default_rng(500 + 10 * case + instance)
    return spec, [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(max(1, s[-1])), "bf16") for s in spec.tensor_shapes()]


@pytest.mark.parametrize("flags", [0, tn.TN_FLAG_TRANSPOSE])
@pytest.mark.parametrize("case", range(len(FACTOR_PAIRS)))
def test_factor_pairs(case, flags):
    """A token; more items than the kernel that spreads a token takes; more tokens than workgroups fit the chip. The steps round the same
    values, so what differs from them is the order of fp32 sums and by it a rounding of 2^-9 of some values."""
    spec, ts = pair_layer(case)
    for tokens in (1, 70, 1100):
        n = spec.M if flags else spec.N
        x = wl.round_to_dtype(np.random.default_rng(case * 7 + tokens).standard_normal((tokens, n)), "bf16")
        y = run_layer(spec, ts, x, flags=flags)
        sep = run_layer(spec, ts, x, flags=flags | tn.TN_FLAG_NO_CHAIN2)
        assert O.rel_max_err(y, sep) <= 1e-2, (case, tokens)
        if not flags and tokens < 100:
            ref = O.forward(spec.format, ts, x, n_out_modes=len(spec.out_modes))
            assert O.rel_max_err(y, ref) <= TOL["bf16"], (case, tokens)


@pytest.mark.parametrize("case", [0, 3])
def test_factor_pairs_of_two_layers(case):
    """Two layers in one call have the bits of each by itself."""
    spec, ta = pair_layer(case)
    _, tb = pair_layer(case, 1)
    for tokens in (1, 40, 700):
        a, b = make_layer(spec, ta, tokens), make_layer(spec, tb, tokens)
        x = to_dev(wl.round_to_dtype(np.random.default_rng(tokens).standard_normal((tokens, spec.N)), "bf16"), "bf16")
        ya, yb = tn.forward2(a, b, x)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(ya), to_host(a(x))) and np.array_equal(to_host(yb), to_host(b(x)))
        a.close()
        b.close()


# out-modes, in-modes, ranks; the forms (side, A, B, P, Q / 32) that 70, 600 and 2100 tokens take: each is held to them by test_create_host.py, and all
# twelve are among them
FORM_PAIRS = [((80, 64), (64, 64), (48, 32, 48, 64), [[("in", 2, 4, 2, 3)]] * 3),
              ((64, 64), (80, 64), (32, 32, 48, 16), [[("out", 2, 3, 2, 3), ("out", 2, 3, 2, 2)]] * 3),
              ((80, 80), (64, 80), (32, 32, 48, 48), [[("in", 2, 3, 2, 2), ("out", 5, 5, 1, 1)]] * 3),
              ((160, 160), (64, 128), (96, 96, 48, 16), [[("in", 2, 4, 2, 2), ("out", 5, 5, 3, 3)]] * 3),
              ((64, 128), (160, 160), (48, 48, 16, 96), [[("out", 2, 4, 2, 3)]] * 3),
              ((16, 16), (160, 160), (16, 16, 96, 96), [[("in", 5, 5, 3, 3)]] * 3),
              ((112, 96), (128, 128), (48, 48, 32, 16), [[("in", 5, 5, 1, 1)]] * 3),
              ((112, 112), (48, 112), (48, 48, 16, 32), [[("out", 5, 5, 2, 2)]] * 3),
              ((64, 80), (112, 112), (32, 32, 64, 64), [[("in", 5, 5, 2, 2), ("out", 2, 3, 2, 2)]] * 3),
              # between 512 and 2048 tokens, or from 512 on, the small ones are a wave's; out-factors from one wide rank always
              ((160, 160), (64, 80), (32, 32, 32, 32), [[("in", 2, 3, 2, 2), ("out", 5, 5, 1, 1)], [("out", 5, 5, 1, 1)], [("in", 2, 3, 2, 2), ("out", 5, 5, 1, 1)]]),
              ((32, 32), (80, 80), (16, 16, 16, 16), [[("in", 5, 5, 1, 1), ("in", 2, 3, 2, 2)], [], []]),
              ((128, 64), (16, 16), (96, 32, 16, 16), [[], [], []])]


@pytest.mark.parametrize("case", range(len(FORM_PAIRS)))
def test_forms_of_factor_pairs(case):
    """As test_factor_pairs, for each form of the two kernels and at the edges of the counts that they take."""
    om, im, rk, _ = FORM_PAIRS[case]
    spec = wl.TNSpec(wl.FORMAT_TUCKER, "bf16", om, im, rk)
    rng = np.random.default_rng(560 + case)
    ts = [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(max(1, s[-1])), "bf16") for s in spec.tensor_shapes()]
    for tokens in (70, 600, 2100):
        x = wl.round_to_dtype(np.random.default_rng(case * 7 + tokens).standard_normal((tokens, spec.N)), "bf16")
        y = run_layer(spec, ts, x, max_tokens=2100)
        assert O.rel_max_err(y, run_layer(spec, ts, x, flags=tn.TN_FLAG_NO_CHAIN2, max_tokens=2100)) <= 1e-2, (case, tokens)
        if tokens < 100:
            assert O.rel_max_err(y, O.forward(spec.format, ts, x, n_out_modes=len(om))) <= TOL["bf16"], (case, tokens)
