"""The matrix-product step kernel (wide bf16 steps with a plain input, more than 64 rows) against the fp64 product, at the
edges of its tiles. Tolerance: inputs are exact in bf16, sums are fp32 over K terms (relative error below K * 2^-24 of the
sum of magnitudes, 1e-3 of the largest result at K = 2304), so one bf16 rounding of the result dominates: 2^-8 of the
largest value, doubled for the two roundings of a Tucker chain's other steps where there are any."""
import numpy as np
import pytest

import oracle as O
import workloads as wl
import paper_2602_01613_amd as tn
from gpu_util import make_layer, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in,n_out", [(64, 40), (128, 129), (192, 264), (2304, 328), (320, 1032), (704, 2056)])
def test_dense_tile_edges(n_in, n_out):
    """K of one tile, two, and many; columns that end inside a tile of 128 or of 256; rows just below, at and above every
    tile height (multiples of 32), from the smallest count the kernel takes; results that do not depend on the rows around
    them."""
    spec = wl.TNSpec(wl.FORMAT_DENSE, "bf16", (n_out,), (n_in,), ())
    rng = np.random.default_rng(n_in + n_out)
    w = wl.round_to_dtype(rng.standard_normal((n_out, n_in)) / np.sqrt(n_in), "bf16")
    x = wl.round_to_dtype(rng.standard_normal((1030, n_in)), "bf16")
    ref = x @ w.T
    layer = make_layer(spec, [w], 1030)
    if n_out % 8 == 0:
        assert layer.query(tn.TN_QUERY_STEP_BASE + 5) == 12
    xd = to_dev(x, "bf16")
    for rows in (65, 95, 96, 97, 128, 159, 161, 224, 255, 257, 320, 513, 1030):
        y = to_host(layer(xd[:rows].contiguous()))
        assert np.max(np.abs(y - ref[:rows])) <= 2.0 ** -8 * np.max(np.abs(ref[:rows])) + 1e-3, (rows, n_in, n_out)
    layer.close()


@pytest.mark.parametrize("k_tiles", [1, 2, 3, 4, 5, 7])
def test_k_tiles_and_stages(k_tiles):
    """As many K tiles as the LDS has stages (two to four), fewer and more, for the tiles that rows and columns of these numbers lead to."""
    n_in = 64 * k_tiles
    rng = np.random.default_rng(k_tiles)
    x = wl.round_to_dtype(rng.standard_normal((2600, n_in)), "bf16")
    xd = to_dev(x, "bf16")
    for n_out in (64, 1032, 5128):
        spec = wl.TNSpec(wl.FORMAT_DENSE, "bf16", (n_out,), (n_in,), ())
        w = wl.round_to_dtype(rng.standard_normal((n_out, n_in)) / np.sqrt(n_in), "bf16")
        ref = x @ w.T
        layer = make_layer(spec, [w], 2600, flags=tn.TN_FLAG_NO_SMALL_CHAIN | (12 << tn.TN_FLAG_VARIANT_SHIFT))
        for rows in (70, 200, 300, 500, 777, 1030, 1500, 2600):
            y = to_host(layer(xd[:rows].contiguous()))
            assert np.max(np.abs(y - ref[:rows])) <= 2.0 ** -8 * np.max(np.abs(ref[:rows])) + 1e-3, (rows, n_in, n_out)
        layer.close()


@pytest.mark.parametrize("n_in,n_out", [(96, 264), (160, 510), (288, 1023), (1056, 1000), (5152, 520), (8192, 511), (2336, 4095)])
def test_k_of_half_a_tile_and_outputs_one_by_one(n_in, n_out):
    """K that ends in the middle of a tile of 64 (one tile, two, many, several ranges), with infinities in the rows that follow: what
    lies behind a row must not reach it. Columns that allow no aligned pieces, from 256 on."""
    spec = wl.TNSpec(wl.FORMAT_DENSE, "bf16", (n_out,), (n_in,), ())
    rng = np.random.default_rng(n_in + n_out)
    w = wl.round_to_dtype(rng.standard_normal((n_out, n_in)) / np.sqrt(n_in), "bf16")
    x = wl.round_to_dtype(rng.standard_normal((1030, n_in)), "bf16")
    ref = x @ w.T
    layer = make_layer(spec, [w], 1030)
    assert layer.query(tn.TN_QUERY_STEP_BASE + 5) == 12
    xd = to_dev(x, "bf16")
    for rows in (64, 65, 97, 128, 161, 257, 513, 1030):
        y = to_host(layer(xd[:rows].contiguous()))
        assert np.max(np.abs(y - ref[:rows])) <= 2.0 ** -8 * np.max(np.abs(ref[:rows])) + 1e-3, (rows, n_in, n_out)
    odd = xd.clone()
    odd[1::2] = float("inf")
    y = to_host(layer(odd))[0::2]
    assert np.max(np.abs(y - ref[0::2])) <= 2.0 ** -8 * np.max(np.abs(ref)) + 1e-3
    layer.close()


@pytest.mark.parametrize("n_out", [1024, 4104])
def test_short_k_between_the_two_kernels(n_out):
    """K = 1024: row counts on both sides of where the split-K kernel in one range gives way to the tiles, and back."""
    spec = wl.TNSpec(wl.FORMAT_DENSE, "bf16", (n_out,), (1024,), ())
    rng = np.random.default_rng(n_out)
    w = wl.round_to_dtype(rng.standard_normal((n_out, 1024)) / 32, "bf16")
    x = wl.round_to_dtype(rng.standard_normal((520, 1024)), "bf16")
    ref = x @ w.T
    layer = make_layer(spec, [w], 520)
    xd = to_dev(x, "bf16")
    for rows in (64, 65, 100, 128, 129, 320, 321, 385, 460, 512, 513, 520):
        y = to_host(layer(xd[:rows].contiguous()))
        assert np.max(np.abs(y - ref[:rows])) <= 2.0 ** -8 * np.max(np.abs(ref[:rows])) + 1e-3, (rows, n_out)
    layer.close()


@pytest.mark.parametrize("om,im,rk,last", [((72, 8), (16, 64), (1, 64, 1), (8, 1024, 72)),           # 8 rows a token
                                           ((160, 160), (8, 16), (1, 64, 1), (160, 512, 160)),
                                           ((104, 8, 8), (8, 8, 8), (1, 64, 64, 1), (64, 512, 104))])
@pytest.mark.parametrize("tokens", [9, 65, 130, 331])
def test_outputs_along_the_rows(om, im, rk, last, tokens):
    """A last step whose output runs along its rows (stores of 8 rows), rows of several tokens in one tile, tokens that end inside
    one, columns that end inside a tile."""
    spec = wl.TNSpec(wl.FORMAT_TT, "bf16", om, im, rk)
    rng = np.random.default_rng(tokens)
    ts = [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(s[0] * s[2]), "bf16") for s in spec.tensor_shapes()]
    flags = tn.TN_FLAG_NO_MERGE | tn.TN_FLAG_NO_SMALL_CHAIN | tn.TN_FLAG_NO_PAIR_CHAIN
    layer = make_layer(spec, ts, tokens, flags=flags)
    step = tn.TN_QUERY_STEP_BASE + 10 * (len(om) - 1)
    assert layer.query(tn.TN_QUERY_NUM_STEPS) == len(om) and layer.query(step + 5) == 12
    assert tuple(layer.query(step + f) for f in range(3)) == last
    x = wl.round_to_dtype(rng.standard_normal((tokens, spec.N)), "bf16")
    err = O.rel_max_err(to_host(layer(to_dev(x, "bf16"))), O.forward(spec.format, ts, x, n_out_modes=len(om)))
    layer.close()
    assert err <= 2e-2


@pytest.mark.parametrize("rows", [65, 129, 200])
def test_ranges_of_k(rows):
    """Few tiles and a long K: partial sums of several ranges, the last one shorter, equal to the single range up to the
    rounding of the result; with the split kernels switched off the same launch runs as one range."""
    spec = wl.TNSpec(wl.FORMAT_DENSE, "bf16", (512,), (6976,), ())
    rng = np.random.default_rng(rows)
    w = wl.round_to_dtype(rng.standard_normal((512, 6976)) / np.sqrt(6976), "bf16")
    x = wl.round_to_dtype(rng.standard_normal((rows, 6976)), "bf16")
    ref = x @ w.T
    for flags in (0, tn.TN_FLAG_NO_SPLIT_K):
        layer = make_layer(spec, [w], rows, flags=flags)
        a = to_host(layer(to_dev(x, "bf16")))
        b = to_host(layer(to_dev(x, "bf16")))
        layer.close()
        assert np.array_equal(a, b)
        assert np.max(np.abs(a - ref)) <= 2.0 ** -8 * np.max(np.abs(ref)) + 1e-3


@pytest.mark.parametrize("n_in", [64, 128])
@pytest.mark.parametrize("n_out", [520, 10248])
def test_short_k_tile_edges(n_in, n_out):
    """K of one and two tiles against many columns: the form that loads all of K at once, with rows and columns that end inside its tiles
    of 160 x 128."""
    rng = np.random.default_rng(n_in + n_out)
    x = wl.round_to_dtype(rng.standard_normal((8000, n_in)), "bf16")
    spec = wl.TNSpec(wl.FORMAT_DENSE, "bf16", (n_out,), (n_in,), ())
    w = wl.round_to_dtype(rng.standard_normal((n_out, n_in)) / np.sqrt(n_in), "bf16")
    layer = make_layer(spec, [w], 8000, flags=tn.TN_FLAG_NO_SMALL_CHAIN | (12 << tn.TN_FLAG_VARIANT_SHIFT))
    xd = to_dev(x, "bf16")
    for rows in (159, 161, 1119, 1441, 8000 if n_out < 1000 else 2560):
        ref = x[:rows] @ w.T
        y = to_host(layer(xd[:rows].contiguous()))
        assert np.max(np.abs(y - ref)) <= 2.0 ** -8 * np.max(np.abs(ref)) + 1e-3, rows
    layer.close()
