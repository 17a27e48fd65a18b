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
PINNED = tn.TN_FLAG_NO_SMALL_CHAIN | (12 << tn.TN_FLAG_VARIANT_SHIFT)      # the matrix-product kernel, at any number of rows


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


# rows that end inside the tiles of 160 x 128 of the form for K of one and two tiles, one short of their end and one past it
SHORT_K_ROWS = {1032: (8000, 9601), 5128: (1281, 1599, 1600, 1601), 10248: (799, 801, 959, 960, 961, 2560), 20488: (319, 320, 639)}


@pytest.mark.parametrize("n_in", [64, 128])
@pytest.mark.parametrize("n_out", sorted(SHORT_K_ROWS))
def test_short_k_tile_edges(n_in, n_out):
    """K of one and two tiles against many columns: the form that loads all of K at once, with rows and columns that end inside its tiles
    of 160 x 128."""
    rng = np.random.default_rng(n_in + n_out)
    rows_of = SHORT_K_ROWS[n_out]
    x = wl.round_to_dtype(rng.standard_normal((max(rows_of), n_in)), "bf16")
    spec = wl.TNSpec(wl.FORMAT_DENSE, "bf16", (n_out,), (n_in,), ())
    w = wl.round_to_dtype(rng.standard_normal((n_out, n_in)) / np.sqrt(n_in), "bf16")
    layer = make_layer(spec, [w], max(rows_of), flags=PINNED)
    xd = to_dev(x, "bf16")
    for rows in rows_of:
        ref = x[:rows] @ w.T
        y = to_host(layer(xd[:rows].contiguous()))
        assert np.max(np.abs(y - ref)) <= 2.0 ** -8 * np.max(np.abs(ref)) + 1e-3, rows
    layer.close()


# (rows and columns of the tile in units of 32, its LDS stages), columns, rows of a call, K: the fewest K tiles with which the tile is
# chosen (the wide ones with three stages pay from 9 on) and the two numbers after it, so that the last tile falls on each of its
# stages; the last K ends in the middle of a tile
TILE_CALLS = [((2, 2, 4), 4104, 66, (192, 256, 320, 224)), ((2, 4, 3), 136, 8215, (64, 128, 96)), ((2, 4, 3), 8200, 66, (192, 256, 320, 160)),
              ((3, 4, 2), 520, 6752, (64, 128, 192, 160)), ((4, 4, 2), 520, 9995, (192, 256, 160)), ((5, 4, 2), 776, 9611, (192, 256, 160)),
              ((2, 8, 3), 8200, 199, (832, 896, 960, 800)), ((3, 8, 3), 8200, 66, (3904, 3968, 4032, 3872)), ((4, 8, 3), 8200, 808, (704, 768, 832, 672)),
              ((5, 8, 3), 8200, 908, (704, 768, 832, 672)), ((6, 4, 3), 8200, 451, (640, 704, 768, 608)), ((8, 4, 3), 8200, 678, (576, 640, 704, 544)),
              ((6, 8, 2), 14344, 641, (192, 256, 160)), ((7, 8, 2), 1032, 9995, (192, 256, 160)), ((8, 8, 2), 1544, 8215, (192, 256, 160))]


@pytest.mark.parametrize("case", range(len(TILE_CALLS)))
def test_every_tile_at_its_fewest_k_tiles(case):
    """Each tile size where its first loads and its last ones meet, K of whole tiles and not. Tolerance as above."""
    _, n_out, rows, ks = TILE_CALLS[case]
    rng = np.random.default_rng(case)
    for n_in in ks:
        x = wl.round_to_dtype(rng.standard_normal((rows, n_in)), "bf16")
        w = wl.round_to_dtype(rng.standard_normal((n_out, n_in)) / np.sqrt(n_in), "bf16")
        layer = make_layer(wl.TNSpec(wl.FORMAT_DENSE, "bf16", (n_out,), (n_in,), ()), [w], rows, flags=PINNED)
        y, ref = to_host(layer(to_dev(x, "bf16"))), x @ w.T
        layer.close()
        assert np.max(np.abs(y - ref)) <= 2.0 ** -8 * np.max(np.abs(ref)) + 1e-3, n_in
