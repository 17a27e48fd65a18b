"""GPU parity of tn_linear_param_gradients (gradients of sum(dY * Y) with respect to every parameter tensor)
against the fp64 oracle. Tolerance per tensor: max|g - g_ref| / max|g_ref| <= 2e-2 (bf16: intermediates and the
back-propagated gradients are rounded to bf16 between steps) or 1e-4 (fp32: sums over tokens x rows of up to 1e5
terms accumulated in fp32)."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as wl
import paper_2602_01613_amd as tn
from gpu_util import make_layer, to_dev, to_host

pytestmark = pytest.mark.gpu

GRAD_TOL = {"bf16": 2e-2, "f32": 1e-4}

CASES = [
    (tn.TN_FORMAT_TT, (2, 3, 2, 2), (2, 2, 3, 2), (1, 4, 2, 4, 1)),      # would merge at create time without the flag
    (tn.TN_FORMAT_TT, (8, 16, 8), (8, 10, 8), (1, 32, 16, 1)),
    (tn.TN_FORMAT_TT, (3, 4, 2), (2, 5, 3), (1, 3, 4, 1)),               # odd extents
    (tn.TN_FORMAT_TT, (2, 3, 2, 2), (5, 2, 3, 2), (1, 2, 5, 3, 1)),      # first step gathers from x
    (tn.TN_FORMAT_TR, (2, 3, 2), (3, 2, 2), (3, 2, 4, 3)),
    (tn.TN_FORMAT_TR, (4, 6, 4), (6, 4, 8), (8, 16, 8, 8)),
    (tn.TN_FORMAT_TR, (5,), (7,), (3, 3)),                               # a ring of one core: gradient on the bond diagonal
    (tn.TN_FORMAT_TUCKER, (4, 5), (3, 6), (2, 3, 2, 4)),
    (tn.TN_FORMAT_TUCKER, (16, 24), (8, 40), (8, 16, 8, 16)),
    (tn.TN_FORMAT_TUCKER, (3, 2, 4), (5,), (2, 2, 3, 4)),
    (tn.TN_FORMAT_DENSE, (200,), (136,), ()),
]


def _check(spec, ts, tokens, seed, flags=0, max_tokens=None, workspace_limit_bytes=0):
    rng = np.random.default_rng(seed)
    x = wl.round_to_dtype(rng.standard_normal((tokens, spec.N)), spec.dtype)
    dy = wl.round_to_dtype(rng.standard_normal((tokens, spec.M)), spec.dtype)
    layer = make_layer(spec, ts, max_tokens or tokens, workspace_limit_bytes, flags=tn.TN_FLAG_TRAINABLE | flags)
    assert layer.query(tn.TN_QUERY_NUM_MERGES) == 0
    grads = layer.param_gradients(to_dev(x, spec.dtype), to_dev(dy, spec.dtype))
    torch.cuda.synchronize()
    again = layer.param_gradients(to_dev(x, spec.dtype), to_dev(dy, spec.dtype))
    torch.cuda.synchronize()
    ref = O.param_gradients(spec.format, ts, x, dy, n_out_modes=len(spec.out_modes))
    errs = []
    for g, g2, r in zip(grads, again, ref):
        assert tuple(g.shape) == r.shape
        assert torch.equal(g, g2)                                        # fixed-order sums: same bits
        errs.append(O.rel_max_err(to_host(g), r))
    # the forward of a trainable layer is the ordinary forward
    y = to_host(layer(to_dev(x, spec.dtype)))
    assert O.rel_max_err(y, O.forward(spec.format, ts, x, n_out_modes=len(spec.out_modes))) <= (2e-2 if spec.dtype == "bf16" else 1e-5)
    layer.close()
    return errs


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_param_gradients_small_shapes(case, dtype):
    fmt, om, im, rk = CASES[case]
    spec = wl.TNSpec(fmt, dtype, tuple(om), tuple(im), tuple(rk))
    rng = np.random.default_rng(2000 + case)
    ts = [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(max(1, s[-1])), dtype) for s in spec.tensor_shapes()]
    for tokens in (1, 17, 130):
        errs = _check(spec, ts, tokens, 3000 + case * 7 + tokens)
        assert max(errs) <= GRAD_TOL[dtype], (case, tokens, errs)


def test_param_gradients_in_several_passes():
    """More tokens than the backward workspace holds: passes whose gradients are added."""
    spec = wl.TNSpec(tn.TN_FORMAT_TT, "bf16", (8, 16, 8), (8, 10, 8), (1, 32, 16, 1))
    rng = np.random.default_rng(2100)
    ts = [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(s[-1]), "bf16") for s in spec.tensor_shapes()]
    layer = make_layer(spec, ts, 100, 1 << 20, flags=tn.TN_FLAG_TRAINABLE)
    chunk = layer.query(tn.TN_QUERY_BACKWARD_CHUNK_TOKENS)
    layer.close()
    assert 0 < chunk < 100
    errs = _check(spec, ts, 100, 2101, workspace_limit_bytes=1 << 20)
    assert max(errs) <= GRAD_TOL["bf16"], errs


@pytest.mark.parametrize("i", [0, 1, 2, 3])
def test_param_gradients_baseline_configs(i):
    """The four single-layer workloads at 64 tokens (the ring at 8: its intermediates are 26 MB per token)."""
    spec, _ = wl.baseline_spec(i)
    ts = wl.make_tensors(spec, i)
    tokens = 8 if i == 3 else (16 if i == 0 else 64)
    errs = _check(spec, ts, tokens, 2200 + i)
    print(f"workload {i}: gradient rel errs {['%.2e' % e for e in errs]}", flush=True)
    assert max(errs) <= GRAD_TOL[spec.dtype], errs


def test_param_gradients_need_a_trainable_handle():
    spec, _ = wl.baseline_spec(0)
    ts = wl.make_tensors(spec, 0)
    layer = make_layer(spec, ts, 4)
    x = to_dev(wl.make_x(spec, 4, 0), "f32")
    with pytest.raises(tn.TNLinearError) as e:
        layer.param_gradients(x, x)
    assert e.value.status == -1
    layer.close()


@pytest.mark.parametrize("seed", range(30))
def test_param_gradients_random_layers(seed):
    """Seeded random layers (the draw of the random forward test, up to 2048 x 2048) against the oracle: shapes nobody
    picked by hand, so that the tile kernel meets every way of loading its operands (pieces along the columns, along
    the rows, single elements), skinny boundary cores and ragged tiles, and the plain kernel the rest."""
    from test_gpu_random import _draw
    rng = np.random.default_rng(99000 + seed)
    while True:
        spec = _draw(rng)
        if spec.M <= 2048 and spec.N <= 2048:
            break
    ts = [wl.round_to_dtype(rng.standard_normal(shp) / np.sqrt(max(1.0, 0.5 * (shp[0] + shp[-1]))), "bf16")
          for shp in spec.tensor_shapes()]
    print(f"seed {seed}: format {spec.format} out {spec.out_modes} in {spec.in_modes} ranks {spec.ranks}", flush=True)
    for tokens in (3, 70):
        errs = _check(spec, ts, tokens, 99500 + seed * 3 + tokens)
        assert max(errs) <= GRAD_TOL["bf16"], (seed, tokens, errs)


# modes of trains: in the first four one pass over dW gives the gradients of both halves
NARROW_BONDS = [((8, 10, 8, 8), (8, 16, 8, 8)),        # halves of several row panels and of whole tiles
                ((4, 4, 8, 8), (4, 4, 4, 8)),          # 256 rows (or less) against more columns
                ((4, 5, 8, 8), (4, 4, 4, 8)),          # a last panel of 64 rows
                ((8, 10, 8, 8), (4, 4, 3, 16)),        # 1280 rows, 96 tiles of columns, modes of no power of two
                ((160, 64), (8, 8))]                   # halves of one core: as two products, like a bond of 128


def narrow_bond(case, rank):
    """The train, and whether its gradients come from one pass over dW."""
    om, im = NARROW_BONDS[case]
    spec = wl.TNSpec(tn.TN_FORMAT_TT, "bf16", om, im, (1,) + tuple(rank if k == len(om) // 2 else min(rank, 32) for k in range(1, len(om))) + (1,))
    return spec, rank < 128 and len(om) == 4


@pytest.mark.parametrize("rank", [32, 64, 96, 128])
@pytest.mark.parametrize("case", range(len(NARROW_BONDS)))
def test_param_gradients_through_a_narrow_bond(case, rank):
    """Trains whose two halves' gradients come from one pass over dW (bonds of 32, 64 and 96), at the edges of its row panels and column
    ranges, and those that two products give. dW and the halves are kept to 2^-16, the sums in fp32: 2^-13 of the largest value allows for
    three such steps."""
    spec, _ = narrow_bond(case, rank)
    rng = np.random.default_rng(rank + spec.M)
    ts = [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(s[0] * s[2]), "bf16") for s in spec.tensor_shapes()]
    tokens = 1000
    layer = make_layer(spec, ts, tokens, flags=tn.TN_FLAG_TRAINABLE)
    assert 0 < layer.query(tn.TN_QUERY_GRADIENT_MATRIX_MIN_TOKENS) <= tokens
    layer.close()
    errs = _check(spec, ts, tokens, 41 + tokens)
    assert max(errs) <= 2.0 ** -13, errs


# Tucker layers and, at 40 and at 333 tokens, the products towards an out-factor's rank that read the output's gradient in runs along its
# rows: (K, columns, rows per token) of each
ROW_RUNS = [((40, 72), (24, 16), (40, 64, 16, 16), [(40, 40, 64)], [(40, 40, 64)]),                     # K below a tile of 64
            ((64, 72), (24, 16), (40, 64, 16, 16), [(64, 40, 72)], [(64, 40, 72)]),                     # at one
            ((136, 160), (24, 16), (72, 136, 8, 16), [], [(136, 72, 160), (160, 136, 72)]),             # two and three, one and two tiles of 128 columns
            ((264, 160), (24, 16), (72, 136, 8, 16), [], [(264, 72, 160), (160, 136, 72)]),
            ((264, 48), (16, 16), (40, 48, 16, 8), [(48, 48, 40)], [(48, 48, 40)]),
            ((33, 40), (16, 24), (33, 40, 16, 16), [(33, 33, 40)], [(33, 33, 40)]),                     # a K of no whole pieces
            ((40, 33), (16, 24), (40, 33, 16, 16), [], [])]                                             # an extent that allows no such runs


@pytest.mark.parametrize("case", range(len(ROW_RUNS)))
def test_input_gradients_along_row_runs(case):
    """Tucker layers whose out-factor steps read the output's gradient in runs along its rows, with rows that end inside a tile of 256."""
    om, im, rk, _, _ = ROW_RUNS[case]
    spec = wl.TNSpec(wl.FORMAT_TUCKER, "bf16", om, im, rk)
    rng = np.random.default_rng(sum(om) + rk[1])
    ts = [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(max(1, s[-1])), "bf16") for s in spec.tensor_shapes()]
    for tokens in (40, 333):
        errs = _check(spec, ts, tokens, 51 + tokens)
        assert max(errs) <= GRAD_TOL["bf16"], (tokens, errs)


# rings through dW: (rank, second in-mode) -> the cores' gradients of both halves in shared launches, or (their halves' too large) one half
# after the other
RING_CORES = {(16, 8): True, (32, 16): False}


def ring_of_cores(rank, mode):
    return wl.TNSpec(wl.FORMAT_TR, "bf16", (8, 8, 8, 8), (8, mode, 8, 8), (rank,) * 5)


@pytest.mark.parametrize("rank,mode", sorted(RING_CORES))
def test_core_gradients_of_rings(rank, mode):
    """Gradients of a ring's cores, with the launches of its two halves shared and not: dW and the halves are kept to 2^-16, as in the
    narrow bonds above."""
    spec = ring_of_cores(rank, mode)
    rng = np.random.default_rng(rank)
    ts = [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(s[0] * s[2]), "bf16") for s in spec.tensor_shapes()]
    layer = make_layer(spec, ts, 48, flags=tn.TN_FLAG_TRAINABLE)
    assert 0 < layer.query(tn.TN_QUERY_GRADIENT_MATRIX_MIN_TOKENS) <= 48
    layer.close()
    errs = _check(spec, ts, 48, 71 + rank)
    assert max(errs) <= 2.0 ** -13, errs


# (layer, tokens, workspace limit): no room for the second half's gradients beside the first's, so one half after the other
def tight_layers():
    return [(narrow_bond(1, 64)[0], 300, 6 << 20), (narrow_bond(2, 96)[0], 300, 7 << 20), (ring_of_cores(16, 8), 48, 146 << 20)]


@pytest.mark.parametrize("n", range(3))
def test_core_gradients_in_little_room(n):
    """A limit that leaves the halves' gradients one place: both halves one after the other, in two passes over the tokens for the trains, as
    exact as above."""
    spec, tokens, limit = tight_layers()[n]
    rng = np.random.default_rng(90 + n)
    ts = [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(s[0] * s[2]), "bf16") for s in spec.tensor_shapes()]
    layer = make_layer(spec, ts, tokens, limit, flags=tn.TN_FLAG_TRAINABLE)
    assert 0 < layer.query(tn.TN_QUERY_GRADIENT_MATRIX_MIN_TOKENS) <= tokens
    layer.close()
    errs = _check(spec, ts, tokens, 91 + n, workspace_limit_bytes=limit)
    assert max(errs) <= 2.0 ** -13, errs


# rings (second modes, inner bond), and the reduction (rows of threads to an element, elements a lane) of their cores' gradients: even bonds two a lane
ODD_BONDS = {(8, 8, 62): (1, 2), (8, 8, 63): (1, 1), (16, 10, 31): (4, 1)}


def ring_of_bond(m, n, inner):
    return wl.TNSpec(wl.FORMAT_TR, "bf16", (8, m, 8, 8), (8, n, 8, 8), (16, inner, 16, inner, 16))


@pytest.mark.parametrize("ring", sorted(ODD_BONDS))
def test_core_gradients_of_odd_bonds(ring):
    """Rows of an odd number of elements: added one to a lane."""
    spec = ring_of_bond(*ring)
    rng = np.random.default_rng(sum(ring))
    ts = [wl.round_to_dtype(rng.standard_normal(s) / np.sqrt(s[0] * s[2]), "bf16") for s in spec.tensor_shapes()]
    errs = _check(spec, ts, 48, 73 + sum(ring))
    assert max(errs) <= 2.0 ** -13, errs
