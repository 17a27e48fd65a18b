"""tn_linear_create on a HIP runtime of the host (fake_hip.cpp): what a layer falls back to when memory is short, and what it holds."""
import json
import os
import re
import subprocess
import sys
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = """
import ctypes, json, os, sys
import paper_2602_01613_amd as tn
import workloads as wl
from paper_2602_01613_amd.binding import _make_desc
lib = tn.load_library()
lib.tn_linear_forward_scratch.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p]
lib.tn_linear_param_gradients.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p]
hip = ctypes.CDLL(os.environ['LD_PRELOAD'])
hip.fake_hip_take_launches.restype = ctypes.c_char_p
def launches():
    return [[l.split()[0]] + [int(v) for v in l.split()[1:]] for l in hip.fake_hip_take_launches().decode().splitlines()]
block = None
def layer(fmt, dtype, out_modes, in_modes, ranks, max_tokens, limit, flags, whats, scratch_tokens, grad_tokens, tokens, wanted, block_bytes):
    global block
    if block_bytes and block is None:
        block = ctypes.create_string_buffer(block_bytes + 256)
    spec = wl.TNSpec(fmt, dtype, tuple(out_modes), tuple(in_modes), tuple(ranks))
    mem = ctypes.create_string_buffer(64)
    ptrs = [ctypes.addressof(mem)] * len(spec.tensor_shapes())
    d, keep = _make_desc(fmt, tn.TN_DTYPE_BF16 if dtype == 'bf16' else tn.TN_DTYPE_F32, out_modes, in_modes, ranks, ptrs, max_tokens, limit, flags, None,
                         (ctypes.addressof(block) + 255) // 256 * 256 if block_bytes else None, block_bytes)
    h = ctypes.c_void_p()
    rc = lib.tn_linear_create(ctypes.byref(h), ctypes.byref(d))
    res = {"rc": rc}
    for w in whats:
        v = ctypes.c_int64(-1)
        if rc == 0:
            assert lib.tn_linear_query(h, w, ctypes.byref(v)) == 0
        res[str(w)] = v.value
    buf = ctypes.create_string_buffer(1024)
    at = (ctypes.addressof(buf) + 255) // 256 * 256
    res["scratch"] = [lib.tn_linear_forward_scratch(h, at, at + 256, t, None) for t in scratch_tokens] if rc == 0 else []
    grads = (ctypes.c_void_p * len(ptrs))(*[at + 512 if wanted is None or i in wanted else None for i in range(len(ptrs))])
    res["launches"], res["gradient_launches"] = [], []
    res["create_launches"] = launches()
    if rc == 0:
        for t in tokens:
            assert lib.tn_linear_forward(h, at, at + 256, t, None) == 0
            res["launches"].append(launches())
    res["gradients"] = []
    for t in grad_tokens if rc == 0 else []:
        res["gradients"].append(lib.tn_linear_param_gradients(h, at, at + 256, grads, t, None))
        res["gradient_launches"].append(launches())
    if rc == 0:
        lib.tn_linear_destroy(h)
    return res
print("RESULT " + json.dumps([layer(*job) for job in json.loads(sys.stdin.read())]))
"""


@pytest.fixture(scope="module")
def fake_hip():
    out = os.path.join(tempfile.mkdtemp(prefix="tn_fake_hip_"), "libfake_hip.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I/opt/rocm/include", os.path.join(HERE, "fake_hip.cpp"), "-o", out])
    return out


def job(spec, max_tokens, whats=(), limit=0, flags=0, scratch_tokens=(), grad_tokens=(), tokens=(), wanted=None, block_bytes=0):
    """A layer to make, and what to do with it."""
    return [spec.format, spec.dtype, list(spec.out_modes), list(spec.in_modes), list(spec.ranks), max_tokens, limit, flags, list(whats),
            list(scratch_tokens), list(grad_tokens), list(tokens), wanted, block_bytes]


def create_all(fake_hip, jobs, refuse=None):
    env = dict(os.environ, LD_PRELOAD=fake_hip)
    if refuse:
        env["FAKE_HIP_REFUSE_FROM"], env["FAKE_HIP_REFUSE_TO"] = str(refuse[0]), str(refuse[1])
    r = subprocess.run([sys.executable, "-c", CHILD], input=json.dumps(jobs), cwd=os.path.dirname(HERE), env=env, capture_output=True, text=True, timeout=300)
    lines = [l for l in r.stdout.splitlines() if l.startswith("RESULT ")]
    assert lines, r.stderr[-800:]
    results = json.loads(lines[0][7:])
    for res in results:
        for k in ("launches", "gradient_launches"):
            res[k] = [[Launch(*l) for l in call] for call in res[k]]
    return results


def create(fake_hip, spec, max_tokens, whats, refuse=None, **kw):
    return create_all(fake_hip, [job(spec, max_tokens, whats, **kw)], refuse)[0]


class Launch:
    """One kernel launch: its name, the numbers among its template arguments in order, grid and dynamic LDS."""

    def __init__(self, mangled, grid_x, grid_y, lds):
        found = re.search(r"\d+([a-z]\w*?kernel)(I.*?EE?v|E?v|E)", mangled)
        self.kernel = found.group(1) if found else mangled
        self.args = tuple(int(v) for v in re.findall(r"L[ib](\d+)E", found.group(2))) if found else ()
        self.grid, self.lds = (grid_x, grid_y), lds

    def __repr__(self):
        return f"{self.kernel}{self.args} {self.grid} {self.lds}"


def test_no_memory_for_w_leaves_the_other_orders(fake_hip):
    """W of a train 5120 -> 8192 is 84 MB: where that allocation, or that of its 148 KB of tables, is refused, the layer is
    made as one that never takes this order."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    spec = wl.baseline_spec(1)[0]
    what = [tn.TN_QUERY_MATRIX_MIN_TOKENS, tn.TN_QUERY_WORKSPACE_BYTES, tn.TN_QUERY_PACKED_BYTES]
    full = create(fake_hip, spec, 8192, what)
    assert full["rc"] == 0 and full[str(what[0])] > 0 and full[str(what[1])] >= 84 << 20 >> 1
    never = create(fake_hip, spec, 8192, what, flags=tn.TN_FLAG_NO_LAZY_MERGE)
    for refuse in ((80 << 20, 90 << 20), (140000, 150000)):
        short = create(fake_hip, spec, 8192, what, refuse=refuse)
        assert short["rc"] == 0 and short[str(what[0])] == 0, refuse
        assert short[str(what[1])] == never[str(what[1])] and short[str(what[2])] == never[str(what[2])], refuse


@pytest.mark.parametrize("fmt,om,im,rk,tokens", [(3, (48, 64), (48, 128), (8, 64, 48, 64), (1719, 2079, 2514)),
                                                 (1, (32, 4, 8), (4, 32, 32), (1, 128, 128, 1), (42, 50, 60))])
def test_scratch_takes_the_ranges_of_k_that_fit(fake_hip, fmt, om, im, rk, tokens):
    """Calls whose intermediates leave less than half of the scratch array: sums of K ranges take what room there is and never
    refuse the call."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    spec = wl.TNSpec(fmt, "bf16", om, im, rk)
    inter = tn.plan_query(fmt, tn.TN_DTYPE_BF16, om, im, rk, tn.TN_QUERY_MAX_INTERMEDIATE, flags=tn.TN_FLAG_NO_MERGE)
    most = (32 << 20) // (4 * inter)
    got = create(fake_hip, spec, 2000, [], flags=tn.TN_FLAG_NO_MERGE, scratch_tokens=list(tokens) + [most + 1])
    assert got["rc"] == 0 and got["scratch"] == [0] * len(tokens) + [-5]


def test_gradient_of_a_tensor_of_more_than_31_bits(fake_hip):
    import paper_2602_01613_amd as tn
    import workloads as wl
    spec = wl.TNSpec(wl.FORMAT_DENSE, "bf16", (46344,), (46400,), ())
    got = create(fake_hip, spec, 8, [], flags=tn.TN_FLAG_TRAINABLE, grad_tokens=[1, 8])
    assert got["rc"] == 0 and got["gradients"] == [0, 0]


def test_work_of_gradients_through_dw(fake_hip):
    """FLOPs beside dW: a dense layer none; a train of two cores its two gradients, each from dW in two parts against a core."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    what = [tn.TN_QUERY_GRADIENT_MATRIX_MIN_TOKENS, tn.TN_QUERY_GRADIENT_MATRIX_FLOPS]
    dense = create(fake_hip, wl.stack_spec(wl.FORMAT_DENSE, 5120, 1024, 0), 512, what, flags=tn.TN_FLAG_TRAINABLE)
    assert dense[str(what[0])] > 0 and dense[str(what[1])] == 0
    spec = wl.TNSpec(wl.FORMAT_TT, "bf16", (64, 32), (64, 64), (1, 128, 1))
    train = create(fake_hip, spec, 4096, what, flags=tn.TN_FLAG_TRAINABLE)
    assert train[str(what[0])] > 0 and train[str(what[1])] == 2 * (2 * 2 * spec.M * spec.N * 128)
    steps = create(fake_hip, spec, 4096, what, flags=tn.TN_FLAG_TRAINABLE | tn.TN_FLAG_NO_LAZY_MERGE)
    assert steps[str(what[0])] == 0


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_form_of_small_layers(fake_hip, dtype):
    """Each layer of the parity test of small layers is one launch of the whole-chain kernel, in the form that it names: tiles where steps have
    rows enough to fill them, an output per thread where they have one or a few."""
    import workloads as wl
    from test_gpu_parity import SMALL_CHAINS
    most = 0
    made = create_all(fake_hip, [job(wl.TNSpec(fmt, dtype, om, im, rk), 4096, tokens=(1, 256, 257, 4096) if dtype == "f32" else (1, 32))
                                 for fmt, om, im, rk, _, _ in SMALL_CHAINS])
    for (_, om, im, _, few, many), got in zip(SMALL_CHAINS, made):
        assert all(len(call) == 1 and call[0].kernel == "small_chain_kernel" for call in got["launches"]), (om, im)
        assert [call[0].args for call in got["launches"]] == ([(int(few),)] * 2 + [(int(many),)] * (2 if dtype == "f32" else 0)), (om, im)
        most = max(most, got["launches"][0][0].lds)
    assert most > 96 << 10


@pytest.mark.parametrize("n_in,n_out,rank", [(5120, 8192, 64), (5120, 25600, 32), (5120, 1024, 96), (25600, 5120, 64)])
def test_order_by_token_count_follows_the_prices(fake_hip, n_in, n_out, rank):
    """Token counts that contract the tensors first come in ranges between the prices' crossings: none is a point of the grid that
    they are looked for on. A row tile of the matrix-product kernel is 32 rows at least, and so are they."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    spec = wl.stack_spec(wl.FORMAT_TT, n_in, n_out, rank)
    most = 2600
    got = create(fake_hip, spec, most, [tn.TN_QUERY_MATRIX_TOKENS_BASE + t for t in range(1, most + 1)])
    taken = [got[str(tn.TN_QUERY_MATRIX_TOKENS_BASE + t)] for t in range(1, most + 1)]
    assert any(taken)
    changes = [t for t in range(1, most) if taken[t] != taken[t - 1]]
    assert all(b - a >= 32 for a, b in zip(changes, changes[1:])), changes


def test_short_k_of_more_than_a_row_tile(fake_hip):
    """From 65 rows on a step of short K is the matrix-product kernel's, also where its outputs are few."""
    import workloads as wl
    shapes = [(k, c) for k in (128, 1024, 1216) for c in (64, 512, 2048)]
    made = create_all(fake_hip, [job(wl.TNSpec(wl.FORMAT_DENSE, "bf16", (c,), (k,), ()), 1000, tokens=(66, 260, 1000)) for k, c in shapes])
    for shape, got in zip(shapes, made):
        assert all("step_gemm_kernel" in [l.kernel for l in call] for call in got["launches"]), (shape, got["launches"])


def test_two_small_products_before_longer_steps(fake_hip):
    """A train of two cores of small modes: W and Y are two short products, the steps two longer ones."""
    import workloads as wl
    spec = wl.TNSpec(wl.FORMAT_TT, "bf16", (40, 8), (32, 16), (1, 24, 1))
    got = create(fake_hip, spec, 1500, [], tokens=(33, 100, 500, 1500))
    assert [[l.kernel for l in call] for call in got["launches"]] == [["step_gemm_kernel"] * 2] * 4


def test_backward_steps_have_room_for_their_sums(fake_hip):
    """Few tokens: steps of a backward pass are cut into ranges of K like those of a forward, also where no forward step needs sums."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    spec = wl.TNSpec(wl.FORMAT_TT, "bf16", (5, 33, 64), (3, 2, 8), (1, 96, 96, 1))
    got = create(fake_hip, spec, 1500, [], flags=tn.TN_FLAG_TRAINABLE, grad_tokens=[2])
    kernels = [l.kernel for l in got["gradient_launches"][0]]
    assert "step_mfma_pipe_kernel" not in kernels and kernels[kernels.index("step_split_reduce_kernel") - 1] == "step_split_kernel", kernels


def test_layers_of_the_direct_kernel_tests(fake_hip):
    """The layers of the GPU tests of slices made on chip: one token takes the instantiation that they name, 64 tokens the slices in memory; and the
    switch of decode fusion keeps them there."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    from test_gpu_direct import DIRECT_LAYERS
    for flags, n in ((0, len(DIRECT_LAYERS)), (tn.TN_FLAG_NO_DECODE_FUSION, 1)):
        made = create_all(fake_hip, [job(wl.TNSpec(fmt, "bf16", om, im, rk), 64, flags=flags, tokens=(1, 64)) for fmt, om, im, rk, _, _ in DIRECT_LAYERS[:n]])
        for (_, om, _, _, cfg, steps), got in zip(DIRECT_LAYERS, made):
            one, many = got["launches"]
            assert (one[0].kernel == "step_krondirect_kernel") == (flags == 0), (om, one)
            assert flags or (one[0].args == (cfg, steps) and len(one) <= 2), (om, one)
            assert all(l.kernel != "step_krondirect_kernel" for l in many), (om, many)


def test_tiles_of_the_matrix_product_tests(fake_hip):
    """The calls of the GPU tests that name a tile of the matrix-product kernel, or its form for short K, take it."""
    import workloads as wl
    from test_gpu_gemm import PINNED, SHORT_K_ROWS, TILE_CALLS
    calls = [(tile, k, n_out, (rows,)) for tile, n_out, rows, ks in TILE_CALLS for k in ks]
    calls += [((5, 4, k // 64), k, n_out, rows) for k in (64, 128) for n_out, rows in SHORT_K_ROWS.items()]
    made = create_all(fake_hip, [job(wl.TNSpec(wl.FORMAT_DENSE, "bf16", (n_out,), (k,), ()), max(rows), flags=PINNED, tokens=rows)
                                 for _, k, n_out, rows in calls])
    for (tile, k, n_out, rows), got in zip(calls, made):
        for call in got["launches"]:
            used = [l.args for l in call if l.kernel == "step_gemm_kernel"]
            form = 3 if k % 64 else 1 if len(rows) == 1 else 4
            assert used == [(*tile, 0, form)], (tile, k, n_out, rows, used)
    assert {t for t, *_ in TILE_CALLS} >= {(8, 8, 2), (7, 8, 2), (6, 8, 2), (5, 8, 3), (4, 8, 3), (3, 8, 3), (2, 8, 3), (8, 4, 3), (6, 4, 3),
                                           (5, 4, 2), (4, 4, 2), (3, 4, 2), (2, 4, 3), (2, 2, 4)}


def test_kernels_of_the_gradient_tests(fake_hip):
    """The layers of the GPU tests of gradients take the kernels that these tests name: one pass over dW, and row runs read in 16-byte pieces."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    from test_gpu_gradients import NARROW_BONDS, ROW_RUNS, narrow_bond
    bonds = [narrow_bond(case, rank) for case in range(len(NARROW_BONDS)) for rank in (32, 64, 96, 128)]
    through_dw = tn.TN_QUERY_GRADIENT_MATRIX_MIN_TOKENS
    made = create_all(fake_hip, [job(spec, 1000, [through_dw], flags=tn.TN_FLAG_TRAINABLE, grad_tokens=[1000]) for spec, _ in bonds])
    for (spec, one_pass), got in zip(bonds, made):
        assert got[str(through_dw)] > 0
        assert [l.args for l in got["gradient_launches"][0] if l.kernel == "bond_grad_kernel"] == ([(spec.ranks[len(spec.out_modes) // 2] // 32,)] if one_pass else [])
    made = create_all(fake_hip, [job(wl.TNSpec(wl.FORMAT_TUCKER, "bf16", om, im, rk), 400, flags=tn.TN_FLAG_TRAINABLE, grad_tokens=(40, 333))
                                 for om, im, rk, _, _ in ROW_RUNS])
    for (om, _, rk, *named), got in zip(ROW_RUNS, made):
        for tokens, steps, call in zip((40, 333), named, got["gradient_launches"]):
            # one workgroup per 256 rows, padded to 8 of them, and 128 columns
            grids = sorted(((tokens * rows + 255) // 256 + 7) // 8 * 8 * ((cols + 127) // 128) for _, cols, rows in steps)
            assert sorted(l.grid[0] for l in call if l.kernel == "step_mfma_pipe_kernel" and l.args[4] == 3) == grids, (om, rk, tokens)


def test_launches_of_the_core_gradient_tests(fake_hip):
    """Rings of that GPU test: one launch for the transposed copies of the activations, one for those of dW, and one for both halves' or
    one for each; a train's halves, and the four products of its cores' gradients, in a launch each."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    from test_gpu_gradients import RING_CORES, narrow_bond, ring_of_cores
    made = create_all(fake_hip, [job(ring_of_cores(*ring), 48, flags=tn.TN_FLAG_TRAINABLE, grad_tokens=(48,)) for ring in sorted(RING_CORES)])
    for ring, got in zip(sorted(RING_CORES), made):
        assert got["gradients"] == [0]
        turns = [l.grid[1] for l in got["gradient_launches"][0] if l.kernel == "transpose_kernel"]
        assert turns == ([2, 2, 4] if RING_CORES[ring] else [2, 2, 2, 2]), (ring, turns)
    spec, one_pass = narrow_bond(0, 64)
    got = create(fake_hip, spec, 1000, [], flags=tn.TN_FLAG_TRAINABLE, grad_tokens=(1000,), tokens=(1000,))
    many = lambda calls: [l.grid[1] for l in calls[0] if l.kernel == "step_gemm_many_kernel"]      # noqa: E731
    assert one_pass and many(got["launches"]) == [2] and many(got["gradient_launches"]) == [2, 4]
    assert [l.grid[1] for l in got["gradient_launches"][0] if l.kernel.startswith("grad_reduce")] == [4]
    # with the gradients of some cores only
    got = create(fake_hip, spec, 1000, [], flags=tn.TN_FLAG_TRAINABLE, grad_tokens=(1000,), wanted=[1])
    assert many(got["gradient_launches"]) == [2] and got["gradients"] == [0]


def test_launches_of_the_factor_pair_layers(fake_hip):
    """Layers of those tests' kind: which side takes a launch with a workgroup to a token, and which instantiation (A, B, P, Q / 32)."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    shapes = [((160, 160), (64, 80), (96, 96, 48, 48), [("in", 2, 3, 2, 2), ("out", 5, 5, 3, 3)]),
              ((64, 80), (160, 160), (32, 32, 48, 48), [("in", 5, 5, 2, 2), ("out", 2, 3, 2, 2)]),
              ((64, 128), (64, 128), (48, 48, 16, 16), [("in", 2, 4, 2, 2), ("out", 2, 4, 2, 3)]),
              ((160, 176), (64, 72), (32, 32, 16, 16), []),                                     # too long, no whole tiles
              ((160, 160), (64, 80), (112, 96, 48, 48), [("in", 2, 3, 2, 2)])]                  # a rank too large
    made = create_all(fake_hip, [job(wl.TNSpec(wl.FORMAT_TUCKER, "bf16", om, im, rk), 1100, tokens=(1, 70, 1100)) for om, im, rk, _ in shapes])
    for (om, im, rk, want), got in zip(shapes, made):
        for tokens, call in zip((1, 70, 1100), got["launches"]):
            used = [(l.kernel[7:-7], *l.args) for l in call if l.kernel in ("factor_in_kernel", "factor_out_kernel")]
            # a token is left to the kernels that spread it, where they hold it (K of the first step up to 128)
            assert used == ([w for w in want if w[:2] == ("in", 5)] if tokens == 1 else want), (om, im, rk, tokens, used)
            for l in call:
                if l.kernel.startswith("factor_"):
                    assert l.grid == (min(tokens, 256 * (3 if l.args[0] < 5 else 2)), 1)
    off = create(fake_hip, wl.TNSpec(wl.FORMAT_TUCKER, "bf16", *shapes[0][:3]), 1100, [], flags=tn.TN_FLAG_NO_CHAIN2, tokens=(1100,))
    assert not [l for l in off["launches"][0] if l.kernel.startswith("factor_")]


def test_launches_of_the_skinny_tests(fake_hip):
    """The dense layers of that GPU test take the kernel that it is about."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    from test_gpu_skinny import SKINNY
    for m, n, tokens, quant in SKINNY:
        got = create(fake_hip, wl.TNSpec(wl.FORMAT_DENSE, "bf16", (m,), (n,), ()), tokens, [], flags=tn.TN_FLAG_QUANT_MXFP4 if quant else 0, tokens=(tokens,))
        assert [l.args for l in got["launches"][0] if l.kernel == "step_skinny_kernel"] == [(2 if tokens > 32 else 1, 0, int(quant))], (m, n, tokens)


def test_room_of_gradients_through_dw(fake_hip):
    """A second place for a half's gradient, for shared launches, is taken only where it takes no tokens from a pass: the smallest limits
    under which these layers took the order through dW still give it, with 64 tokens to a pass, and each further 64 tokens' X and dY make
    a pass 64 tokens longer."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    from test_gpu_gradients import ring_of_cores, tight_layers
    whats = [tn.TN_QUERY_GRADIENT_MATRIX_MIN_TOKENS, tn.TN_QUERY_BACKWARD_CHUNK_TOKENS]
    layers = [(wl.baseline_spec(1)[0], 189.5e6), (wl.stack_spec(wl.FORMAT_TT, 25600, 5120, 96), 564.8e6), (ring_of_cores(16, 8), 152.2e6), (ring_of_cores(8, 8), 78.8e6)]
    more = (0, 1, 3, 10)
    made = create_all(fake_hip, [job(spec, 1000, whats, int(limit) + k * 64 * 2 * (spec.M + spec.N), tn.TN_FLAG_TRAINABLE) for spec, limit in layers for k in more])
    for n, got in enumerate(made):
        assert got["rc"] == 0 and got[str(whats[0])] > 0 and got[str(whats[1])] == 64 * (1 + more[n % len(more)]), (n, got)
    # the layers of the GPU test of this: a half's sums and its cores' products, then the other's
    made = create_all(fake_hip, [job(spec, tokens, whats, limit, tn.TN_FLAG_TRAINABLE, grad_tokens=(tokens,)) for spec, tokens, limit in tight_layers()])
    for (spec, tokens, _), got in zip(tight_layers(), made):
        assert got["gradients"] == [0] and got[str(whats[1])] == (192 if tokens == 300 else 64)
        calls = got["gradient_launches"][0]
        passes = (tokens + got[str(whats[1])] - 1) // got[str(whats[1])]
        assert [l.grid[1] for l in calls if l.kernel == "grad_reduce_many_kernel"] == [2, 2] * passes
        assert [l.grid[1] for l in calls if l.kernel == "step_split_reduce_parts_two_kernel"] == ([1, 1] * passes if spec.format == wl.FORMAT_TT else [])


def test_launches_of_one_range_and_of_most_tokens(fake_hip):
    """The calls of that GPU test: without ranges of K the on-chip kernel alone, at the most tokens it and the launch that adds its sums."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    from test_gpu_direct import DIRECT_LAYERS, MOST_TOKENS, ONE_RANGE
    for calls, tokens, flags in ((ONE_RANGE, (2, 7), tn.TN_FLAG_NO_SPLIT_K), (MOST_TOKENS, (16,), 0)):
        made = create_all(fake_hip, [job(wl.TNSpec(fmt, "bf16", om, im, rk), 16, flags=flags, tokens=tokens, block_bytes=(1 << 30) * in_block)
                                     for (fmt, om, im, rk, _, _), in_block in ((DIRECT_LAYERS[n], b) for n, b in calls)])
        for (n, _), got in zip(calls, made):
            for call in got["launches"]:
                assert call[0].kernel == "step_krondirect_kernel" and call[0].args == DIRECT_LAYERS[n][4:], (n, call)
                assert len(call) == (1 if flags else 2), (n, call)
    assert {DIRECT_LAYERS[n][4] for n, _ in ONE_RANGE} == {0, 1, 2, 4}


def test_slices_on_chip_of_resident_cores_in_lds(fake_hip):
    """A train 25600 -> 5120 of rank 96, whose resident cores go to LDS, 45 KB a turn: from 12 tokens on a workgroup has so many turns that the
    slices in memory are the faster way. Rank 64 has fewer and shorter ones."""
    import workloads as wl
    made = create_all(fake_hip, [job(wl.stack_spec(wl.FORMAT_TT, 25600, 5120, rank), 16, tokens=(1, 8, 12, 16)) for rank in (64, 96)])
    assert [[call[0].kernel == "step_krondirect_kernel" for call in got["launches"]] for got in made] == [[True] * 4, [True, True, False, False]]


def test_slices_on_chip_without_ranges(fake_hip):
    """Rank-96 layers without ranges of K: at one token, which four waves share there, the slices stay in memory; a ring's are made on chip from two
    tokens on, those of a train 25600 -> 5120, each with its turn of resident cores, never."""
    import paper_2602_01613_amd as tn
    import workloads as wl
    layers = [(wl.FORMAT_TR, 5120, 8192), (wl.FORMAT_TR, 25600, 5120), (wl.FORMAT_TT, 25600, 5120)]
    made = create_all(fake_hip, [job(wl.stack_spec(fmt, n, m, 96), 16, flags=tn.TN_FLAG_NO_SPLIT_K, tokens=(1, 2, 16)) for fmt, n, m in layers])
    assert [[call[0].kernel == "step_krondirect_kernel" for call in got["launches"]] for got in made] == [[False, True, True]] * 2 + [[False] * 3]


def test_forms_of_the_factor_pair_tests(fake_hip):
    """The layers of that GPU test: of the forms that hold a pair the one with the least work, and the calls that stay with a wave to a token."""
    import workloads as wl
    from test_gpu_factor_pairs import FORM_PAIRS
    made = create_all(fake_hip, [job(wl.TNSpec(wl.FORMAT_TUCKER, "bf16", om, im, rk), 2100, tokens=(70, 600, 2100)) for om, im, rk, _ in FORM_PAIRS])
    seen = set()
    for (om, im, rk, want), got in zip(FORM_PAIRS, made):
        used = [[(l.kernel[7:-7], *l.args) for l in call if l.kernel in ("factor_in_kernel", "factor_out_kernel")] for call in got["launches"]]
        assert used == want, (om, im, rk, used)
        seen |= {f for call in used for f in call}
    assert len(seen) == 12


def test_reductions_of_the_odd_bond_tests(fake_hip):
    import paper_2602_01613_amd as tn
    from test_gpu_gradients import ODD_BONDS, ring_of_bond
    rings = sorted(ODD_BONDS)
    made = create_all(fake_hip, [job(ring_of_bond(*ring), 48, flags=tn.TN_FLAG_TRAINABLE, grad_tokens=(48,)) for ring in rings])
    for ring, got in zip(rings, made):
        assert [(l.args, l.grid[1]) for l in got["gradient_launches"][0] if l.kernel == "grad_reduce_many_kernel"] == [(ODD_BONDS[ring], 4)], ring


def test_operands_of_a_layer_are_written_together(fake_hip):
    """Layers in a shared block have the operands of the slices, in memory and on chip: eight, one launch."""
    import workloads as wl
    made = create_all(fake_hip, [job(wl.stack_spec(fmt, 5120, 8192, rank), 16, block_bytes=1 << 28) for fmt, rank in ((wl.FORMAT_TT, 32), (wl.FORMAT_TR, 96))])
    for got in made:
        written = [l for l in got["create_launches"] if "operand_source_kernel" in l[0]]
        assert len(written) == 1, written
