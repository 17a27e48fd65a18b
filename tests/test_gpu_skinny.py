"""Up to 64 rows against a streamed tensor, 256 columns to a workgroup: rows that are requested ahead of the stream, against the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as wl
import paper_2602_01613_amd as tn
from gpu_util import TOL, make_layer, to_dev, to_host

pytestmark = pytest.mark.gpu

# dense M x N, tokens, stored in 4 bits
SKINNY = [(520, 1000, 33, False),         # K ends inside a piece of 64; a last column block of 8, seven waves without columns
          (264, 4096, 64, False),         # every thread's pieces end inside the rows requested ahead
          (5120, 25600, 64, False),       # and go on behind them
          (256, 1056, 14, True),          # 4 bits: K of no whole piece
          (520, 4096, 40, True),
          (1024, 25600, 64, True)]


@pytest.mark.parametrize("case", range(len(SKINNY)))
def test_rows_ahead_of_the_stream(case):
    m, n, tokens, quant = SKINNY[case]
    spec = wl.TNSpec(wl.FORMAT_DENSE, "bf16", (m,), (n,), ())
    rng = np.random.default_rng(800 + case)
    w = wl.round_to_dtype(rng.standard_normal((m, n)) / np.sqrt(n), "bf16")
    x = wl.round_to_dtype(rng.standard_normal((tokens, n)), "bf16")
    layer = make_layer(spec, [w], tokens, flags=tn.TN_FLAG_QUANT_MXFP4 if quant else 0)
    y = to_host(layer(to_dev(x, "bf16")))
    layer.close()
    if quant:
        w = O.mxfp4_dequantized([w])[0]
    assert O.rel_max_err(y, O.apply_linear(w, x)) <= TOL["bf16"]
