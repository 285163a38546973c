"""The matrix-core product of fp32 stages on either of its tilings, with and without 16-byte loads: whole small
stages against the CPU oracle (tests/parity.py), whose fp32 gate (1e-5 in norm) is far above the error of a sum
of at most a few thousand fp32 products and far below one lost or doubled term of it."""
import pytest

import workloads as W
from tests.parity import run_parity, worst_entries

pytestmark = pytest.mark.gpu

# sequence x minibatch x width x heads x FFN: less than one tile and less than one k chunk; one vector past and short
# of a 32- and a 64-wide tile and of a 128-long chunk; head widths of 3 and 33, whose rows no 16-byte load takes
# (every element by itself); more than two 64x64 tiles to a compute unit
SHAPES = [(4, 1, 4, 1, 4), (36, 1, 60, 5, 132), (68, 2, 132, 44, 124), (100, 3, 132, 4, 260), (1028, 4, 260, 2, 2052)]


@pytest.mark.parametrize("key", ["gpt", "bert"])
@pytest.mark.parametrize("seq,microbatch,width,heads,ffn", SHAPES)
def test_products(key, seq, microbatch, width, heads, ffn):
    w = W.TINY[key].with_(n_layers=1, d_model=width, n_heads=heads, d_ffn=ffn, seq_len=seq, microbatch=microbatch, depth=2,
                          pipelines=1, stage=1, threshold=2)
    rep = run_parity(w, n_windows=1, verbose=False)
    assert rep["ok"], worst_entries(rep)
