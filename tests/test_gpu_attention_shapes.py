"""The fused attention where a head is narrower than its tile or a sequence ends inside a block of 128
queries or 64 keys: whole small stages against the CPU oracle (tests/parity.py) in its tolerances."""
import pytest

import workloads as W
from tests.parity import run_parity, worst_entries

pytestmark = pytest.mark.gpu

# sequence x heads x head width: the shortest sequence; one 8-wide step past and short of a block of 64 keys and
# of 128 queries; a last block of which only one wave has queries; widths with a tail of 2, 4 and 6 columns,
# below one vector, one column pair short of either tile and past the smaller one
SHAPES = [(8, 2, 64), (56, 4, 6), (72, 1, 64), (120, 4, 50), (136, 1, 128), (136, 4, 62), (152, 3, 32), (200, 4, 66), (256, 4, 84),
          (264, 4, 126), (384, 1, 96)]


@pytest.mark.parametrize("key", ["gpt_tile", "bert_tile"])
@pytest.mark.parametrize("seq,heads,width", SHAPES)
def test_ragged_attention(key, seq, heads, width):
    w = W.TINY[key].with_(n_layers=1, d_model=heads * width, n_heads=heads, d_ffn=2 * heads * width, seq_len=seq, microbatch=2,
                          depth=2, pipelines=1, stage=1, threshold=2)
    rep = run_parity(w, n_windows=1, verbose=False)
    assert rep["ok"], worst_entries(rep)
