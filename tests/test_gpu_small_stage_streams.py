"""A small stage keeps its gradient leaves on the caller's stream until the side stream is asked for: the default, both
times of asking (at the start and between a backward and its accumulation) and the side stream off end in the same bits."""
import numpy as np
import pytest

import workloads as W
from tests.parity import GpuStage
from paper_2605_29664_amd.binding import OPT_LEAF_FORKS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("key", ["gpt_tile64", "bert_tile", "embed_tile", "gpt", "lmhead_tile"])
def test_leaves_on_either_stream(key):
    from oracle.stage import Stage as OStage
    w = W.TINY[key]
    theta0 = W.make_theta(w, OStage.from_workload(w).layout)
    states = []
    for mode in ("default", "overlap", "overlap_two_forks", "overlap_later", "off"):
        gpu = GpuStage(w, act_slots=2, stash_slots=1, options={OPT_LEAF_FORKS: 2} if mode == "overlap_two_forks" else None)
        if mode in ("overlap", "overlap_two_forks", "off"):
            gpu.stage.amdp_stage_set_overlap(mode != "off")
        gpu.set_state(theta0)
        out = []
        for mb in range(3):
            x = None if w.has_embedding else W.make_x(w, mb)
            out.append(gpu.forward(mb, 0, x, W.make_aux(w, mb)))
            out += [r for r in gpu.backward(mb, 0, None if w.has_lm_head else W.make_dy(w, mb)) if r is not None]
            if mode == "overlap_later" and mb == 1:
                gpu.stage.amdp_stage_set_overlap(True)
            gpu.accumulate(mb)
        gpu.update(w, 1.0 / 3)
        s = gpu.state()
        states.append(out + [s[k] for k in ("theta", "m", "v", "G")])
        gpu.stage.close()
    for other in states[1:]:
        for a, b in zip(states[0], other):
            assert np.array_equal(a, b)


# multiply-adds of a layer's weight gradients on either side of the line (6e9 in bf16, 1e9 in fp32)
@pytest.mark.parametrize("key,sizes,used", [
    ("gpt_tile", {}, False), ("gpt", {}, False), ("gpt_tile", dict(d_model=512, n_heads=8, d_ffn=2048, seq_len=1024, microbatch=1), False),
    ("gpt_tile", dict(d_model=512, n_heads=8, d_ffn=2048, seq_len=1024, microbatch=2), True),
    ("gpt", dict(d_model=256, n_heads=4, d_ffn=1024, seq_len=1264, microbatch=1), False),
    ("gpt", dict(d_model=256, n_heads=4, d_ffn=1024, seq_len=1280, microbatch=2), True)])
def test_overlap_reads_back_what_the_stage_does(key, sizes, used):
    """The default is off for a small stage and reads as off; saving it, switching and restoring it ends in the default."""
    gpu = GpuStage(W.TINY[key].with_(**sizes))
    assert gpu.stage.amdp_stage_get_overlap() == used
    for on in (not used, used):
        gpu.stage.amdp_stage_set_overlap(on)
        assert gpu.stage.amdp_stage_get_overlap() == on
    gpu.stage.close()
