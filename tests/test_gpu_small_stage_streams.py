"""A small stage keeps its gradient leaves on the caller's stream until the side stream is asked for: the default, both
ways of asking (at the start and between a backward and its accumulation) and the side stream off end in the same bits."""
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
    for mode in ("default", "forks", "overlap", "forks_later", "off"):
        gpu = GpuStage(w, act_slots=2, stash_slots=1, options={OPT_LEAF_FORKS: 0} if mode == "forks" else None)
        if mode in ("overlap", "off"):
            gpu.stage.amdp_stage_set_overlap(mode == "overlap")
        gpu.set_state(theta0)
        out = []
        for mb in range(3):
            x = None if w.has_embedding else W.make_x(w, mb)
            out.append(gpu.forward(mb, 0, x, W.make_aux(w, mb)))
            out += [r for r in gpu.backward(mb, 0, None if w.has_lm_head else W.make_dy(w, mb)) if r is not None]
            if mode == "forks_later" and mb == 1:
                gpu.stage.amdp_stage_set_option(OPT_LEAF_FORKS, 2)
            gpu.accumulate(mb)
        gpu.update(w, 1.0 / 3)
        s = gpu.state()
        states.append(out + [s[k] for k in ("theta", "m", "v", "G")])
        gpu.stage.close()
    for other in states[1:]:
        for a, b in zip(states[0], other):
            assert np.array_equal(a, b)
