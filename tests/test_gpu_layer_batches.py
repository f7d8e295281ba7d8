"""Layers run in batches: as many as the workspace holds (cmoe_step) or the
scratch array (cmoe_step_noalloc).  One configuration whose two entry points
batch differently, a ragged last batch included, must give the same outputs,
logits, caches, priorities, counters and slot maps bit for bit, with the
refinement's prediction handed from batch to batch and from token to token."""
import numpy as np
import pytest

import synth
from gpu_util import say
from test_zz_no_alloc import compare

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("mode,policy,slots", [
    (synth.MODE_TEMPORAL, synth.POLICY_ROUTER, 0),
    (synth.MODE_SPATIO_TEMPORAL, synth.POLICY_ROUTER, 0),
    (synth.MODE_SPATIO_ONLY, synth.POLICY_LRU, 0),
    (synth.MODE_SPATIO_TEMPORAL, synth.POLICY_ROUTER, 60),   # FFN rounds
])
def test_batches_of_layers_agree(mode, policy, slots):
    from paper_2609_04895_amd import cmoe as B
    from paper_2609_04895_amd.workload import engine_for
    # 2 to 3 MB of partial sums and 6.3 MB of gated outputs a layer: all 13
    # layers fit one batch of the workspace, not the 64 MiB scratch array
    w = synth.WORKLOADS["qwen3_30b"].replace(name=f"batches_{mode}_{slots}", L=13, N=130, K=5, d=2112, F=64, S=301,
                                             C=20, R=3 if mode else 0, mode=mode, policy=policy, arena_slots=slots)
    T = 3
    say(f"layer batches {w.name}")
    inp = synth.device_inputs(w, T=T)
    ea = engine_for(w, inp)
    eb = engine_for(w, inp)
    ya = torch.empty((w.S, w.L, w.d), dtype=torch.float32, device="cuda:0")
    yb = torch.full_like(ya, float("nan"))
    for t in range(T):
        ea.cmoe_step(inp["hidden"][t], ya)
        eb.cmoe_step_noalloc(inp["hidden"][t], yb)
        compare(B, ea, eb, ya, yb, f"{w.name} token {t}")
        assert np.array_equal(ea.cmoe_read(B.CMOE_VIEW_PRIORITY).view(np.uint32),
                              eb.cmoe_read(B.CMOE_VIEW_PRIORITY).view(np.uint32))
    ea.cmoe_destroy()
    eb.cmoe_destroy()
