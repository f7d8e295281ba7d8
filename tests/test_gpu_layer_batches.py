"""Layers run in batches: as many as the workspace holds (cmoe_step) or the
scratch array (cmoe_step_noalloc).  One configuration whose two entry points
batch differently, a ragged last batch included, must give the same outputs,
logits, caches, priorities, counters and slot maps bit for bit, with the
refinement's prediction handed from batch to batch and from token to token:
each entry point alone, both in turn on one handle, and with proactive fills on
the side stream, where a last batch of one layer keeps them on the main stream."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import compare_step, say
from test_gpu_cache_parity import logits_sequence, packed_from_plain
from test_gpu_e2e_parity import run_e2e
from test_zz_no_alloc import compare

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


SCRATCH = 64 << 20


def scratch_batch(B, w):
    """Layers per batch on the scratch array, from the sizes that cmoe_query
    states: the workspace of L layers in one batch is L times the buffers of a
    layer, of which the logits, selections, gates, events and fill counts are
    held for every layer whatever the batch (buffer sizes are rounded to 256
    bytes, which the assertions below leave room for)."""
    from paper_2609_04895_amd.workload import config_for
    total = B.cmoe_query(config_for(w)).workspace_bytes
    assert total < 190 << 20, "all layers in one batch of the workspace"
    assert total > SCRATCH, "not on the scratch array"
    n_r = len(B.router_slots(config_for(w)))
    kept = w.L * (w.S * (n_r * w.N + 2 * w.K + 4) * 4 + 8)
    per_layer = (total - kept) / w.L
    G = int((SCRATCH - kept) / per_layer)
    assert abs((SCRATCH - kept) / per_layer - round((SCRATCH - kept) / per_layer)) > 1e-2, "rounding could decide"
    return G


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
    G = scratch_batch(B, w)
    assert 1 < G < w.L and w.L % G != 0
    say(f"layer batches {w.name}: {G} layers a batch on the scratch array")
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


@pytest.mark.parametrize("mode,policy,slots", [
    (synth.MODE_TEMPORAL, synth.POLICY_ROUTER, 0),
    (synth.MODE_SPATIO_TEMPORAL, synth.POLICY_ROUTER, 0),
    (synth.MODE_SPATIO_ONLY, synth.POLICY_LRFU, 60),
])
@pytest.mark.parametrize("L", [16, 0], ids=["ragged", "last_of_one"])
def test_sides_and_entry_points_agree(L, mode, policy, slots):
    from paper_2609_04895_amd import cmoe as B
    from paper_2609_04895_amd.workload import engine_for
    w = synth.WORKLOADS["qwen3_30b"].replace(name=f"batches_side_{mode}_{slots}_{L}", L=L or 9, N=130, K=5, d=2112,
                                             F=64, S=301, C=20, R=3 if mode else 0, mode=mode, policy=policy,
                                             arena_slots=slots)
    if not L:  # a last batch of one layer on the scratch array
        w = w.replace(L=next(l for l in range(9, 20) if l % scratch_batch(B, w.replace(L=l)) == 1))
    T, G = 4, scratch_batch(B, w)
    assert 1 < G < w.L and (w.L % G > 1 if L else w.L % G == 1)
    say(f"layer batches {w.name}: L={w.L}, {G} a batch on the scratch array")
    inp = synth.device_inputs(w, T=T)
    plain = engine_for(w, inp)
    others = [engine_for(w, inp), engine_for(w, inp, fills="side"), engine_for(w, inp, fills="side"),
              engine_for(w, inp, fills="side", workspace=False)]
    y = torch.empty((w.S, w.L, w.d), dtype=torch.float32, device="cuda:0")
    yo = torch.full_like(y, float("nan"))
    for t in range(T):
        plain.cmoe_step(inp["hidden"][t], y)
        # in turn (starting with either), side stream on the workspace, in turn
        # on the side stream, side stream on the scratch array
        for i, e in enumerate(others):
            noalloc = (i == 0 and t % 2 == 0) or (i == 2 and t % 2 == 1) or i == 3
            (e.cmoe_step_noalloc if noalloc else e.cmoe_step)(inp["hidden"][t], yo)
            compare(B, plain, e, y, yo, f"{w.name} token {t} engine {i}")
            yo.fill_(float("nan"))
    for e in [plain] + others:
        e.cmoe_destroy()


def test_more_layers_than_a_batch_holds():
    """64 layers at most share a launch: 65 and 130 small layers, every one with
    copies, against the oracle; the side stream and the main stream."""
    from paper_2609_04895_amd import cmoe as B
    N, K, C, S, R, d = 12, 2, 4, 3, 2, 64
    dev = torch.device("cuda", 0)
    for L, side in ((65, False), (130, True)):
        say(f"layer batches: {L} layers, side={side}")
        w = torch.zeros((L, N, d), dtype=torch.bfloat16, device=dev)
        bits = torch.randint(0, 2 ** 15, (L, N, 3 * d * d), generator=torch.Generator().manual_seed(L),
                             dtype=torch.int32).to(torch.int16)
        cfg = B.make_config(L, N, K, d, d, C, R, S, B.CMOE_MODE_SPATIO_TEMPORAL, B.CMOE_BF16,
                            flags=B.CMOE_FLAG_FILL_ON_SIDE if side else 0)
        eng = B.Engine(cfg, w, w, w, None, bits.view(torch.bfloat16).to(dev),
                       side_stream=torch.cuda.Stream() if side else None)
        run = oracle.Run(L, N, K, C, R, S, 1)
        z = logits_sequence(np.random.default_rng(L), 5, S, L, N, ties=True)
        src = bits.numpy().view(np.uint16)
        n_slots = min(N, S * C)
        for t in range(5):
            eng.cmoe_step_logits(*(torch.from_numpy(z[t, i]).to(dev) for i in range(3)))
            compare_step(eng, run, run.step(z[t, 0], z[t, 1], z[t, 2], want="all"), f"{L} layers token {t}")
        slots = eng.cmoe_read(B.CMOE_VIEW_SLOTS)
        arena = eng.arena[: L * n_slots * 6 * d * d].view(torch.int16).cpu().numpy().view(np.uint16)
        arena = arena.reshape(L, n_slots, 3 * d * d)
        for l in range(L):
            for e in np.nonzero(slots[l] >= 0)[0]:
                assert np.array_equal(arena[l, slots[l, e]], packed_from_plain(src[l, e], d, d)), (l, e)
        eng.cmoe_destroy()


def test_more_layers_than_a_batch_holds_outputs():
    w = synth.WORKLOADS["gptoss_20b"].replace(name="batches_66", L=66, N=8, K=2, C=3, R=2, S=3, d=64, F=64)
    run_e2e(w, T=3, tol=2e-2)
