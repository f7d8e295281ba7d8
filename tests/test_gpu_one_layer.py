"""One layer per handle, where a token without refinement decides its residency
event and copies its experts in one launch: cache decisions, slot maps, counters
and copies against the oracle bit for bit, and every slot's contents, while the
refinement budget moves tokens between that launch and the separate ones.  Sizes:
cache words in less and more than one batch of loads per thread, three words per
stream (N = 130), part-filled copy pieces, more copies than one, and arenas that
do not hold the union of the caches, in one FFN round and in several."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import compare_step, say, stable_seed
from test_gpu_cache_parity import logits_sequence, packed_from_plain
from test_gpu_e2e_parity import run_e2e

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,K,C,S,d,F,dtype,pool_kind,P", [
    (1, 1, 1, 1, 64, 64, "bf16", "device", 0),
    (11, 2, 4, 2, 320, 192, "bf16", "device", 0),
    (11, 2, 4, 2, 576, 64, "bf16", "host", 0),
    (9, 3, 4, 3, 64, 192, "f32", "device", 0),
    (130, 5, 20, 37, 64, 64, "bf16", "device", 0),
    (256, 8, 40, 300, 64, 64, "f32", "host", 0),
    (8, 2, 3, 1100, 64, 64, "bf16", "device", 0),
    (16, 2, 8, 1, 320, 192, "bf16", "device", 4),   # one round, eight cached experts
    (40, 2, 12, 2, 128, 576, "bf16", "device", 5),
    (64, 4, 16, 9, 64, 64, "bf16", "device", 10),   # rounds
])
def test_one_layer(N, K, C, S, d, F, dtype, pool_kind, P):
    from paper_2609_04895_amd import cmoe as B
    name = f"one_layer_{N}_{K}_{C}_{S}_{d}_{F}_{dtype}_{pool_kind}_{P}"
    say(name)
    bf, host = dtype == "bf16", pool_kind == "host"
    dt, raw = (torch.bfloat16, torch.int16) if bf else (torch.float32, torch.int32)
    dev = torch.device("cuda", 0)
    per = 3 * d * F
    gen = torch.Generator().manual_seed(stable_seed(name))
    bits = torch.randint(0, 2 ** 15, (1, N, per), generator=gen, dtype=torch.int32).to(raw)
    pool = bits.view(dt).pin_memory() if host else bits.view(dt).to(dev)
    src = bits.numpy().view(np.uint16 if bf else np.uint32)
    w = torch.zeros((1, N, d), dtype=dt, device=dev)
    R = min(3, N)
    cfg = B.make_config(1, N, K, d, F, C, 0, S, B.CMOE_MODE_SPATIO_TEMPORAL, B.CMOE_BF16 if bf else B.CMOE_F32,
                        B.CMOE_POOL_HOST_PINNED if host else B.CMOE_POOL_DEVICE, warmup_tokens=1, arena_slots=P)
    eng = B.Engine(cfg, w, w, w, None, pool)
    run = oracle.Run(1, N, K, C, 0, S, 1, 1, arena_slots=P)
    T = 8
    z = logits_sequence(np.random.default_rng(stable_seed(name)), T, S, 1, N, ties=True)
    n_slots = P or min(N, S * C)
    for t in range(T):
        if t in (3, 5, 6):  # R = 0, 0, 0, R, R, 0, R, R
            budget = 0 if t == 5 else R
            eng.cmoe_set_R(budget)
            run.set_R(budget)
        eng.cmoe_step_logits(*(torch.from_numpy(z[t, i]).to(dev) for i in range(3)))
        out = run.step(z[t, 0], z[t, 1], z[t, 2], want="all")
        compare_step(eng, run, out, f"{name} token {t}")
        if t not in (0, 2, 3, 5, T - 1):
            continue
        slots = eng.cmoe_read(B.CMOE_VIEW_SLOTS)[0]
        arena = eng.arena[: n_slots * per * (2 if bf else 4)].view(raw).cpu().numpy().view(src.dtype).reshape(n_slots, per)
        for e in np.nonzero(slots >= 0)[0]:
            x = src[0, e]
            want = packed_from_plain(x, d, F) if bf else np.concatenate(
                [x[:F * d].reshape(F, d).T.ravel(), x[F * d:2 * F * d].reshape(F, d).T.ravel(),
                 x[2 * F * d:].reshape(d, F).T.ravel()])
            assert np.array_equal(arena[slots[e]], want), (name, t, e)
    eng.cmoe_destroy()


@pytest.mark.parametrize("S,N,K,shape", [(1, 16, 2, None), (9, 16, 4, "single"), (140, 6, 2, "grouped"),
                                         (300, 4, 2, "grouped")])
def test_one_layer_outputs(S, N, K, shape):
    # work units of one pass, of several, and of both lists; bf16 tolerance
    w = synth.WORKLOADS["qwen3_30b"].replace(name=f"one_layer_{S}_{N}_{K}", L=1, N=N, K=K, d=128, F=192, S=S, C=K)
    run_e2e(w, T=4, tol=2e-2, ffn_shape=shape)
