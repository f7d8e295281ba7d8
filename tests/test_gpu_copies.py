"""Expert copies into the slots: every piece of every listed copy lands, at k
chunk counts that leave part-filled pieces (of 4 and 8 chunks), over several
layers with different numbers of copies, from both pools and for both types."""
import numpy as np
import pytest

from gpu_util import say
from test_gpu_cache_parity import logits_sequence, packed_from_plain

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("pool_kind", ["device", "host"])
@pytest.mark.parametrize("dtype,d,F", [("bf16", 64, 64), ("bf16", 320, 576), ("bf16", 576, 256), ("f32", 64, 128),
                                       ("f32", 192, 64)])
def test_slots_hold_their_experts(pool_kind, dtype, d, F):
    from paper_2609_04895_amd import cmoe as B
    L, N, K, C, S, R = 5, 11, 2, 4, 2, 2
    say(f"copies: {dtype}, {pool_kind} pool, d={d} F={F}")
    dev = torch.device("cuda", 0)
    bf = dtype == "bf16"
    dt, raw = (torch.bfloat16, torch.int16) if bf else (torch.float32, torch.int32)
    w = torch.zeros((L, N, d), dtype=dt, device=dev)
    per = 3 * d * F
    gen = torch.Generator().manual_seed(5)
    bits = torch.randint(0, 2 ** 15, (L, N, per), generator=gen, dtype=torch.int32).to(raw)
    host = pool_kind == "host"
    pool = bits.view(dt).pin_memory() if host else bits.view(dt).to(dev)
    cfg = B.make_config(L, N, K, d, F, C, R, S, B.CMOE_MODE_SPATIO_TEMPORAL, B.CMOE_BF16 if bf else B.CMOE_F32,
                        B.CMOE_POOL_HOST_PINNED if host else B.CMOE_POOL_DEVICE)
    eng = B.Engine(cfg, w, w, w, None, pool)
    z = logits_sequence(np.random.default_rng(6), 4, S, L, N, ties=False)
    n_slots = min(N, S * C)
    src = bits.numpy().view(np.uint16 if bf else np.uint32)
    for t in range(4):  # proactive copies from the second token on
        eng.cmoe_step_logits(*(torch.from_numpy(z[t, i]).to(dev) for i in range(3)))
        slots = eng.cmoe_read(B.CMOE_VIEW_SLOTS)
        arena = eng.arena[: L * n_slots * per * (2 if bf else 4)].view(raw).cpu().numpy().view(src.dtype)
        arena = arena.reshape(L, n_slots, per)
        for l in range(L):
            for e in np.nonzero(slots[l] >= 0)[0]:
                x = src[l, e]
                if bf:
                    want = packed_from_plain(x, d, F)
                else:
                    want = np.concatenate([x[:F * d].reshape(F, d).T.ravel(), x[F * d:2 * F * d].reshape(F, d).T.ravel(),
                                           x[2 * F * d:].reshape(d, F).T.ravel()])
                assert np.array_equal(arena[l, slots[l, e]], want), (t, l, e)
    assert eng.cmoe_stats()[0]["proactive_loads"] > 0
    eng.cmoe_destroy()
