"""bf16 FFN of units of more than 16 tokens against the fp64 oracle, at the
edges of the token groups (16, 32, 64, 96, 128 and a second unit of one), with
row tiles that leave wavefronts of the last workgroup without work (d = 192:
six 32-row tiles, F = 192: twelve 16-row tiles, of eight) and k loops that do
not divide by the chunk blocks; below 64 tokens per expert all units share one
launch, from 64 on the big ones have their own."""
import numpy as np
import pytest

import synth
from gpu_util import host_routers, oracle_logits
from test_gpu_e2e_parity import run_e2e

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,d,F", [(16, 192, 192), (17, 192, 192), (32, 64, 64), (33, 320, 192), (63, 192, 320),
                                   (64, 192, 192), (65, 192, 192), (96, 64, 64), (97, 320, 192), (128, 192, 320),
                                   (129, 192, 192), (161, 192, 64)])
def test_one_expert_takes_every_token(S, d, F):
    w = synth.WORKLOADS["qwen3_30b"].replace(name=f"groups_{S}_{d}_{F}", L=1, N=1, K=1, d=d, F=F, S=S, C=1)
    # bf16 SwiGLU intermediate and gated outputs (2^-9 each) on sums of d and F
    # products: the library's bf16 tolerance
    run_e2e(w, T=1, tol=2e-2, ffn_shape="grouped")


def bucket_sizes(w, T):
    """Tokens per executed expert of every layer step, from the oracle's logits."""
    WR, WT, WS = host_routers(w)
    bias = synth.zipf_bias(w)
    H = {(s, l): synth.hidden_host(w, s, l, T=T) for s in range(w.S) for l in range(w.L)}
    sizes = set()
    for t in range(T):
        z = oracle_logits(w, WR, WT, WS, bias, H, t, range(w.S))[:, :, 0]
        sel = np.argsort(-z, axis=-1, kind="stable")[:, :, :w.K]
        for l in range(w.L):
            sizes |= set(np.bincount(sel[:, l].ravel(), minlength=w.N).tolist())
    return sizes - {0}


def last_passes(sizes):
    """Tokens of the last work unit of each bucket that takes several (128 each)."""
    return {(m - 1) % 128 + 1 for m in sizes if m > 128}


# what each case is there for, as a condition on its bucket sizes
MIXED = [
    # one launch for all units: hot experts of 65 to 127 tokens; of 128 and a rest
    (150, 5, 1, 1.1, lambda m: any(64 < n < 128 for n in m) and any(16 < n <= 32 for n in m)),
    (220, 5, 1, 1.1, lambda m: any(16 < n < 32 for n in last_passes(m)) and any(n > 32 for n in last_passes(m))),
    # launches of their own for the big units: last passes of either list
    (250, 6, 2, 1.1, lambda m: any(n <= 16 for n in last_passes(m)) and any(n > 96 for n in last_passes(m))),
    (400, 6, 2, 1.1, lambda m: max(m) > 256 and 32 in m and any(32 < n <= 64 for n in m) and any(n < 16 for n in m)),
    # big units only, buckets on both sides of 64
    (90, 4, 3, 0.0, lambda m: min(m) > 32 and any(n <= 64 for n in m) and any(64 < n <= 96 for n in m)),
]


@pytest.mark.parametrize("S,N,K,zipf,covers", MIXED, ids=[f"{c[0]}-{c[1]}-{c[2]}" for c in MIXED])
def test_mixed_units(S, N, K, zipf, covers):
    w = synth.WORKLOADS["qwen3_30b"].replace(name=f"mixed_{S}_{N}_{K}", L=2, N=N, K=K, d=192, F=128, S=S, C=K,
                                             zipf=zipf or None)
    sizes = bucket_sizes(w, 2)
    assert covers(sizes), sorted(sizes)
    run_e2e(w, T=2, tol=2e-2)
