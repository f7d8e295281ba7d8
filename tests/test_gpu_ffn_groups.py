"""bf16 FFN of units of more than 16 tokens against the fp64 oracle, at the
edges of the token groups (16, 32, 64, 96, 128 and a second unit of one), with
row tiles that leave wavefronts of the last workgroup without work (d = 192:
six 32-row tiles, F = 192: twelve 16-row tiles, of eight) and k loops that do
not divide by the chunk blocks; below 64 tokens per expert all units share one
launch, from 64 on the big ones have their own."""
import pytest

import synth
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


@pytest.mark.parametrize("S,N,K,zipf", [(220, 5, 1, 1.1), (400, 6, 2, 1.1), (90, 4, 3, 0.0)])
def test_mixed_units(S, N, K, zipf):
    # hot experts of 65 to 128 tokens in the shared launch; units of 128 with
    # last passes of either list; buckets of 60 to 75 on both sides of 64
    w = synth.WORKLOADS["qwen3_30b"].replace(name=f"mixed_{S}_{N}_{K}", L=2, N=N, K=K, d=192, F=128, S=S, C=K,
                                             zipf=zipf or None)
    run_e2e(w, T=2, tol=2e-2)
