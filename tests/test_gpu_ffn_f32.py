"""fp32 expert FFN on the fp32 matrix core against the fp64 oracle, at bucket
sizes around its token groups (one group of up to 16, passes of 32, units of 64
or 128 tokens) and k ranges that its four wavefronts split unevenly or that
leave some of them without work."""
import pytest

import synth
from test_gpu_e2e_parity import run_e2e

pytestmark = pytest.mark.gpu

# one fp32 rounding per product and add, a tree of four chains: the relative
# error of a sum of n <= 704 terms stays far below n 2^-24 = 4e-5; the
# sequential sums that the fp32 path had before were held to 1e-5
TOL = 1e-5


@pytest.mark.parametrize("S,N,K,d,F,shape", [
    (1, 4, 1, 64, 64, None),        # one token; four blocks of k, one a wavefront
    (3, 3, 2, 704, 192, None),      # 44 and 12 blocks
    (17, 2, 1, 128, 64, None),      # buckets around 16
    (33, 2, 2, 64, 128, "single"),  # 33 tokens in both buckets: a pass of 32 and one of 1
    (150, 2, 1, 192, 64, "single"),  # units of 64: passes of 32 and a rest
    (150, 2, 2, 64, 320, "grouped"),  # 150 tokens: units of 128 and 22
])
def test_fp32_ffn(S, N, K, d, F, shape):
    w = synth.WORKLOADS["tiny"].replace(name=f"f32_{S}_{N}_{K}_{d}_{F}", L=2, N=N, K=K, d=d, F=F, S=S, C=K)
    run_e2e(w, T=2, tol=TOL, ffn_shape=shape)
