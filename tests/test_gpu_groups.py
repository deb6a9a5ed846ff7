"""The F-stage's default antenna groups: one round of transforms or two, by size."""
import numpy as np
import pytest

import oracle
import paper_1102_0148_amd as corr
import synth
from test_gpu_parity import TOL, coef_error, raw_to_complex

pytestmark = pytest.mark.gpu


# (N, K, S, precision, group): padding that the rule takes and refuses, too few tiles, and
# counts that leave a group's last antennas out
@pytest.mark.parametrize("N,K,S,prec,group", [(44, 256, 1100, "fp32", 16), (20, 256, 1100, "fp32", 8),
                                              (40, 256, 700, "fp32", 16), (13, 512, 1030, "fp32", 8),
                                              (9, 512, 1030, "fp32", 8), (4, 512, 1030, "fp32", 4),
                                              (8, 512, 64, "fp32", 4), (5, 1024, 1030, "fp32", 4),
                                              (37, 1024, 131, "fp32", 4), (3, 1024, 1100, "fp16", 2),
                                              (37, 1024, 130, "fp16", 2), (3, 1024, 70, "fp16", 1)])
def test_default_groups(N, K, S, prec, group):
    print(f"\n[groups] N={N} K={K} S={S} {prec}", flush=True)
    packed = synth.packed(synth.recipe_plain(N=N, two_k=2 * K, rho=0.3, seed=N + K), 0, S).contiguous()
    c = corr.Correlator(N, K, S, precision=prec)
    c.process(packed.cuda())
    assert c.tiles()["f_group"] == group
    err = coef_error(raw_to_complex(c.read_cps_raw()), oracle.correlate(packed.numpy(), S, N, K), N)
    assert err <= TOL[corr.PRECISIONS[prec]]
    c.close()
