"""corr_process_noalloc over whatever the last call left in its scratch: nothing of it is cleared."""
import numpy as np
import pytest
import torch

import paper_1102_0148_amd as corr
import synth

pytestmark = pytest.mark.gpu


def _call(N, K, S, prec, seed):
    x = synth.packed(synth.recipe_plain(N=N, two_k=2 * K, rho=0.3, seed=seed), 0, S, device="cuda").contiguous()
    cps = torch.full((N * (N + 1) // 2, K, 2), float("nan"), dtype=torch.float64, device="cuda")
    scales = torch.zeros((N, K), dtype=torch.float32, device="cuda")
    corr.corr_process_noalloc(N, K, S, corr.PRECISIONS[prec], x.data_ptr(), cps.data_ptr(), scales.data_ptr(),
                              torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return x, cps.cpu().numpy()


# spectra that end inside a record and a step, one past a step, several chunks; antennas
# with whole lines of padding
@pytest.mark.parametrize("prec", ["fp32", "fp16", "int8", "int16"])
@pytest.mark.parametrize("N,K,S", [(5, 128, 9), (17, 256, 70), (35, 512, 33), (20, 1024, 129), (65, 256, 41),
                                   (90, 512, 1100)])
def test_noalloc_over_a_full_scratch(N, K, S, prec):
    print(f"\n[scratch reuse] N={N} K={K} S={S} {prec}", flush=True)
    _call(96, 512, 600, "fp32", 1)  # fills the scratch with other records and sums
    x, got = _call(N, K, S, prec, 2)
    c = corr.Correlator(N, K, S, precision=prec)
    c.process(x)
    ref = c.read_cps_raw().reshape(got.shape)
    if prec in ("int8", "int16"):
        np.testing.assert_array_equal(got, ref)
    else:  # the same products in other partials
        assert np.max(np.abs(got - ref)) <= 2.0 ** -24 * S * np.max(np.abs(ref))
    c.close()
