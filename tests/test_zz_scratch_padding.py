"""corr_process_noalloc above 96 antennas, over scratch that reads as NaN where the records of
padding antennas lie: regions off the diagonal and whole-channel groups, float records as
halves among them."""
import numpy as np
import pytest
import torch

import paper_1102_0148_amd as corr
import synth
from test_zz_scratch_reuse import _call

pytestmark = pytest.mark.gpu


def _fill_with_codes():
    """Fill the scratch from 50 to 250 MB with 8-bit codes (48 antennas: no padding among them)."""
    N, K, S = 48, 256, 16384
    x = torch.randint(0, 256, (S, N, K), dtype=torch.uint8, device="cuda")
    c = corr.Correlator(N, K, 64, precision="int8")
    c.process(x[:64].contiguous())
    buf, _ = c.debug_read_spectra()
    c.close()
    assert np.isnan(buf.view(np.float32)).any() and np.isnan(buf.view(np.float16)).any()
    cps = torch.empty((N * (N + 1) // 2, K, 2), dtype=torch.float64, device="cuda")
    scales = torch.empty((N, K), dtype=torch.float32, device="cuda")
    corr.corr_process_noalloc(N, K, S, corr.CORR_INT8, x.data_ptr(), cps.data_ptr(), scales.data_ptr(),
                              torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()


# records from 70 MB on (an odd number of region rows) and from 123 MB on (16 blocks)
@pytest.mark.parametrize("prec", ["fp32", "fp16", "int8", "int16"])
@pytest.mark.parametrize("N,K,S", [(130, 128, 97), (200, 128, 70)])
def test_noalloc_over_padding_that_reads_as_nan(N, K, S, prec):
    print(f"\n[scratch padding] N={N} K={K} S={S} {prec}", flush=True)
    _fill_with_codes()
    x, got = _call(N, K, S, prec, 2)
    c = corr.Correlator(N, K, S, precision=prec)
    c.process(x)
    ref = c.read_cps_raw().reshape(got.shape)
    assert np.all(np.isfinite(got))
    if prec in ("int8", "int16"):
        np.testing.assert_array_equal(got, ref)
    else:  # the same products in other partials
        assert np.max(np.abs(got - ref)) <= 2.0 ** -24 * S * np.max(np.abs(ref))
    c.close()
