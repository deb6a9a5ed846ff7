"""The fused pipeline's partials: how many spectra one of them sums."""
import numpy as np
import pytest

import oracle
import paper_1102_0148_amd as corr
import synth
from test_gpu_parity import TOL, coef_error, raw_to_complex

pytestmark = pytest.mark.gpu


# fp32 units take whole steps of 16 spectra, so a chunk of 4 steps over 8 units gives some of
# them 16 spectra of every chunk; layouts of 8, 23 and 9 units that do not divide the steps
@pytest.mark.parametrize("K,chunks,chunk,f_cus", [(128, 256, 64, 0), (128, 85, 192, 0), (128, 28, 1536, 1),
                                                  (256, 36, 448, 8)])
def test_fp32_partials_sum_at_most_2048_spectra(K, chunks, chunk, f_cus):
    N, S = 3, chunks * chunk
    packed = synth.packed(synth.recipe_plain(N=N, two_k=2 * K, rho=0.3, seed=K), 0, S).contiguous()
    c = corr.Correlator(N, K, S, pipeline=dict(chunk_spectra=chunk, f_cus_per_xcd=f_cus))
    t = c.tiles()
    one = corr.Correlator(N, K, chunk, pipeline=dict(chunk_spectra=chunk, f_cus_per_xcd=f_cus))
    nsplit = one.tiles()["x_splits"]  # units per channel
    one.close()
    steps = -(-chunk // 16)
    of_a_chunk = -(-steps // nsplit) * 16
    assert t["chunk_spectra"] == chunk and t["x_splits"] % nsplit == 0
    epochs = t["x_splits"] // nsplit
    assert -(-chunks // epochs) * of_a_chunk <= 2048
    c.process(packed.cuda())
    err = coef_error(raw_to_complex(c.read_cps_raw()), oracle.correlate(packed.numpy(), S, N, K), N)
    assert err <= TOL[corr.CORR_FP32]
    c.close()


# partials of under 32 spectra: products of the staged pipeline's form, the same sums to the bit
# (one k-block of 8 spectra, three, and all of a channel's to a unit)
@pytest.mark.parametrize("N,K,S", [(8, 128, 64), (17, 128, 64), (44, 128, 64), (33, 512, 48), (20, 1024, 24)])
def test_fp32_short_partials_are_the_staged_ones(N, K, S):
    x = synth.packed(synth.recipe_plain(N=N, two_k=2 * K, rho=0.3, seed=N), 0, S).contiguous().cuda()
    c = corr.Correlator(N, K, S, pipeline="fused")
    splits = c.tiles()["x_splits"]
    assert S < 32 * splits
    s = corr.Correlator(N, K, S, tiles=dict(x_splits=splits))
    c.process(x)
    s.process(x)
    np.testing.assert_array_equal(c.read_cps_raw(), s.read_cps_raw())
    c.close()
    s.close()
