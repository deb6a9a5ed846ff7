"""The float X-stage's products as f16 halves against the f32 products.

corr_process multiplies its own float records as halves; the same records given
to corr_process_spectra are multiplied by the f32 matrix instructions.  Both are
held to the float64 sums of those very records."""
import numpy as np
import pytest
import torch

import paper_1102_0148_amd as corr
import synth

pytestmark = pytest.mark.gpu


# one to six blocks in one region, regions off the diagonal, whole-channel
# groups; sums of an odd number of steps, of one step and of several, splits
# that divide them unevenly, and spectra past the last whole record
@pytest.mark.parametrize("N,K,S,splits", [(17, 128, 64, 2), (33, 128, 67, 2), (48, 256, 203, 3), (64, 128, 128, 1),
                                          (80, 128, 101, 3), (96, 128, 96, 1), (130, 128, 97, 2), (193, 128, 33, 1),
                                          (256, 128, 49, 1), (256, 128, 240, 3), (300, 128, 65, 2)])
def test_halves_against_float64_of_the_records(N, K, S, splits):
    print(f"\n[halves] N={N} K={K} S={S} splits={splits}", flush=True)
    r = synth.recipe_sources(N=N, two_k=2 * K, seed=N + S)
    packed = synth.packed(r, 0, S, device="cuda").contiguous()
    c = corr.Correlator(N, K, S, tiles=dict(x_splits=splits, chunk_spectra=(S + 63) // 64 * 64))
    c.process(packed)
    buf, n = c.debug_read_spectra()
    assert n == S
    got = c.read_cps_raw()
    c.process_spectra(torch.from_numpy(buf).cuda(), S)
    f32 = c.read_cps_raw()
    x = corr.records_to_spectra(buf, corr.CORR_FP32, N, K, S).astype(np.complex128).transpose(2, 1, 0)  # [K][N][S]
    v = x @ x.conj().transpose(0, 2, 1)
    a, b = np.triu_indices(N)
    ref = v[:, a, b].T
    scale = np.sqrt(np.abs(v[:, a, a] * v[:, b, b])).T
    err = np.abs(got[..., 0] + 1j * got[..., 1] - ref) / scale
    # at most S / 16 roundings of a sum of at most the autocorrelations' size in
    # each component for each of three products, and 2^-22 of the products left out
    assert np.max(err) <= np.sqrt(2) * (3 * (S / 16 + 1) * 2.0 ** -24 + 2.0 ** -22)
    assert np.max(np.abs(f32[..., 0] + 1j * f32[..., 1] - ref) / scale) <= 1e-5
    assert np.all(got[a == b][..., 1] == 0.0)
    c.close()
