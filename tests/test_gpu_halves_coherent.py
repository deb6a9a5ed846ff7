"""Float records as f16 halves on a coherent signal: the same block in every spectrum, so that
what a product is off by does not average out over them."""
import numpy as np
import pytest
import torch

import paper_1102_0148_amd as corr

pytestmark = pytest.mark.gpu


def _tone(N, K, S, seed):
    """Packed samples of a tone between two bins, of another phase in every antenna."""
    rng = np.random.default_rng(seed)
    n = np.arange(2 * K)
    x = 6.5 * np.cos(2 * np.pi * (rng.uniform(0.1, 0.9) * n / 2 + rng.uniform(0, 1, (N, 1))))
    x = np.clip(np.rint(x), -8, 7).astype(np.int64)
    block = ((x[:, 0::2] & 15) | ((x[:, 1::2] & 15) << 4)).astype(np.uint8)
    return torch.from_numpy(np.broadcast_to(block, (S, N, K)).copy())


# two and three blocks of antennas, off-diagonal regions, whole-channel groups; 64 partials
# of 32 spectra, which add up in float64
@pytest.mark.parametrize("N,K", [(17, 128), (44, 256), (90, 128), (130, 128), (200, 128)])
def test_halves_on_a_repeated_tone(N, K):
    S, splits = 2048, 64
    c = corr.Correlator(N, K, S, tiles=dict(x_splits=splits, chunk_spectra=S))
    c.process(_tone(N, K, S, N).cuda())
    buf, n = c.debug_read_spectra()
    assert n == S
    got = c.read_cps_raw()
    x = corr.records_to_spectra(buf, corr.CORR_FP32, N, K, S).astype(np.complex128)[0]  # [N][K]
    assert np.all(corr.records_to_spectra(buf, corr.CORR_FP32, N, K, S) == x)
    a, b = np.triu_indices(N)
    err = np.abs(got[..., 0] + 1j * got[..., 1] - S * x[a] * x[b].conj()) / S
    m = np.abs(x)
    # Per product of two components, the operands' 2^-23 each (2^-25 of a component below 1/4)
    # and the 2^-22 of the lower halves' product; in each of the two components of a sum,
    # roundings of three products over the two steps of a partial and of the sums combined.
    of_products = 2 * 2.0 ** -23 + 2.0 ** -22 + 3 * 3 * 2.0 ** -24
    bound = np.sqrt(2) * (2 * of_products * m[a] * m[b] + 2 * 2.0 ** -25 * (m[a] + m[b]))
    assert np.all(err <= bound)
    assert np.all(got[a == b][..., 1] == 0.0)
    c.close()
