"""The X-stage's sums do not depend on what the records of padding antennas hold."""
import numpy as np
import pytest
import torch

import paper_1102_0148_amd as corr

pytestmark = pytest.mark.gpu


# one, eight and nine antennas in the last block (a line of 8 alone, full, both), of one to
# six blocks, regions, groups and whole channels
@pytest.mark.parametrize("prec", ["fp32", "fp16", "int8", "int16"])
@pytest.mark.parametrize("N", [2, 8, 9, 17, 24, 41, 49, 65, 89, 97, 136, 200])
def test_padding_records_do_not_matter(N, prec):
    K, S = 128, 70
    rng = np.random.default_rng(N)
    if prec in ("int8", "int16"):
        q = rng.integers(-127, 128, (S, N, K, 2)).astype(np.int8 if prec == "int8" else np.int16)
    else:
        q = (rng.standard_normal((S, N, K)) + 1j * rng.standard_normal((S, N, K))).astype(np.complex64)
    code = corr.PRECISIONS[prec]
    buf = corr.spectra_to_records(q, code)
    bad = buf.copy()
    bad.view(np.uint8).reshape(-1, K, corr.TQB, corr.a_pad_of(N), 16)[:, :, :, N:] = 0xFF  # NaN as floats
    out = []
    for b in (buf, bad):
        c = corr.Correlator(N, K, S, precision=prec)
        c.process_spectra(torch.from_numpy(b).cuda(), S)
        out.append(c.read_cps_raw())
        c.close()
    assert np.all(np.isfinite(out[0]))
    np.testing.assert_array_equal(out[0], out[1])
