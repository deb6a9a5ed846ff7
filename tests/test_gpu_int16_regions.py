"""int16 X-stage: every region of a channel in one launch, single-block regions included."""
import numpy as np
import pytest
import torch

import oracle
import paper_1102_0148_amd as corr

pytestmark = pytest.mark.gpu


# 4 blocks (2-block regions) just past three, 5 blocks (single-block regions) first and
# full, 6 blocks, 8 blocks with a padded region; splits that leave waves past the end
@pytest.mark.parametrize("N,K,S,splits", [(49, 128, 40, 1), (65, 128, 70, 3), (80, 128, 32, 2), (96, 128, 33, 1),
                                          (113, 128, 65, 2)])
def test_int16_regions_in_one_launch(N, K, S, splits):
    rng = np.random.default_rng(N + S)
    q = rng.integers(-32512, 32513, (S, N, K, 2)).astype(np.int16)
    q[rng.random(q.shape) < 0.02] = -32512
    buf = torch.from_numpy(corr.spectra_to_records(q, corr.CORR_INT16)).cuda()
    c = corr.Correlator(N, K, S, precision="int16", tiles=dict(x_splits=splits))
    c.process_spectra(buf, S)
    np.testing.assert_array_equal(c.read_cps_raw(), oracle.cmac_i64_16(q).astype(np.float64))
    c.close()
