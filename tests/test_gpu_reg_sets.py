"""The register transform's sets of four units as workgroups take them: the first two rounds
by rank, what is left by ticket."""
import numpy as np
import pytest

import oracle
import paper_1102_0148_amd as corr
import synth

pytestmark = pytest.mark.gpu


# 8 antennas are one set a record of 8 spectra, 512 workgroups: a set short of a round, one
# round, one past it, two rounds, past them, and tickets for half a round
@pytest.mark.parametrize("S", [4088, 4096, 4160, 8192, 8256, 10300])
def test_every_set_is_transformed(S):
    N, K = 8, 256
    packed = synth.packed(synth.recipe_plain(N=N, two_k=2 * K, rho=0.3, seed=S), 0, S).contiguous()
    c = corr.Correlator(N, K, S, precision="int8", tiles=dict(chunk_spectra=(S + 63) // 64 * 64))
    x = packed.cuda()
    for _ in range(2):  # the second over the first one's tickets
        c.process(x)
        buf, n = c.debug_read_spectra()
        assert n == S
        q = corr.records_to_spectra(buf, corr.CORR_INT8, N, K, S)
        diff = q.astype(np.int32) - oracle.quantise(oracle.spectra(packed.numpy(), S, N, K), c.read_scales()).astype(np.int32)
        assert np.max(np.abs(diff)) <= 1 and np.mean(diff != 0) <= 1e-3
        np.testing.assert_array_equal(c.read_cps_raw(), oracle.cmac_i64(q).astype(np.float64))
    c.close()
