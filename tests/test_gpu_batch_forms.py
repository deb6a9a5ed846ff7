"""The persistent batch kernel multiplies a job's float records in the form a single correlator does."""
import numpy as np
import pytest

import paper_1102_0148_amd as corr
import synth

pytestmark = pytest.mark.gpu


# one block of antennas, few spectra and many to a partial, several regions to a channel
JOBS = [(12, 256, 640, "fp32"), (24, 256, 50, "fp32"), (44, 256, 100, "fp32"), (44, 256, 3000, "fp32"),
        (96, 128, 300, "fp32"), (130, 128, 70, "fp32"), (33, 1024, 40, "fp32")]


def test_persistent_float_jobs_are_the_single_ones():
    inputs = [synth.packed(synth.recipe_plain(N=N, two_k=2 * K, rho=0.3, seed=N + S), 0, S).contiguous().cuda()
              for N, K, S, _ in JOBS]
    b = corr.Batch(JOBS, mode="persistent")
    b.process(inputs)
    for j, (N, K, S, prec) in enumerate(JOBS):
        print(f"  job {j}: N={N} K={K} S={S}", flush=True)
        c = corr.Correlator(N, K, S, precision=prec, tiles=dict(chunk_spectra=(S + 63) // 64 * 64))
        c.process(inputs[j])
        # the same products in the same order: the same sums to the bit
        np.testing.assert_array_equal(b.read_cps_raw(j), c.read_cps_raw())
        c.close()
    b.close()
