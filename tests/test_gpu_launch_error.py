"""A call that reports an error after its F-stage was enqueued leaves nothing behind for the next one."""
import pytest
import torch

import oracle
import paper_1102_0148_amd as corr
import synth
from test_gpu_parity import TOL, coef_error, raw_to_complex

pytestmark = pytest.mark.gpu


# A failed allocation leaves its error pending in the thread, and the next kernel launch
# reports it although the kernel runs: the F-stage of the first call below.
@pytest.mark.parametrize("prec,K", [("fp32", 128), ("fp16", 256)])
def test_process_after_a_reported_launch_error(prec, K):
    N, S = 5, 70
    packed = synth.packed(synth.recipe_plain(N=N, two_k=2 * K, rho=0.3, seed=4), 0, S).contiguous()
    x = packed.cuda()
    other = torch.randint(0, 256, packed.shape, dtype=torch.uint8, device="cuda")
    c = corr.Correlator(N, K, S, precision=prec)
    c.tiles()  # allocates
    huge = corr.Correlator(512, 1024, 1 << 24, tiles=dict(chunk_spectra=1 << 24))
    with pytest.raises(corr.CorrError):
        huge.tiles()  # 70 TB of records
    with pytest.raises(corr.CorrError) as e:
        c.process(other)
    assert e.value.code == corr.CORR_EHIP
    c.process(x)
    err = coef_error(raw_to_complex(c.read_cps_raw()), oracle.correlate(packed.numpy(), S, N, K), N)
    assert err <= TOL[corr.PRECISIONS[prec]]
    c.close()
    huge.close()
