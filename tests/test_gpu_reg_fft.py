"""The register transform of the reduced-precision records (512- and 1024-point): the
units' split into sets of four, their remainders and the padding, against the oracle."""
import math

import numpy as np
import pytest

import oracle
import paper_1102_0148_amd as corr
import synth

pytestmark = pytest.mark.gpu


# antenna groups of 1, 2 or 4: counts with every remainder over four, fewer than four, one
# antenna past a group, past a line and past a block; spectra that end inside a record,
# inside a set's time records, and past a time block
@pytest.mark.parametrize("prec", ["fp16", "int8", "int16"])
@pytest.mark.parametrize("N,K,S", [(2, 256, 1), (3, 512, 9), (5, 256, 33), (7, 512, 129), (11, 256, 70), (13, 256, 200),
                                   (18, 512, 40), (23, 256, 131), (37, 512, 65), (45, 256, 129), (97, 256, 20),
                                   (100, 512, 33)])
def test_register_transform_records(N, K, S, prec):
    print(f"\n[register transform] N={N} K={K} S={S} {prec}", flush=True)
    r = synth.recipe_tone(N=N, two_k=2 * K, seed=N + S, tone_bin=K // 2 + 3)
    packed = synth.packed(r, 0, S).contiguous()
    c = corr.Correlator(N, K, S, precision=prec, tiles=dict(chunk_spectra=(S + 63) // 64 * 64))
    c.process(packed.cuda())
    buf, n = c.debug_read_spectra()
    assert n == S
    got = corr.records_to_spectra(buf, c.precision, N, K, S)
    ref = oracle.spectra(packed.numpy(), S, N, K)
    # the float32 transform's error budget, of the spectrum's rms
    budget = 2e-6 * np.sqrt(np.mean(np.abs(ref) ** 2)) * math.log2(2 * K)
    if prec == "fp16":
        for g, x in ((got.real, ref.real), (got.imag, ref.imag)):
            step = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(x), 2.0 ** -14))) - 10)
            assert np.all(np.abs(g - x) <= 0.5 * step + budget)
        for b in (0, K // 2):  # integers below 2048 here
            np.testing.assert_array_equal(got[:, :, b], ref[:, :, b].round())
    else:
        lim, scales = (127, c.read_scales()) if prec == "int8" else (32512, c.read_scales())
        x = np.stack([ref.real, ref.imag], axis=-1) * scales[None, :, :, None].astype(np.float64)
        room = 0.5 + budget * scales[None, :, :, None] + np.abs(x) * 2.0 ** -23  # rounding, the transform, the float product
        assert np.all(np.abs(got - np.clip(x, -lim, lim)) <= room)
        raw = c.read_cps_raw()
        exact = oracle.cmac_i64(got) if prec == "int8" else oracle.cmac_i64_16(got)
        np.testing.assert_array_equal(raw, exact.astype(np.float64))
    dt = {"fp16": np.float16}.get(prec, np.int8)
    rec = buf.view(dt).reshape(-1, K, corr.TQB, corr.a_pad_of(N), 16 // np.dtype(dt).itemsize)
    assert np.all(rec[:, :, :, N:] == 0)
    c.close()


# layouts of three workgroups per CU, cut to what two can run: a second F workgroup, X
# waves fewer than channels, a chunk above what its partials may sum
@pytest.mark.parametrize("K,S,layout", [(256, 130, dict(f_workgroups_per_cu=2)), (512, 130, dict(f_workgroups_per_cu=2)),
                                        (256, 130, dict(f_cus_per_xcd=29)), (512, 130, dict(f_cus_per_xcd=26)),
                                        (256, 65536, dict(f_cus_per_xcd=20, chunk_spectra=65536))])
def test_fused_layouts_of_three_workgroups(K, S, layout):
    N = 3
    r = synth.recipe_tone(N=N, two_k=2 * K, seed=K, tone_bin=K // 2 + 3)
    x = synth.packed(r, 0, S).contiguous().cuda()
    for prec in ("fp16", "int8"):
        print(f"\n[fused layout] K={K} S={S} {prec} {layout}", flush=True)
        c = corr.Correlator(N, K, S, precision=prec, pipeline=layout)
        c.process(x)
        s = corr.Correlator(N, K, S, precision=prec)
        s.process(x)
        a, b = c.read_cps_raw(), s.read_cps_raw()
        if prec == "int8":
            np.testing.assert_array_equal(a, b)
        else:  # float32 partials of the same products, in another order
            assert np.max(np.abs(a - b)) <= 2.0 ** -24 * 16384 * np.max(np.abs(b)) / 64
    for bad in (dict(f_workgroups_per_cu=3), dict(f_cus_per_xcd=31 if K == 256 else 30)):
        c = corr.Correlator(N, K, 64, precision="int8", pipeline=bad)
        with pytest.raises(corr.CorrError) as e:
            c.process(x[:64])
        assert e.value.code == corr.CORR_EINVAL
