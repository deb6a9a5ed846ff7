"""The F groups that the tuner times (CPU)."""
import pytest

from paper_1102_0148_amd import tune


# records that the register transform makes have one group; the others every one that fits
@pytest.mark.parametrize("K,prec,expect", [(256, "fp16", [4]), (256, "int8", [2]), (256, "int16", [4]), (512, "fp16", [2]),
                                           (512, "int8", [1]), (512, "int16", [2]), (256, "fp32", [1, 2, 4, 8, 16]),
                                           (1024, "fp16", [1, 2, 4]), (128, "int8", [1, 2, 4, 8, 16])])
def test_groups(K, prec, expect):
    assert tune.groups_to_time(K, prec) == expect
    # the library takes others too
    assert set(expect) <= {c["f_group"] for c in tune.candidates(44, K, 4096, prec)} == set(tune.groups(K, prec))
