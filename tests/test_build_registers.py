"""The build refuses kernels with accumulation registers."""
import pytest

from paper_2304_05639_amd import build

TAG = " [-Rpass-analysis=kernel-resource-usage]"


def _remarks(kernel, agprs):
    at = "csrc/x.hip:98:1: remark: "
    return [at + f"Function Name: {kernel}" + TAG, "   98 | {", "      | ^", at + "    VGPRs: 46" + TAG,
            at + f"    AGPRs: {agprs}" + TAG, at + "    VGPRs Spill: 0" + TAG]


def test_remarks_are_read_and_removed():
    text = _remarks("_Z1av", 0) + ["csrc/x.hip:7:3: warning: unused variable 'y' [-Wunused-variable]", "    7 |   int y;",
                                   "      |       ^"] + _remarks("_Z1bv", 12)
    agprs, rest = build.split_remarks("\n".join(text))
    assert agprs == {"_Z1av": 0, "_Z1bv": 12}
    assert rest.splitlines() == text[6:9]
    with pytest.raises(RuntimeError, match="_Z1bv"):
        build.check_registers(agprs)
    build.check_registers({"_Z1av": 0})


def test_build_asks_for_the_remarks():
    assert "-Rpass-analysis=kernel-resource-usage" in build.COMMON
