"""CPU: what the build makes of the compiler's report on registers."""
from paper_2508_06041_amd import build

REPORT = """gemv.hpp:1105:1: remark: Function Name: _Z1aPKc [-Rpass-analysis=kernel-resource-usage]
gemv.hpp:1105:1: remark:     TotalSGPRs: 81 [-Rpass-analysis=kernel-resource-usage]
gemv.hpp:1105:1: remark:     VGPRs: 128 [-Rpass-analysis=kernel-resource-usage]
gemv.hpp:1105:1: remark:     ScratchSize [bytes/lane]: %d [-Rpass-analysis=kernel-resource-usage]
gemv.hpp:1105:1: remark:     SGPRs Spill: 382 [-Rpass-analysis=kernel-resource-usage]
gemv.hpp:1105:1: remark:     VGPRs Spill: %d [-Rpass-analysis=kernel-resource-usage]
gemv.hpp:1105:1: remark:     LDS Size [bytes/block]: 65536 [-Rpass-analysis=kernel-resource-usage]
"""


def test_a_kernel_that_spills_vector_registers_is_named():
    whole, spills, scratch = REPORT % (0, 0), REPORT % (16, 3), REPORT % (8, 0)
    assert build.spilled("warning: something else\n" + whole) == []
    assert build.spilled(whole + spills.replace("_Z1a", "_Z1b") + whole + scratch.replace("_Z1a", "_Z1c")) == ["_Z1bPKc", "_Z1cPKc"]
