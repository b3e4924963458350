"""Register use of the kernels that a linear layer and a conversion run in one launch, compiled here with the resource-usage
remarks on (no GPU needed): nothing is spilled, and which of them leave the room that another lane's GEMM wave (256 + 120 of
a SIMD's 512 registers) leaves a streaming wave, 136, is what their comments say."""
import os
import re
import subprocess

import pytest


def usage(source):
    import __graft_entry__ as ge
    out = subprocess.run([ge.HIPCC, *ge.HIP_FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
                          "-c", os.path.join(ge.CSRC, source), "-o", os.devnull], capture_output=True, text=True)
    assert out.returncode == 0, out.stderr[-2000:]
    rows = re.findall(r"Function Name: (\S+).*?VGPRs: (\d+).*?AGPRs: (\d+).*?ScratchSize \[bytes/lane\]: (\d+)", out.stderr, flags=re.S)
    names = subprocess.run(["c++filt"], input="\n".join(r[0] for r in rows), capture_output=True, text=True).stdout.splitlines()
    return [(n.replace("(anonymous namespace)::", ""), int(v), int(a), int(sc)) for n, (_, v, a, sc) in zip(names, rows)]


# kernels that need more than 136 registers, and the most they may need (168: three waves to a SIMD, 256: two)
WIDER = {"k_relu_fused<2, 2, 1, true>": 168, "k_relu_fused<3, 2, 0, false>": 168, "k_relu_fused_msb<2, true>": 168, "k_relu_fused_msb<2, false>": 168,
         "k_maxpool_fused<2, false, 1>": 168, "k_maxpool_fused<3, false, 0>": 168,
         "k_open_recode<2, (OpenPlanes)0>": 168, "k_open_recode<3, (OpenPlanes)2>": 168,
         "k_open_recode<2, (OpenPlanes)1>": 256, "k_open_recode<3, (OpenPlanes)1>": 256}


@pytest.mark.parametrize("source,kernels", [("relu_fused.hip", 18), ("open_recode.hip", 4), ("mul_fused.hip", 8)])
def test_one_launch_kernels(source, kernels):
    rows = usage(source)
    assert len(rows) == kernels, [r[0] for r in rows]
    for name, vgprs, agprs, scratch in rows:
        assert scratch == 0, (name, scratch)
        kernel = name.replace("void ", "").split(">(")[0] + ">"
        assert vgprs + agprs <= WIDER.get(kernel, 136), (name, vgprs, agprs)
