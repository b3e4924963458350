"""Register use of the kernels that a linear layer and a conversion run in one launch, compiled here with the resource-usage
remarks on (no GPU needed): nothing is spilled."""
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


@pytest.mark.parametrize("source,kernels", [("relu_fused.hip", 18), ("open_recode.hip", 4), ("mul_fused.hip", 8)])
def test_one_launch_kernels_do_not_spill(source, kernels):
    rows = usage(source)
    assert len(rows) == kernels, [r[0] for r in rows]
    for name, _, _, scratch in rows:
        assert scratch == 0, (name, scratch)
