"""No scratch memory in the kernels that a denoising step runs at the register limit: a value that the compiler spills is
written and read per lane in the middle of a loop. From the compiler's own resource report for the sources (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2604_04451_amd import build


def _scratch(source, tmp_path):
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(build.CSRC, source), "-o", str(tmp_path / "k.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    sizes = [int(v) for v in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert names and len(names) == len(sizes)
    return dict(zip(names, sizes))


@pytest.mark.parametrize("source,kernels,at_least", [
    ("glue.hip", r"head_update_kernel", 18),  # six widths, three updates
    ("gemm.hip", r"gemm_w16_kernel", 26),  # five tiles and the far one, four epilogues; two tiles with a second product
    # all but plain queries with factors over 512 keys or more, which a block does not run
    ("attention.hip", r"attention_pp16_kernelILi\d+E(?!Lb0ELi2ELi2E)", 38),
])
def test_no_scratch(source, kernels, at_least, tmp_path):
    got = {n: v for n, v in _scratch(source, tmp_path).items() if re.search(kernels, n)}
    assert len(got) >= at_least, sorted(got)
    assert not {n: v for n, v in got.items() if v}
