"""What the compiler makes of the kernels: no instance keeps registers in scratch memory (a spill to it is traffic the
kernel pays for on every launch, and a kernel that needs scratch may make the runtime allocate some)."""
import os
import re
import subprocess

import pytest

from paper_2512_24086_amd import build as b


@pytest.mark.parametrize("source", ["rf2_attn.hip", "rf2_mask.hip", "rf2_permute.hip"])
def test_no_instance_uses_scratch_memory(source, tmp_path):
    out = subprocess.run([b.hipcc(), *b.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                          os.path.join(b.CSRC, source), "-o", str(tmp_path / "device.o")], check=True, capture_output=True, text=True)
    found = re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+).*?VGPRs Spill: (\d+)", out.stderr, re.S)
    assert len(found) >= 10
    assert not [f for f in found if f[1:] != ("0", "0")]
