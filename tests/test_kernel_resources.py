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


def test_four_workgroups_of_the_mask_kernel(tmp_path):
    """At d = 64 LDS holds four workgroups of eight wavefronts for rows of up to 512 columns, which is eight wavefronts per SIMD:
    1/8 of its 512 vector registers each, and of its 800 scalar ones in steps of 16, less 16 for the trap handler."""
    out = subprocess.run([b.hipcc(), *b.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                          os.path.join(b.CSRC, "rf2_mask.hip"), "-o", str(tmp_path / "device.o")], check=True, capture_output=True, text=True)
    found = re.findall(r"Function Name: \S+predict_mask_kernelILi64ELi([2468])ELb0ELi8E.*?TotalSGPRs: (\d+).*?VGPRs: (\d+)", out.stderr, re.S)
    assert len(found) == 4
    assert all(int(s) <= 80 and int(v) <= 64 for _, s, v in found), found


def test_lanes_of_the_mask_kernel_exchange_keys_in_order(tmp_path):
    """Lanes turn a tile of K through LDS: whatever one writes 16 bytes at a time another may read next, so a barrier of the
    wavefront or the workgroup stands between every such write and the next such read of the compiled code, in each instance, and
    behind the read of a tile's chunk, whose place the next chunk takes."""
    out = tmp_path / "mask.s"
    subprocess.run([b.hipcc(), *b.FLAGS, "--cuda-device-only", "-S", os.path.join(b.CSRC, "rf2_mask.hip"), "-o", str(out)], check=True,
                   capture_output=True)
    kernels = re.findall(r"^(\S*predict_mask_kernelILi(\d+)\S*):(.*?)^\.Lfunc_end", out.read_text(), re.S | re.M)
    assert len(kernels) == 80
    for name, d, body in kernels:
        events = re.findall(r"\b(ds_write_b128|ds_read_b128|s_barrier|wave barrier)\b", body)
        writes = [i for i, e in enumerate(events) if e == "ds_write_b128"]
        assert len(writes) >= int(d) // 16, name
        for i in writes:
            rest = [e for e in events[i + 1:] if e != "ds_write_b128"]
            assert rest[0] != "ds_read_b128", name
        assert events.count("wave barrier") == 2 * (int(d) // 16), name
