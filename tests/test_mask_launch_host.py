"""LDS of the mask kernel's launches at every width, on the host: no more than a strip of keys, the Q operand and the rows'
sums take (a workgroup more or less on a compute unit is a quarter of the time), and enough for the last row's reads of keys."""
import os
import re
import subprocess

from paper_2512_24086_amd import build as b

LDS = 160 * 1024            # of a compute unit


def static_lds(folder):
    """(head_dim, wavefronts, cumulative mass) -> {keys per lane: bytes that the instance itself declares}"""
    out = subprocess.run([b.hipcc(), *b.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                          os.path.join(b.CSRC, "rf2_mask.hip"), "-o", str(folder / "device.o")], check=True, capture_output=True, text=True)
    found = {}
    for d, width, cdf, nw, size in re.findall(
            r"Function Name: \S+predict_mask_kernelILi(\d+)ELi(\d+)ELb(\d)ELi(\d+)E.*?LDS Size \[bytes/block\]: (\d+)", out.stderr, re.S):
        found.setdefault((int(d), int(nw), int(cdf)), {})[int(width)] = int(size)
    return found


def test_lds_of_every_width(tmp_path):
    objs = [os.path.join(b.PKG, "_build", os.path.splitext(s)[0] + ".o") for s in b.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        b.build(verbose=False)
    exe = str(tmp_path / "mask_launch")
    here = os.path.dirname(os.path.abspath(__file__))
    subprocess.run([b.hipcc(), *b.FLAGS, "-c", os.path.join(here, "mask_launch_host.cpp"), "-o", str(tmp_path / "driver.o")],
                   check=True, capture_output=True)
    subprocess.run([b.hipcc(), "--offload-arch=gfx950", str(tmp_path / "driver.o"), *objs, "-o", exe], check=True, capture_output=True)
    rows = [tuple(map(int, line.split())) for line in
            subprocess.run([exe], check=True, capture_output=True, text=True, timeout=300).stdout.splitlines()]
    assert len(rows) == 2 * 2 * 128 * 2
    static = static_lds(tmp_path)
    assert len(static) == 8 and all(len(s) == 10 for s in static.values())
    resident = {}
    for d, heads, columns, mode, threads, dynamic, limit in rows:
        wavefronts = threads // 64
        of = static[d, wavefronts, mode]
        width = min(w for w in of if 64 * w >= columns)
        pitch, case = columns + 4, (d, heads, columns, mode)
        total = of[width] + dynamic
        assert total == 4 * (16 * pitch + 16 * (d + 4) + 2 * 16 * wavefronts), case
        assert 15 * pitch + 64 * width <= dynamic // 4, case
        assert dynamic <= 32 * 1024 or limit == dynamic, case
        resident[d, wavefronts, columns] = LDS // total
    # (the widest rows that leave room for three and for two workgroups, by the bytes)
    for d, of_three, of_two in ((64, 752, 1184), (128, 688, 1120)):
        assert [resident[d, 8, of_three + x] for x in (0, 16)] == [3, 2]
        assert [resident[d, 8, of_two + x] for x in (0, 16)] == [2, 1]
