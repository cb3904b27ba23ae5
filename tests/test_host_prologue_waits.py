"""The key-split prefix kernel's first products wait for the queries and the first key tile and leave the younger tiles in flight:
checked in the assembly that the compiler makes of its source, since it adds waits of its own for the loads that it counts."""
import os
import re
import subprocess

from paper_2505_20776_amd import build


def test_first_products_leave_later_tiles_in_flight(tmp_path):
    out = str(tmp_path / "prefix_mfma.s")
    src = "prefix_mfma.hip"
    subprocess.run(build.compile_command(src) + ["--cuda-device-only", "-S", os.path.join(build.CSRC, src), "-o", out], check=True,
                   stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL, timeout=250)
    text = open(out).read()
    kernels = re.findall(r"^(\w*prefix_mfma_kernel\w*):", text, re.M)
    assert len(kernels) == 2
    for name in kernels:
        body = text[text.index(name + ":"):]
        lines = body[:body.index("s_endpgm")].splitlines()
        products = [i for i, line in enumerate(lines) if "v_mfma" in line]
        # the eight products of the first tile's logits stand first, behind the loads of the prologue
        waits = [int(n) for line in lines[:products[7]] for n in re.findall(r"s_waitcnt.*vmcnt\((\d+)\)", line)]
        # at the least V0 (eight loads) is in flight: a split of one tile per wave
        assert waits and min(waits) == 8, (name, waits)
        assert not any(re.search(r"global_load_dword|flat_load", line) for line in lines[:products[0]]), name
