"""Registers of the merge kernel, as the compiler reports them: the part for deep trees may not cost the others their waves per SIMD
(a launch of 128 nodes of 32 heads has four workgroups per compute unit, of 64 heads eight, each a wave on every SIMD)."""
import os
import re
import subprocess

from paper_2505_20776_amd import build

# (head_dim, bf16 inputs, fp16 partials, splits per wave): waves per SIMD at the least
LEAST = {(128, 1, 1, 1): 7, (128, 1, 1, 2): 7, (128, 1, 1, 4): 6, (128, 1, 1, 8): 5, (128, 1, 1, 16): 4,
         (128, 0, 0, 1): 5, (128, 0, 0, 2): 4, (128, 0, 0, 4): 4, (128, 0, 0, 8): 3, (128, 0, 0, 16): 2,
         (64, 1, 0, 1): 8, (64, 1, 0, 2): 8, (64, 1, 0, 4): 8, (64, 0, 0, 1): 8, (64, 0, 0, 2): 7}


def test_waves_per_simd(tmp_path):
    src = "tree_merge.hip"
    run = subprocess.run(build.compile_command(src) + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                                                       os.path.join(build.CSRC, src), "-o", str(tmp_path / "merge.o")],
                         stdout=subprocess.DEVNULL, stderr=subprocess.PIPE, text=True, timeout=250)
    assert run.returncode == 0, run.stderr[-4000:]
    seen = {}
    for block in run.stderr.split("Function Name: ")[1:]:
        form = re.match(r"\S*tree_merge_shared_kernelILi(\d+)ELb(\d)ELb(\d)ELi(\d+)", block)
        if form:
            assert re.search(r"ScratchSize \[bytes/lane\]: 0\b", block), block[:200]
            seen[tuple(map(int, form.groups()))] = int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", block).group(1))
    for form, least in LEAST.items():
        assert seen[form] >= least, (form, seen[form])
