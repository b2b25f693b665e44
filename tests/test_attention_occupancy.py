"""Every instantiation of the attention kernels of many queries leaves room for two workgroups of four waves per CU (two waves per SIMD) and
spills nothing: the compiler's own resource report at the library's flags."""
import os
import re
import subprocess

from paper_2305_17423_amd import build


def test_attention_kernels_run_two_waves_per_simd(tmp_path):
    src = os.path.join(build.CSRC, "attention.hip")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-Rpass-analysis=kernel-resource-usage", "--offload-device-only", "-x", "hip",
                        "-c", src, "-o", str(tmp_path / "attention.co")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    kernels = {}
    for l in r.stderr.splitlines():
        m = re.search(r"remark:.*?(Function Name|ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]): (\S+)", l)
        if not m:
            continue
        if m.group(1) == "Function Name":
            name = m.group(2)
        elif "attention_kernel" in name or "attention_turns_kernel" in name:
            kernels.setdefault(name, {})[m.group(1).split()[0]] = int(m.group(2))
    assert len(kernels) >= 13 and sum("turns" in k for k in kernels) == 3, sorted(kernels)
    for name, k in kernels.items():
        assert k["Occupancy"] >= 2 and k["ScratchSize"] == 0, (name, k)
