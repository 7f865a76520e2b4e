"""What the compiler made of the kernels for gfx950: its resource report and its assembly (cross-compiled, no GPU needed)."""
import os
import re
import subprocess

import pytest

import paper_2101_05600_amd as m

SRC = os.path.join(os.path.dirname(os.path.abspath(m.__file__)), "csrc", "ctcbs.hip")


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "ctcbs.s")
    flags = [f for f in m.HIP_FLAGS if f not in ("-shared", "-fPIC")]
    r = subprocess.run(["hipcc", *flags, "--cuda-device-only", "-S", "-Rpass-analysis=kernel-resource-usage", "-o", out, SRC],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    report, name = {}, None
    for line in r.stderr.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].split()[0]
            report[name] = {}
        for key in ("ScratchSize", "VGPRs Spill"):
            hit = re.search(r"\s" + key + r"(?: \[[^\]]*\])?: (\d+)", line)
            if hit and name:
                report[name][key] = int(hit.group(1))
    with open(out) as f:
        return report, f.read()


def test_no_kernel_spills_vector_registers(compiled):
    report, _ = compiled
    assert len(report) > 40
    assert {k: v for k, v in report.items() if v != {"ScratchSize": 0, "VGPRs Spill": 0}} == {}


def test_no_packed_fp32_arithmetic(compiled):
    assert not re.search(r"v_pk_(add|mul|fma)_f32", compiled[1])
