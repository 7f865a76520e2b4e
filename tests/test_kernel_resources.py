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
        for key in ("ScratchSize", "VGPRs Spill", "LDS Size"):
            hit = re.search(r"\s" + key + r"(?: \[[^\]]*\])?: (\d+)", line)
            if hit and name:
                report[name][key] = int(hit.group(1))
    with open(out) as f:
        return report, f.read()


def test_no_kernel_spills_vector_registers(compiled):
    report, _ = compiled
    assert len(report) > 40
    assert {k: v for k, v in report.items() if v["ScratchSize"] != 0 or v["VGPRs Spill"] != 0} == {}


def test_score_kernels_own_lds_is_what_the_host_counts(compiled):
    report, _ = compiled
    with open(SRC) as f:
        counted = int(re.search(r"#define STATIC_LDS (\d+)", f.read()).group(1))
    sizes = [v["LDS Size"] for k, v in report.items() if "k_score" in k]
    assert len(sizes) >= 16 and max(sizes) <= counted


def test_select_kernels_fit_64_kb(compiled):
    """Own LDS and what the host asks for: beam 32, 1024 list entries; every id a candidate (the last template argument): no keys,
    640 bytes a beam slot, or the longest input's f terms."""
    report, _ = compiled
    sizes = {k: v["LDS Size"] for k, v in report.items() if "k_select" in k}
    dense = [v for k, v in sizes.items() if re.search(r"k_select(_split)?I[^v]*Lb1EEv", k) and not re.search(r"_splitILi\d+ELb1ELb0E", k)]
    lists = [v for k, v in sizes.items() if re.search(r"k_select(_split)?I[^v]*Lb0EEv", k)]
    assert len(dense) == 10 and len(lists) == 12 and len(sizes) == 22
    assert max(dense) + max(20 * 1024 + 640 * 32, 4 * 6176) <= 65536
    assert max(lists) + 36 * 1024 + 32 <= 65536


def test_no_packed_fp32_arithmetic(compiled):
    assert not re.search(r"v_pk_(add|mul|fma)_f32", compiled[1])


def test_no_readlane_right_behind_the_write_of_its_source(compiled):
    """gfx950 wants one instruction between a VALU write of a vector register and a v_readlane of it, in inline assembly
    too, where the compiler does not see to it."""
    before, bad, seen = "", [], 0
    for line in compiled[1].splitlines():
        t = line.split(";")[0].strip()
        if not t or t.startswith(".") or t.endswith(":"):
            continue
        hit = re.match(r"v_readlane_b32\s+\S+,\s*v(\d+)", t)
        if hit:
            seen += 1
            wrote = re.match(r"v_(?!cmp|readlane|readfirstlane)\S+\s+v(?:(\d+)|\[(\d+):(\d+)\])", before)
            if wrote:
                lo = int(wrote.group(1) or wrote.group(2))
                hi = int(wrote.group(1) or wrote.group(3))
                if lo <= int(hit.group(1)) <= hi:
                    bad.append((before, t))
        before = t
    assert seen > 1000 and bad == []
