"""bench.py's command line, as far as it can be checked without a GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 2
    assert "ONE GPU" in r.stderr and r.stdout.strip() == ""


def test_product_path_does_not_import_the_oracle():
    """The package and bench.py's timed path never pull in oracle/ (only bench's cpu_baseline leg and
    the tests do): importing the package must not import it, and the package has no fallback."""
    code = "import sys; import paper_2101_05600_amd as m; print(any(k == 'oracle' or k.startswith('oracle.') for k in sys.modules))"
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120, cwd=ROOT)
    assert r.returncode == 0 and r.stdout.strip() == "False"
    src = open(os.path.join(ROOT, "paper_2101_05600_amd", "__init__.py")).read()
    assert "import oracle" not in src and "from oracle" not in src


def test_committed_counter_summaries_are_readable_by_the_bench_line():
    """The roofline object's profiler-side figures come from the committed summaries under profiles/:
    each must parse and carry traffic, the kernel's own duration and when it was measured."""
    sys.path.insert(0, ROOT)
    import bench
    for wl in ("cfg2", "cfg4b"):
        traffic, us, when = bench.read_profile_summary(os.path.join(ROOT, "profiles", f"k_score_{wl}_traffic.txt"))
        assert traffic and traffic > 1e6 and us and 1.0 < us < 1000.0 and when and "MI355X" in when
    assert bench.read_profile_summary(os.path.join(ROOT, "profiles", "no_such_file.txt")) == (None, None, None)


def test_profiles_are_told_from_those_of_other_sources():
    """The bench line says whether the profiler's figures it quotes are of the present sources: by a hash that comments and
    blanks do not change."""
    sys.path.insert(0, ROOT)
    import bench
    import re
    for wl in ("cfg2", "cfg4b"):
        assert re.fullmatch("[0-9a-f]{12}", bench.profile_hash(os.path.join(ROOT, "profiles", f"k_score_{wl}_traffic.txt")))
    assert re.fullmatch("[0-9a-f]{12}", bench.source_hash())
    assert bench.profile_hash(os.path.join(ROOT, "profiles", "no_such_file.txt")) is None


def test_rate_of_the_matrix_form_is_that_of_the_bytes_it_reads():
    """Every id a candidate: frames without a share are skipped, so the rate comes from the counters' bytes; without them there is none."""
    sys.path.insert(0, ROOT)
    import bench
    traffic, us, _ = bench.read_profile_summary(os.path.join(ROOT, "profiles", "k_dense_cfg4a_u32_traffic.txt"))
    r = bench.dense_roofline(1e-3 * us * 10, 10, 4e11, 20, traffic)
    assert abs(r["achieved"] - traffic / us * 1e-3) < 1e-6 * r["achieved"] and 0.0 < r["frac"] < 0.8
    assert r["bytes_of_all_frames_per_launch"] == 4e11 * 4 / 20 / 10 and "frac_of_fp32_matrix_peak" not in r
    r = bench.dense_roofline(1.0, 10, 4e11, 20, None)
    assert r["achieved"] is None and r["frac"] is None
