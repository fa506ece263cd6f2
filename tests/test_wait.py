"""The host's wait for the report of a running solve leaves the core to other threads."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_polling_gives_up_the_core(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", os.path.join(ROOT, "tests", "wait_check.cpp"), "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout)
    solver = open(os.path.join(ROOT, "paper_1204_2586_amd", "csrc", "hip", "solver.hip")).read()
    loop = solver[solver.index("__atomic_load_n(&cg_report->word"):]
    assert "poll.pause();" in loop[:loop.index("limit = iter + kAhead")]


def test_report_is_coherent_memory():
    """The report is read while kernels write it, which only coherent host memory promises."""
    solver = open(os.path.join(ROOT, "paper_1204_2586_amd", "csrc", "hip", "solver.hip")).read()
    call = solver[solver.index("hipHostMalloc((void **)&cg_report"):]
    assert "hipHostMallocCoherent" in call[:call.index(";")]
