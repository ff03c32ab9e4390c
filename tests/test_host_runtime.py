"""Host logic of the runtime without a device: small programs that stand in
for the HIP runtime, linked against the built library."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2504_12858_amd")


def test_step_graphs_against_a_counting_runtime(tmp_path):
    exe = str(tmp_path / "step_graphs")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-rdynamic",
                    "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "host", "step_graphs.cpp"),
                    os.path.join(PKG, "libgrainenv.so"), "-Wl,--allow-shlib-undefined",
                    f"-Wl,-rpath,{PKG}", "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "step graphs clean" in r.stdout, (r.stdout + r.stderr)[-2000:]
