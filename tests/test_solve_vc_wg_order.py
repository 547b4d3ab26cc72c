"""The one-workgroup variable-coefficient solve under every order of its
wavefronts: the kernel's own source, its lanes run as fibers on the CPU
(tests/lanes/), against whole-grid sweeps written out plainly."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_no_order_of_wavefronts_changes_the_solve(tmp_path):
    exe = str(tmp_path / "solve_vc_wg")
    lanes = os.path.join(HERE, "lanes")
    # -ffp-contract=off as in the library: the iterates agree bit for bit
    subprocess.run(["g++", "-std=c++20", "-O1", "-ffp-contract=off", "-mfma", "-D__HIP_PLATFORM_AMD__", "-w", "-I", lanes,
                    "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "paper_2006_16465_amd", "csrc"),
                    os.path.join(lanes, "solve_vc_wg_main.cpp"), "-o", exe], check=True, timeout=300)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert p.returncode == 0 and p.stdout.strip() == "0 failures", p.stdout[-4000:] + p.stderr
