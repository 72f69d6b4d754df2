"""The mapping of a launch's blocks to workgroups and XCDs, and the cap of
workgroups per CU by unused LDS (tests/host/xcd_deal.cpp; no GPU)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_every_workgroup_once_and_evenly(tmp_path):
    exe = str(tmp_path / "xcd_deal")
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2305_15116_amd", "csrc"), os.path.join(HERE, "host", "xcd_deal.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout
