"""The library's host side on several devices, played by a HIP runtime of the driver's own (tests/launch_driver.c): dynamic LDS is
granted to a kernel on every device it is launched on, and a refusal is reported and not kept."""
import os
import subprocess

from conftest import ROOT


def test_dynamic_lds_is_granted_per_device(tmp_path):
    from paper_2506_03206_amd import build, rdk
    if not os.path.exists(rdk.LIB_PATH):
        build.build()
    exe = str(tmp_path / "launch_driver")
    made = subprocess.run(["gcc", "-std=c99", "-Wall", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                           os.path.join(ROOT, "tests", "launch_driver.c"), rdk.LIB_PATH, "-Wl,-rpath," + os.path.dirname(rdk.LIB_PATH),
                           "-Wl,--allow-shlib-undefined", "-o", exe], capture_output=True, text=True)
    assert made.returncode == 0, made.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
