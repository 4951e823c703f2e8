"""What the library does with device memory, on the host: a driver that
defines the HIP calls itself (tests/host_memory_driver.c) runs it on a device
whose memory is a number of bytes.  Networks and contexts are made where they
fit once idle scratch memory is given back, and the images that share launches
come with the first call over symmetries."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_device_memory_on_a_device_of_bytes(tmp_path):
    if shutil.which("gcc") is None:
        pytest.skip("gcc is not available")
    from paper_1711_03244_amd import build
    lib = build.LIB if os.path.exists(build.LIB) else build.build()
    exe = tmp_path / "host_memory_driver"
    b = subprocess.run(["gcc", "-std=gnu99", "-O1", "-w", "-rdynamic", "-o", str(exe),
                        os.path.join(HERE, "host_memory_driver.c"), lib,
                        f"-Wl,-rpath,{os.path.dirname(lib)}", "-Wl,--allow-shlib-undefined"],
                       capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
