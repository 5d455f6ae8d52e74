"""Builds host_bins_driver.cpp: pm_api.cpp with g++ over launchers that do no work (not collected by
pytest)."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2211_09958_amd", "csrc")
HIP = "/opt/rocm/include"


def no_work(header, done):
    """Definitions with an empty body of the launchers that `done` does not define."""
    out = ["namespace pmx {"]
    for name, args in re.findall(r"^void (launch_\w+)\(([^;{]*)\);", header, re.M):
        if not re.search(rf"^(void|bool) {name}\(", done, re.M):
            args = re.sub(r" = [^,]+", "", args)   # default arguments
            out.append(f"void {name}({args}) {{}}")
    return "\n".join(out + ["}"]) + "\n"


def build(tmp_path):
    """Path of the driver, built in tmp_path."""
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(os.path.join(HIP, "hip", "hip_runtime.h")):
        pytest.skip("g++ or the HIP headers not available")
    driver = os.path.join(HERE, "host_bins_driver.cpp")
    with open(os.path.join(CSRC, "kernels.h")) as h, open(driver) as d:
        header = re.sub(r"//[^\n]*", "", h.read())
        (tmp_path / "no_work.inc").write_text(no_work(header, d.read()))
    exe = str(tmp_path / "host_bins_driver")
    cmd = [gxx, "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{HIP}", f"-I{CSRC}",
           f"-I{os.path.join(ROOT, 'include')}", f"-I{tmp_path}", driver,
           os.path.join(CSRC, "pm_api.cpp"), os.path.join(CSRC, "host_cosmo.cpp"), "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    return exe
