"""What the C ABI asks of the device, with a device of counters in place of
the HIP runtime (no GPU): see tests/host/device_calls_check.cpp."""
import os
import subprocess
import tempfile

import pytest

import paper_1908_07038_amd as pa
from paper_1908_07038_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def checker():
    pa.lib()
    exe = os.path.join(tempfile.mkdtemp(prefix="device_calls_"), "device_calls_check")
    libdir = os.path.dirname(pa.LIB_PATH)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", build.INCLUDE,
                    "-I", os.path.join(build.ROCM, "include"), "-rdynamic", "-o", exe,
                    os.path.join(HERE, "host", "device_calls_check.cpp"), "-L", libdir, "-latlas_nabla",
                    "-Wl,-rpath," + libdir, "-Wl,--allow-shlib-undefined"], check=True)
    return exe


@pytest.mark.parametrize("scenario", ["short_columns_out_of_memory", "short_columns_captured",
                                      "short_columns_beside_a_capture", "short_columns_table_budget",
                                      "plan_out_of_memory", "field_plan_pair", "described_kernels", "tile_orders", "plan_rule"])
def test_device_calls(checker, scenario):
    r = subprocess.run([checker, scenario], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout + r.stderr
