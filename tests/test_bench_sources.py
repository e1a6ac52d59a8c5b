"""The hash that ties the recorded counters to the device code covers all of it."""
import os
import re

import bench
from paper_1904_02033_amd import build


def test_every_device_source_is_hashed():
    # functions of the device (sanns_api.hip holds a variable of it)
    code = re.compile(r"__global__|__device__ (?!__align__)[^;{]*\(")
    device = {f for f in os.listdir(build.CSRC) if f.endswith((".hip", ".h"))
              and code.search(open(os.path.join(build.CSRC, f)).read())}
    assert {"kernels.hip", "mfma.hip", "kmeans.hip"} <= device <= set(bench.DEVICE_SOURCES)
    assert set(bench.DEVICE_SOURCES) <= set(os.listdir(build.CSRC))
