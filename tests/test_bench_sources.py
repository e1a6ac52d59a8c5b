"""The hash that ties the recorded counters to the device code covers all of it."""
import os

import bench
from paper_1904_02033_amd import build


def test_every_device_source_is_hashed():
    device = {f for f in os.listdir(build.CSRC) if f.endswith((".hip", ".h")) and any(
        k in open(os.path.join(build.CSRC, f)).read() for k in ("__global__", "__device__"))}
    assert device <= set(bench.DEVICE_SOURCES)
    assert set(bench.DEVICE_SOURCES) <= set(os.listdir(build.CSRC))
