import ctypes
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")


def pytest_collection_modifyitems(config, items):
    # A GPU test on a machine without a GPU is an environment error, not a pass:
    # skip it explicitly only when the user deselected nothing and no device exists.
    try:
        import torch
        has_gpu = torch.cuda.is_available()
    except Exception:  # pragma: no cover
        has_gpu = False
    if has_gpu:
        return
    skip = pytest.mark.skip(reason="no GPU in this environment")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)


@pytest.fixture(scope="session")
def host_shim(tmp_path_factory):
    """The library's HIP-free host units behind tests/host_shim.cpp, built with g++."""
    csrc = os.path.join(ROOT, "paper_2605_30519_amd", "csrc")
    so = str(tmp_path_factory.mktemp("shim") / "host_shim.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(ROOT, "tests", "host_shim.cpp"),
                    *(os.path.join(csrc, f) for f in ("validate.cpp", "plan.cpp", "lru_core.cpp", "numa.cpp")), "-o", so],
                   check=True)
    shim = ctypes.CDLL(so)
    shim.shim_key_streams.argtypes = [ctypes.c_int32, ctypes.c_int64, ctypes.c_int32, ctypes.c_int64, ctypes.c_int32]
    return shim


@pytest.fixture(scope="session")
def golden_dir():
    return os.path.join(ROOT, "tests", "golden")
