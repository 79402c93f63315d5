import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def pytest_collection_modifyitems(config, items):
    # GPU tests are skipped, not failed, when collected on a box without a device and not
    # explicitly selected with -m gpu.
    markexpr = config.getoption("-m") or ""
    if "gpu" in markexpr and "not gpu" not in markexpr:
        return
    try:
        import torch
        has_gpu = torch.cuda.is_available()
    except Exception:
        has_gpu = False
    if has_gpu:
        return
    skip = pytest.mark.skip(reason="no GPU in this container")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)


@pytest.fixture(scope="session")
def gemm_unit_asm(tmp_path_factory):
    """gfx950 assembly of every unit that instantiates the grouped GEMM kernel: {unit name: lines}."""
    from paper_2605_19945_amd import build as moe_build
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = tmp_path_factory.mktemp("gemm_units")
    units = [u[:-len(".hip")] for u in moe_build.SOURCES if u.startswith("moe_gemm_")]

    def compile_one(unit):
        path = out / (unit + ".s")
        r = subprocess.run([hipcc, *moe_build.FLAGS, "-S", "--cuda-device-only", "-o", str(path),
                            os.path.join(moe_build.CSRC, unit + ".hip")], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return path.read_text().splitlines()

    with ThreadPoolExecutor(len(units)) as ex:
        return dict(zip(units, ex.map(compile_one, units)))
