import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")


@pytest.fixture(scope="session")
def native(tmp_path_factory):
    """native(name) builds tests/native/<name>.cpp for the host, with the
    library's own headers and liboc.so; the result runs it with arguments."""
    lib = os.path.join(ROOT, "paper_2607_23844_amd")
    out = tmp_path_factory.mktemp("native")

    def build(name):
        exe = str(out / name)
        if not os.path.exists(exe):
            for cmd in (["/opt/rocm/bin/hipcc", "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-fPIC", "-O1",
                         "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(lib, "csrc"), "-c",
                         os.path.join(ROOT, "tests", "native", name + ".cpp"), "-o", exe + ".o"],
                        ["g++", exe + ".o", "-o", exe, "-L", lib, "-loc", "-L/opt/rocm/lib", "-lamdhip64",
                         f"-Wl,-rpath,{lib}", "-Wl,-rpath,/opt/rocm/lib"]):
                r = subprocess.run(cmd, capture_output=True, text=True)
                assert r.returncode == 0, r.stderr[-2000:]
        return lambda *a: subprocess.run([exe, *map(str, a)], capture_output=True, text=True, timeout=60)

    return build
