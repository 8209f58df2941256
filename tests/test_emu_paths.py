"""Device paths of the library on the CPU emulation build (tests/emu/paths.py),
each case in a child process under AddressSanitizer."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def emu_lib(tmp_path_factory):
    from tests.emu import build_emu
    if not os.path.exists(build_emu.CLANG) or not os.path.exists(build_emu.asan_runtime()):
        pytest.skip("host clang with AddressSanitizer not available")
    lib = str(tmp_path_factory.mktemp("emu") / "libsdgp_emu.so")
    build_emu.build(os.path.join(ROOT, "paper_2205_09070_amd", "csrc"), lib)
    yield lib
    shutil.rmtree(lib + ".src", ignore_errors=True)


@pytest.mark.parametrize("case", ["timing"])
def test_path(emu_lib, case):
    from tests.emu import emu_ctx
    r = subprocess.run([sys.executable, "-u", os.path.join(ROOT, "tests", "emu", "paths.py"), emu_lib, case],
                       env=emu_ctx.emu_env(), capture_output=True, text=True, timeout=600, cwd=ROOT)
    print(r.stdout[-4000:])
    print(r.stderr[-6000:])
    assert r.returncode == 0 and "case %s holds" % case in r.stdout
