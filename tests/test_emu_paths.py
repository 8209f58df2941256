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


@pytest.mark.parametrize("case", ["timing", "cap", "cap_lists", "refused_trial", "csr_grid", "sides", "canonical", "block_members", "few_rows", "tile_flags"])
def test_path(emu_lib, case, tmp_path):
    from tests.emu import emu_ctx
    r = subprocess.run([sys.executable, "-u", os.path.join(ROOT, "tests", "emu", "paths.py"), emu_lib, case],
                       env=emu_ctx.emu_env({"SDGP_TUNE_CACHE": str(tmp_path / "tune.json")}), capture_output=True,
                       text=True, timeout=600, cwd=ROOT)
    print(r.stdout[-4000:])
    print(r.stderr[-6000:])
    assert r.returncode == 0 and "case %s holds" % case in r.stdout


@pytest.mark.parametrize("order", ["up", "down"])
def test_sums_do_not_depend_on_block_order(emu_lib, order, tmp_path):
    """k_cg_colsum's blocks run in any order: the one that ends the iteration
    may come first, and every sum of the launch is written all the same."""
    from tests.emu import build_emu
    src = emu_lib + ".src"
    emu = os.path.join(ROOT, "tests", "emu")
    exe = str(tmp_path / "colsum")
    objs = sorted(os.path.join(src, f) for f in os.listdir(src) if f.endswith(".o") and f != "cg.cpp.o")
    r = subprocess.run([build_emu.CLANG, "-std=c++17", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer",
                        "-Wno-everything", "-I", os.path.join(emu, "include"), "-I", emu, "-I", src, "-I",
                        os.path.join(ROOT, "include"), os.path.join(emu, "colsum.cpp")] + objs
                       + ["-lpthread", "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    env = dict(os.environ, EMU_ORDER=order, EMU_THREADS="1", ASAN_OPTIONS="detect_leaks=0")
    r = subprocess.run([exe], env=env, capture_output=True, text=True, timeout=300)
    print(r.stdout[-2000:])
    print(r.stderr[-4000:])
    assert r.returncode == 0
