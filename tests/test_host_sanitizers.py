"""The host code under AddressSanitizer and UndefinedBehaviorSanitizer: the ABI
tests (argument checks, work lists, overlap checks, error paths, all before any
device call) run in a child process against a build of libgnmr whose host code is
instrumented and aborts on any report, and the tests of the per-step calls'
marshalling against such a build of its module.  CPU only."""
import glob
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def test_abi_tests_are_clean_under_host_sanitizers(tmp_path):
    from paper_2606_00539_amd import _build

    runtime = _build.sanitizer_runtime()
    if runtime is None:
        pytest.skip("no clang AddressSanitizer runtime in this toolchain")
    lib = _build.build_host_sanitized(str(tmp_path / "libgnmr_hostsan.so"))
    log = tmp_path / "san"
    env = dict(os.environ, GNMR_LIBRARY=lib, LD_PRELOAD=runtime,
               ASAN_OPTIONS=f"detect_leaks=0:alloc_dealloc_mismatch=0:log_path={log}",
               UBSAN_OPTIONS=f"print_stacktrace=1:log_path={log}")
    r = subprocess.run([sys.executable, "-m", "pytest", "-q", "-p", "no:cacheprovider",
                        "-m", "not gpu", os.path.join(ROOT, "tests", "test_abi.py")],
                       cwd=ROOT, env=env, capture_output=True, text=True, timeout=600)
    reports = sorted(glob.glob(str(log) + "*"))
    text = "".join(open(f).read()[:4000] for f in reports)
    assert not reports, f"sanitizer reports:\n{text}"
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    assert " passed" in r.stdout


def test_marshalling_tests_are_clean_under_sanitizers(tmp_path):
    from paper_2606_00539_amd import _build

    r = subprocess.run(["gcc", "-print-file-name=libasan.so"], capture_output=True, text=True)
    if r.returncode != 0 or not os.path.isabs(r.stdout.strip()):
        pytest.skip("no gcc AddressSanitizer runtime")
    copy = shutil.copytree(_build.PKG, tmp_path / "paper_2606_00539_amd",
                           ignore=shutil.ignore_patterns("__pycache__", "csrc", "_calls*"))
    calls = str(copy / os.path.basename(_build.CALLS))
    subprocess.run(_build.calls_command(calls, "-g", "-fsanitize=address", "-fsanitize=undefined",
                                        "-fno-sanitize-recover=undefined"), check=True)
    (tmp_path / "tests").mkdir()
    for f in ("conftest.py", "test_native_calls.py"):
        shutil.copy(os.path.join(ROOT, "tests", f), tmp_path / "tests")
    log = tmp_path / "san"
    env = {k: v for k, v in os.environ.items() if k not in ("PYTHONPATH", "GNMR_LIBRARY")}
    env.update(LD_PRELOAD=r.stdout.strip(), PYTHONPATH=str(tmp_path),
               ASAN_OPTIONS=f"detect_leaks=0:alloc_dealloc_mismatch=0:log_path={log}",
               UBSAN_OPTIONS=f"print_stacktrace=1:log_path={log}")
    r = subprocess.run([sys.executable, "-m", "pytest", "-q", "-p", "no:cacheprovider",
                        str(tmp_path / "tests" / "test_native_calls.py")], cwd=tmp_path, env=env,
                       capture_output=True, text=True, timeout=600)
    text = "".join(open(f).read()[:4000] for f in sorted(glob.glob(str(log) + "*")))
    assert not text, f"sanitizer reports:\n{text}"
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    assert " passed" in r.stdout
