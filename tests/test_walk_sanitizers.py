"""The lane code of the walks and of the whole-ordering evaluation (the headers that
the kernels share) built for the CPU under AddressSanitizer and
UndefinedBehaviorSanitizer, against the C oracle: equal times, no access outside the
queue, no undefined conversion or shift, whichever arm of a selection is taken."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_walks_under_asan_and_ubsan(tmp_path):
    san = ["-fsanitize=address,undefined,float-cast-overflow", "-fno-sanitize-recover=all"]
    obj, exe = str(tmp_path / "oracle.o"), str(tmp_path / "walk")
    subprocess.run(["gcc", "-O2", "-std=c11", "-c", os.path.join(ROOT, "oracle", "tgo_oracle.c"), "-o", obj], check=True)
    src = os.path.join(HERE, "sanitize", "walk.cpp")
    b = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wno-unknown-pragmas", *san,
                        "-I", os.path.join(HERE, "sanitize"), src, obj, "-pthread", "-o", exe],
                       capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe, "90", "7"], capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, UBSAN_OPTIONS="print_stacktrace=1"))
    assert r.returncode == 0 and "walks done, 0 differ" in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]
