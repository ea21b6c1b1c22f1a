"""CPU check of the lazy bounds of every transform schedule (tests/host_bounds.cpp),
and that it notices a bound that does not hold."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2109_14704_amd", "csrc")


def run(src, exe):
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-o", exe, src])
    return subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_bounds_hold(tmp_path):
    r = run(os.path.join(ROOT, "tests", "host_bounds.cpp"), str(tmp_path / "bounds"))
    assert r.returncode == 0 and r.stdout.startswith("OK"), r.stdout[-2000:]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
@pytest.mark.parametrize("was,now", [
    ("return k - 34u <= 21u;", "return k - 34u <= 24u;"),               # 56 to 58 bits without corrections
    ("return bound > (1 << LBOUT);", "return bound > (4 << LBOUT);"),   # words leave a round too large
    ("return y || (u & 1) || u == R - 1;", "return y || u == R - 1;"),  # X sides of 60 bits grow on
    (": k < 34 ? 4u + v : 3u;", ": k < 34 ? 2u + v : 3u;"),             # an offset below the word it covers
])
def test_a_wrong_bound_is_noticed(tmp_path, was, now):
    os.makedirs(str(tmp_path / "paper_2109_14704_amd" / "csrc"))
    os.makedirs(str(tmp_path / "tests"))
    for f in ("schedule.hpp", "host_tables.hpp", "records.hpp"):
        s = open(os.path.join(CSRC, f)).read()
        if f == "schedule.hpp":
            assert s.count(was) == 1
            s = s.replace(was, now)
        open(str(tmp_path / "paper_2109_14704_amd" / "csrc" / f), "w").write(s)
    src = str(tmp_path / "tests" / "host_bounds.cpp")
    shutil.copy(os.path.join(ROOT, "tests", "host_bounds.cpp"), src)
    r = run(src, str(tmp_path / "bounds"))
    assert r.returncode == 1 and "FAIL" in r.stdout, r.stdout[-2000:]
