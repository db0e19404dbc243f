"""Launch arithmetic (host only): the C++ headers compiled with the host compiler."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2112_14640_amd", "csrc")


def _run(tmp_path, header, body, *args):
    """Compile a program around `body` (int main's statements) with the header, run it, return its output's integers."""
    cxx = shutil.which("g++") or shutil.which("c++")
    assert cxx, "no host C++ compiler"
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(f'#include <cstdio>\n#include <cstdlib>\n#include "{header}"\nint main(int argc, char** argv) {{\n'
                   f"using namespace dirac;\n{body}\nreturn 0;\n}}\n")
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True, timeout=120)
    out = subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True, timeout=120).stdout
    return [[int(x) for x in line.split()] for line in out.splitlines()]


@pytest.mark.parametrize("blocks,threads", [
    (1, 256), (9, 64), (2 ** 24, 256), (2 ** 24 - 8, 256), (67633152, 64), (25165824 // 4 * 4, 192), (34078720 // 16 * 8, 256),
    (2 ** 31, 64), (2 ** 31, 1024), (22369621, 192), (22369622, 192)])
def test_launch_slices_cover_the_work_in_launches_hip_takes(tmp_path, blocks, threads):
    rows = _run(tmp_path, "launch.h",
                'launch_slices(atoll(argv[1]), atoi(argv[2]), [](int64_t first, unsigned n) '
                '{ std::printf("%lld %u\\n", static_cast<long long>(first), n); });', blocks, threads)
    at = 0
    for first, n in rows:
        assert first == at and n % 8 == 0 and n * threads < 2 ** 32
        at += n
    assert blocks <= at < blocks + 8
    assert len(rows) == 1 or (blocks + 7) // 8 * 8 * threads >= 2 ** 32  # one launch wherever one is enough
