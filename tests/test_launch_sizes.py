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


# (n_x, rows, N_c, N_v, bytes of an element, clover) -> the form that was fastest by 10 % or more (0: one thread, in FP64
# one per chirality; 1: one per chirality and colour row; 2: one per colour row; 3: one thread in FP64; -1: the direct
# kernel), timed for every form; the costs of the forms in relation to each other depend on N_c
MEASURED_FORMS = [
    ((8, 1024, 2, 12, 8, 0), 0), ((10, 864, 2, 8, 4, 0), 0), ((13, 3080, 1, 24, 8, 0), 0), ((12, 3456, 1, 16, 4, 0), 0),
    ((10, 864, 4, 12, 4, 0), 0), ((8, 1024, 4, 12, 8, 0), 0), ((22, 7560, 1, 8, 16, 0), 3), ((16, 8192, 1, 12, 16, 1), 3),
    ((8, 1024, 3, 4, 8, 0), 1), ((8, 1024, 3, 4, 8, 1), 0), ((16, 8192, 3, 12, 8, 0), 0), ((16, 8192, 3, 12, 16, 0), 0),
    ((22, 7560, 3, 2, 8, 0), 1), ((13, 3080, 3, 24, 16, 0), -1), ((12, 3456, 2, 1, 16, 0), 1), ((24, 2304, 4, 1, 8, 0), 1)]


def _plans(tmp_path, shapes):
    body = """
    for (int i = 1; i + 5 < argc; i += 6) {
        const RowShape s{atoi(argv[i + 2]), atoi(argv[i + 3]), atoi(argv[i + 4]), atoi(argv[i]), atoll(argv[i + 1]),
                         argv[i + 5][0] == '1'};
        const int units = s.nc * 4 * s.nv * s.storage / 16;
        auto lds = [&](const RowForm&, int d) {
            const int sites = d + (d != s.nx ? 2 : 0);
            return static_cast<std::size_t>(sites) * ((units + units / 4 + 1) * 16 + 3 * s.nc * s.nc * (s.storage == 16 ? 16 : 8));
        };
        const RowPlan p = plan_rows(s, lds);
        const RowForm f = row_form(s.storage == 16, std::max(p.form, 0));
        std::printf("%d %d %d %d %d %lld\\n", p.form, p.seg, p.entries, s.nv * (f.chirality ? 2 : 1) * (f.colour ? s.nc : 1),
                    units, p.form < 0 ? 0LL : static_cast<long long>(lds(f, p.seg)));
    }"""
    return _run(tmp_path, "brillouin_plan.h", body, *[x for s in shapes for x in s])


def test_brillouin_forms_by_colours(tmp_path):
    plans = _plans(tmp_path, [s for s, _ in MEASURED_FORMS])
    assert [(s, p[0]) for (s, _), p in zip(MEASURED_FORMS, plans)] == MEASURED_FORMS


def test_brillouin_plans_fit_the_kernel(tmp_path):
    """What the row kernel assumes of a plan, over every shape class: threads, halo, link window, LDS, clover term."""
    shapes = [(nx, 6 * nx + 1, nc, nv, storage, clover) for nx in (2, 3, 5, 16, 22, 47, 128, 509, 745673) for nc in (1, 2, 3, 4)
              for nv in (1, 2, 5, 12, 24, 65, 129, 256) for storage in (4, 8, 16) for clover in (0, 1)
              if nc * 4 * nv * storage % 16 == 0]
    taken = 0
    for (nx, _, nc, nv, storage, clover), (form, seg, entries, per_site, units, lds) in zip(shapes, _plans(tmp_path, shapes)):
        if form < 0:
            continue
        taken += 1
        sites = seg + (2 if seg < nx else 0)
        assert 1 <= seg <= nx and 32 <= seg * per_site <= 512 and lds <= 64 * 1024
        assert 1 <= entries <= 3 and sites * nc * nc <= entries * seg * per_site
        assert seg == nx or units <= seg * per_site
        assert form in (0, 3) or not clover
        assert form <= (3 if storage == 16 else 1) and (form != 3 or nc <= 2)
    assert taken > len(shapes) // 4
