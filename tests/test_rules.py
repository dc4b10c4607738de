"""The host runtime's rules (csrc/ph_rules.h) in a program of their own, without a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2411_11547_amd", "csrc")


def run(tmp_path, body):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include <cstdio>\n#include <vector>\n#include "ph_rules.h"\nusing namespace ph;\nint main()\n{\n' + body + "}\n")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")[:-1]


def test_builtin_entry_is_the_tables(tmp_path):
    out = run(tmp_path, """
    TuneEntry t[64];
    const int n = builtin_table(t);
    for (int m = 1; m <= 1023; ++m) {
        int e = 0;
        while (e < n - 1 && t[e].max_m < m) ++e;
        if (e != builtin_entry(m)) printf("%d\\n", m);
    }
    printf("%d\\n", t[n - 1].max_m);
""")
    assert out == ["1023"]


def test_one_pair_launch_holds_its_pairs(tmp_path):
    """Threads of a launch are counted in 32 bits: 2^26 - 1 pairs at most, whatever the
    other way would take (one haplotype of 10^7 bases beside pairs of one base)."""
    out = run(tmp_path, """
    const int64_t far = 10000000;
    const double ends = tile_ns(far, 16, 1);
    for (int64_t pairs : {(int64_t)1 << 25, ((int64_t)1 << 26) - 1, (int64_t)1 << 26, (int64_t)1 << 30}) {
        const double steps = (double)pairs * (1 + kOneSteps);
        printf("%d\\n", (int)within_binned(one_pair_ns(pairs, steps, steps, 1, 1, 0), 55e3, steps * step_ns(1) / 4, ends));
    }
    printf("%d %d\\n", (int)std::isinf(one_pair_ns(2000, 1e6, 1e6, 300, 300, 768)),
           (int)std::isinf(one_pair_ns(2000, 1e6, 1e6, 300, 300, 769)));
""")
    assert out == ["1", "1", "0", "0", "0 1"]


def test_adjoint_lanes(tmp_path):
    """32 or 64 lanes: reads with one row per lane stay in 32, no read takes fewer rows
    than it has, and plans of one configuration take 64 where that measured shorter."""
    out = run(tmp_path, """
    for (int m = 1; m <= 320; ++m)
        for (int wide = 0; wide < 2; ++wide) {
            int P = 0, K = 0;
            const bool ok = adj_config(m, wide, P, K);
            if (ok != (m <= 319) || (ok && (P * K < m + 1 || K > 5 || (m < 32) != (wide ? P == 32 : P == 32 && K == 1))))
                printf("%d %d: %d %d\\n", m, wide, P, K);
        }
    // K of 32 lanes, haplotypes, pairs, 64 lanes
    const int t[][4] = {{1, 40, 160, 0}, {1, 300, 2000, 0}, {2, 300, 800, 1}, {2, 300, 1500, 0}, {4, 1000, 800, 1},
                        {4, 1000, 1500, 1}, {5, 2000, 800, 1}, {5, 2000, 1500, 0}, {5, 600, 2049, 0}, {0, 600, 2048, 1}};
    for (auto &r : t)
        if (adj_wide(r[2], r[0], r[1], r[2] > 1024 ? r[1] : 0) != (r[3] == 1)) printf("%d %d %d\\n", r[0], r[1], r[2]);
    printf("done\\n");
""")
    assert out == ["done"]


def test_adjoint_launch_groups(tmp_path):
    """Tiles of 1,280 steps and twice that again and again; a launch apart for one long
    tile pays with many other tiles, not with few (27,000 and 3,600 pairs of 50-300 x
    1,300-2,000 bases beside one of 100 x 20,000, which leaves 447 workgroups)."""
    out = run(tmp_path, """
    for (int s : {8, 1280, 1288, 2560, 2568, 5120, 5128, 10240, 20480, 20488, 40960, 50000}) printf("%d ", adj_group(s));
    printf("\\n");
    const double far = 20033.0 * adj_step(4), near = 2033.0 * adj_step(5), mean = 0.8 * near;
    for (int tiles : {2900, 21800})
        printf("%d\\n", (int)(adj_launch_time(far, far + tiles * mean, 447) >
                             adj_launch_time(far, far, 1) + adj_launch_time(near, tiles * mean, 1792)));
""")
    assert out == ["0 0 1 1 2 2 3 3 4 5 5 5 ", "0", "1"]
