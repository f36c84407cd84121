"""Group formation of the persistent sequential kernel (csrc/seq_groups.h), compiled for the host: on any set of XCDs every sample
belongs to exactly one group that can hold it, and the members of a group are numbered without gaps."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "seq_groups.h"
#define CHECK(c) do { if (!(c)) { std::printf("line %d: mask %d xpg %d B %d rows %d\n", __LINE__, mask, xpg, B, rows); return 1; } } while (0)
int main() {
    for (int mask = 1; mask < 256; ++mask)
        for (int xpg = 1; xpg <= 8; xpg *= 2)
            for (int B = 1; B <= 256; ++B)
                for (int rows = 16; rows <= 32; rows += 16) {
                    int count[8], present = 0;
                    for (int x = 0; x < 8; ++x) { count[x] = (mask >> x) & 1 ? 3 + x : 0; present += count[x] > 0; }
                    std::vector<std::vector<int>> seen(8);
                    std::vector<int> size(8, 0);
                    int groups = 0, per = 0;
                    for (int x = 0; x < 8; ++x)
                        for (int slot = 0; slot < count[x]; ++slot) {
                            const sjd::SeqGroup g = sjd::seq_group_of(count, x, xpg, B, rows);
                            CHECK(g.index >= 0 && g.index < g.groups && g.groups <= present);
                            CHECK(groups == 0 || (groups == g.groups && per == g.per));
                            groups = g.groups; per = g.per;
                            size[g.index] = g.members;
                            seen[g.index].resize(g.members, 0);
                            CHECK(g.before + slot < g.members);
                            ++seen[g.index][g.before + slot];
                        }
                    for (int g = 0; g < groups; ++g)
                        for (int m = 0; m < size[g]; ++m) CHECK(seen[g][m] == 1);
                    CHECK(per * groups >= B);
                    // what fits with a group per XCD fits
                    CHECK(per <= rows || (B + present - 1) / present > rows);
                    // and a choice that fits is kept
                    const int asked = (present + xpg - 1) / xpg;
                    CHECK((B + asked - 1) / asked > rows || groups == asked);
                }
    std::puts("ok");
    return 0;
}
"""


def test_every_sample_has_a_group_on_any_set_of_xcds(tmp_path):
    gxx = shutil.which("g++")
    assert gxx, "g++ is part of the image"
    src = tmp_path / "groups.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "groups")
    subprocess.run([gxx, "-O1", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2505_24791_amd", "csrc"), str(src), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
