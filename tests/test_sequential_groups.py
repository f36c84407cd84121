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


def test_xcds_of_a_group_where_an_xcd_has_fewer_cus(launch_rules):
    """Width 512: all CUs of an XCD pull a step's weights through its L2 fast enough for a group of its own, half of them do not (64 samples on 128
    CUs: 82.4 us a step with two XCDs a group, 93.7 with one)."""
    on = launch_rules.xcds_per_group_on
    for n in (64, 128, 224):
        assert [on(512, b, n) for b in (1, 4, 5, 64, 65, 256)] == [4, 4, 2, 2, 1, 1]
        assert [on(256, b, n) for b in (1, 256)] == [1, 1]
        assert [on(768, b, n) for b in (4, 5, 32, 64, 65)] == [8, 4, 4, 2, 1]
    for w in (256, 512, 768, 1024):
        for b in range(1, 257):
            assert on(w, b, 256) == launch_rules.xcds_per_group(w, b)
    assert [on(512, b, 256) for b in (4, 5, 64)] == [4, 1, 1]


def test_cached_rows_go_ahead_only_where_members_have_a_second_pair(launch_rules):
    """Requests between the stages cost every member; they pay where the busiest members have more than one pair (width 512, 32 samples of 256
    tokens, one pair each: 64.0 us a step without, 66.8 with; width 1024, 16 samples of 777 tokens: 188, 192)."""
    ahead = launch_rules.rows_ahead
    # width 512, two XCDs a group: 64 members share the pairs of a quarter of the batch
    assert [b for b in range(1, 129) if ahead(b, 8, 512, 256, 256, 2)] == list(range(41, 129))
    assert not ahead(64, 8, 512, 255, 256, 2)
    # the same share of pairs on half of the CUs
    assert [b for b in range(1, 129) if ahead(b, 8, 512, 256, 128, 2)] == list(range(21, 129))
    # wider flows, four XCDs a group: 128 members and half of the batch
    assert [b for b in range(1, 33) if ahead(b, 16, 1024, 513, 256, 4)] == list(range(17, 33))
    assert [b for b in range(1, 33) if ahead(b, 12, 768, 600, 256, 4)] == list(range(21, 33))
    assert not ahead(32, 16, 1024, 512, 256, 4) and not ahead(32, 12, 768, 599, 256, 4)
    # no room beside two row blocks; width 256 has no such kernel
    assert not ahead(129, 16, 1024, 4096, 256, 1) and not ahead(128, 4, 256, 4096, 256, 1)
