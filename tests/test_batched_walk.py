"""Host-only checks of how the LDS-staged batched kernels walk their work (csrc/batched_walk.h, compiled here as plain C++), at extents
that no test can afford on the device."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1705_05249_amd", "csrc")


def compiled(tmp_path, source):
    """the program's standard output, line by line; signed overflow ends it"""
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=signed-integer-overflow", "-fno-sanitize-recover=all", "-I", CSRC,
                    str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.split("\n")


@pytest.mark.parametrize("chunk", [32, 64])
def test_the_longest_sums_end(tmp_path, chunk):
    """k up to the largest the interface takes: the last chunk holds what is left, and no counter passes the largest int"""
    lines = compiled(tmp_path, """
        #include <climits>
        #include <cstdint>
        #include <cstdio>
        #include <initializer_list>
        #include "batched_walk.h"
        int main()
        {
            for (int k : {0, 1, CHUNK - 1, CHUNK, CHUNK + 1, 5 * CHUNK, INT_MAX - CHUNK, INT_MAX - CHUNK + 1, INT_MAX - 1, INT_MAX}) {
                int64_t chunks = 0, expected = k;
                bool ok = true;
                mg::batchwalk::for_chunks<CHUNK>(k, [&](int left) {
                    ok = ok && left == expected;
                    expected -= CHUNK;
                    ++chunks;
                });
                if (!ok || chunks != (int64_t(k) + CHUNK - 1) / CHUNK) printf("k = %d\\n", k);
            }
        }""".replace("CHUNK", str(chunk)))
    assert lines == [""]


def test_every_tile_has_its_work_group_and_no_xcd_idles(tmp_path):
    """each tile of each instance is taken once, whatever the counts are, and the XCDs (work-group index modulo 8) share them
    evenly: to within one of fewer than 128 instances, to within an instance of more"""
    lines = compiled(tmp_path, """
        #include <cstdio>
        #include <cstdlib>
        #include <initializer_list>
        #include <vector>
        #include "batched_walk.h"
        int main()
        {
            for (int batch : {1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 15, 16, 31, 41, 127, 128, 129, 135, 136, 517})
                for (int tiles : {1, 2, 3, 7, 8, 9, 12, 64, 65}) {
                    std::vector<int> seen(batch * tiles, 0);
                    const int64_t groups = mg::batchwalk::work_groups(batch, tiles);
                    int per_xcd[8] = {0}, wrong = 0;
                    for (int64_t g = 0; g < groups; ++g) {
                        const mg::batchwalk::Place at = mg::batchwalk::place(static_cast<uint32_t>(g), batch, tiles);
                        if (at.inst < 0 || at.inst >= batch || at.tile >= static_cast<uint32_t>(tiles)) continue;      // (an idle one)
                        wrong += ++seen[at.inst * tiles + at.tile] != 1;
                        ++per_xcd[g % 8];
                    }
                    for (int s : seen) wrong += s != 1;
                    int low = per_xcd[0], high = per_xcd[0];
                    for (int c : per_xcd) { low = c < low ? c : low; high = c > high ? c : high; }
                    if (wrong || high - low > (batch < 128 ? 1 : tiles) || (batch < 128 && groups != batch * tiles)) printf("batch %d tiles %d: %d wrong, %d to %d per XCD\\n", batch, tiles, wrong, low, high);
                }
        }""")
    assert lines == [""]
