"""Host-only checks of how the LDS-staged batched kernels walk their work (csrc/batched_walk.h, compiled here as plain C++), at extents
that no test can afford on the device."""
import os
import subprocess
import sys

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


def test_division_by_a_kernel_argument(tmp_path):
    """quotients at and around every multiple that a 31-bit numerator can be next to, for small, large, even and odd divisors"""
    lines = compiled(tmp_path, """
        #include <climits>
        #include <cstdio>
        #include "batched_walk.h"
        int main()
        {
            uint64_t seed = 1;
            for (int i = 0; i < 4000; ++i) {
                seed = seed * 6364136223846793005ull + 1442695040888963407ull;
                const uint32_t d = i < 2000 ? i + 1 : (i < 2060 ? (1u << ((i - 2000) / 2)) - (i & 1) + 1 : static_cast<uint32_t>(seed >> 33) >> (seed % 31));
                if (d == 0 || d > INT_MAX) continue;
                const mg::batchwalk::Divisor by = mg::batchwalk::divisor(d);
                for (int j = 0; j < 500; ++j) {
                    seed = seed * 6364136223846793005ull + 1442695040888963407ull;
                    uint64_t q = j == 0 ? 0 : (j == 1 ? INT_MAX : seed >> 33);
                    if (j % 2) q = q / d * d + (j % 4 == 1 ? d - 1 : 0);
                    if (q > INT_MAX) q = INT_MAX;
                    if (by.quot(static_cast<uint32_t>(q)) != q / d) { printf("%llu / %u\\n", (unsigned long long)q, d); break; }
                }
            }
        }""")
    assert lines == [""]


def test_every_tile_has_its_work_group_and_no_xcd_idles(tmp_path):
    """each tile of each instance is taken once, whatever the counts are, and the XCDs (work-group index modulo 8) share them
    evenly: to within one, or to within an instance where that idles at most a sixth of them"""
    lines = compiled(tmp_path, """
        #include <cstdio>
        #include <cstdlib>
        #include <initializer_list>
        #include <vector>
        #include "batched_walk.h"
        int main()
        {
            for (int batch : {1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 13, 15, 16, 17, 20, 31, 33, 34, 41, 127, 128, 129, 135, 136, 517})
                for (int tiles : {1, 2, 3, 7, 8, 9, 12, 64, 65}) {
                    std::vector<int> seen(batch * tiles, 0);
                    const int64_t groups = mg::batchwalk::work_groups(batch, tiles);
                    int per_xcd[8] = {0}, wrong = 0;
                    for (int64_t g = 0; g < groups; ++g) {
                        const mg::batchwalk::Place at = mg::batchwalk::place(mg::batchwalk::walk(batch, tiles), static_cast<uint32_t>(g));
                        if (at.inst < 0 || at.inst >= batch || at.tile >= static_cast<uint32_t>(tiles)) continue;      // (an idle one)
                        wrong += ++seen[at.inst * tiles + at.tile] != 1;
                        ++per_xcd[g % 8];
                    }
                    for (int s : seen) wrong += s != 1;
                    int low = per_xcd[0], high = per_xcd[0];
                    for (int c : per_xcd) { low = c < low ? c : low; high = c > high ? c : high; }
                    if (wrong || (high - low > 1 && (high - low > tiles || 5 * batch < 4 * ((batch + 7) / 8 * 8) || 6 * (groups - batch * tiles) > groups))) printf("batch %d tiles %d: %d wrong, %d to %d per XCD\\n", batch, tiles, wrong, low, high);
                }
        }""")
    assert lines == [""]


def test_the_pieces_of_a_call_cover_it(tmp_path):
    """any accepted number of instances and any size of one: launches of fewer than 2^32 threads that take each tile once"""
    lines = compiled(tmp_path, """
        #include <cstdio>
        #include <initializer_list>
        #include "batched_walk.h"
        using namespace mg::batchwalk;
        int main()
        {
            const int64_t most = (int64_t(1) << 31) - 1;
            for (int64_t per_group : {0, 4})
                for (int64_t batch : {int64_t(1), int64_t(7), int64_t(1000), (int64_t(1) << 24) - 8, int64_t(1) << 24, int64_t(1) << 25, most})
                    for (int64_t tiles : {int64_t(1), int64_t(3), int64_t(2100000), MOST_GROUPS, MOST_GROUPS + 1, int64_t(1) << 26}) {
                        if (per_group > 0 && tiles > 1) continue;
                        if (tiles > 3 && batch > 1000) continue;                   // (beyond any memory)
                        int64_t at_inst = 0, at_tile = 0;
                        bool ok = true;
                        for_pieces(batch, tiles, per_group, [&](int64_t i, int64_t count, int64_t t, int64_t n) {
                            const int64_t groups = per_group > 0 ? (count + per_group - 1) / per_group : work_groups(count, n);
                            ok = ok && i == at_inst && t == at_tile && count > 0 && n > 0 && groups <= MOST_GROUPS && groups * 256 < (int64_t(1) << 32);
                            ok = ok && (n == tiles || count == 1);
                            at_tile += n;
                            if (at_tile == tiles) { at_tile = 0; at_inst += count; }
                            return true;
                        });
                        if (!ok || at_inst != batch || at_tile != 0) printf("batch %lld tiles %lld\\n", (long long)batch, (long long)tiles);
                    }
        }""")
    assert lines == [""]


def test_no_number_of_instances_is_refused():
    """more instances than one launch has work-groups for, and one instance of more tiles: there is a kernel for each (without a
    device the launch fails; a call that no kernel takes fails before it)"""
    program = """
import sys
sys.path.insert(0, sys.argv[1])
import torch
assert torch.cuda.device_count() == 0
from paper_1705_05249_amd import gemm as G
C, N, P = G.MG_COL_MAJOR, G.MG_NO_TRANS, 0x1000
for call in (G.mg_sgemm_strided_batched, G.mg_hgemm_strided_batched):
    for m, n, k, batch in ((40, 1, 1, 17000000), (33, 4, 4, 20000000), (40, 1, 8, 2 ** 24 - 8), (40, 1, 8, 2 ** 24), (1, 40, 8, 2 ** 25),
                           (8, 8, 40, 2 ** 25), (131072, 131072, 8, 1), (131072, 131072, 8, 3)):
        print(m, n, k, batch, call(C, N, N, m, n, k, 1.0, P, m, m * k, P, k, k * n, 0.0, P, m, m * n, batch, stream=0, check=False))
"""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1")
    run = subprocess.run([sys.executable, "-c", program, ROOT], capture_output=True, text=True, timeout=300, env=env)
    assert run.returncode == 0, run.stderr
    lines = run.stdout.split("\n")[:-1]
    assert len(lines) == 16 and all(line.endswith(" -12") for line in lines), run.stdout
