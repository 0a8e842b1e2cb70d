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
