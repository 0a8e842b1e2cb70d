"""What the kernel whose wavefronts share a sum reads (csrc/tiny.hip), on the CPU: no piece of a whole pair of K-steps ends behind the operand, and the checked
pairs behind them cover the rest of the sum."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_whole_pairs_end_inside_the_operand(tmp_path):
    """every piece of every line of the whole pairs, operands along their rows with 1 to 40 rows and few or many elements between the lines"""
    src, exe = tmp_path / "reach.cpp", tmp_path / "reach"
    src.write_text("""
        #include <cstdint>
        #include <cstdio>
        #include "shared_sum.h"
        int main()
        {
            const int piece = 8, pair = 64;
            for (int rows = 1; rows <= 40; ++rows)
                for (int ld = rows; ld <= rows + 9; ++ld)
                    for (int other = 0; other < 8; ++other)               // lines that the other operand of the product keeps back
                        for (int k = 1; k < 400; ++k) {
                            const int own = mg::lines_kept_back(rows, ld, piece), kept = own > other ? own : other;
                            const int whole = mg::whole_pairs(k, kept, pair) * pair;
                            const int64_t end = static_cast<int64_t>(k - 1) * ld + rows;
                            for (int l = 0; l < whole; ++l)
                                for (int row = 0; row < rows; row += piece)
                                    if (static_cast<int64_t>(l) * ld + row + piece > end) {
                                        printf("%d rows, ld %d, k %d: line %d\\n", rows, ld, k, l);
                                        l = whole;
                                        break;
                                    }
                            if (whole < 0 || whole > k || k - whole >= pair + 8) printf("%d rows, ld %d, k %d: %d values left\\n", rows, ld, k, k - whole);
                        }
        }""")
    csrc = os.path.join(ROOT, "paper_1705_05249_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", csrc, str(src), "-o", str(exe)], check=True)
    found = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    assert found == "", found[:500]
