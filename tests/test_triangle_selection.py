"""Which kernel a product with a triangular operand takes (csrc/select.hip), on the CPU: FP16 ones of short sums stay on the macro tiles."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_1705_05249_amd")


@pytest.fixture(scope="module")
def chosen(tmp_path_factory):
    """kernel names of column-major products with a lower triangular op(A), m x m, and a dense op(B), m x n, from the built library's own rule and table"""
    from paper_1705_05249_amd import gemm as G
    G.lib()
    folder = tmp_path_factory.mktemp("triangles")
    src, exe = folder / "choose.cpp", folder / "choose"
    src.write_text("""
        #include <cstdio>
        #include "select.h"
        int main()
        {
            std::vector<mg::KernelEntry> table;
            mg::register_direct(table);
            mg::register_mfma(table);
            mg::register_gemv(table);
            int f32, at, bt;
            long long m, n;
            while (scanf("%d %lld %lld %d %d", &f32, &m, &n, &at, &bt) == 5) {
                mg::Problem p{};
                p.dtype = f32 ? MG_F32 : MG_F16;
                p.m = p.k = m; p.n = n;
                p.a_trans = at; p.b_trans = bt;
                p.lda = m; p.ldb = bt ? n : m; p.ldc = m;
                p.alpha = 1.f;
                p.shape = mg::MG_SHAPE_A_LOWER;
                int32_t kernel = -1, split = 0;
                mg::select_config(table, p, 256, size_t(1) << 30, &kernel, &split);
                puts(kernel < 0 ? "none" : table[kernel].name);
            }
        }""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(PACKAGE, "csrc"), str(src),
                    os.path.join(PACKAGE, "libmg_gemm.so"), "-Wl,-rpath," + PACKAGE, "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-o", str(exe)],
                   check=True)

    def choose(calls):
        lines = "".join(f"{int(t == 'f32')} {m} {n} {at} {bt}\n" for t, m, n, at, bt in calls)
        return subprocess.run([str(exe)], input=lines, check=True, capture_output=True, text=True, timeout=60).stdout.split()
    return choose


def test_short_sums_of_fp16_stay_on_the_tiles(chosen):
    calls = [("f16", m, n, at, bt) for m, n in ((64, 64), (64, 192), (55, 83), (122, 325), (66, 34)) for at in (0, 1) for bt in (0, 1)]
    for call, name in zip(calls, chosen(calls)):
        assert not name.startswith(("htiny", "direct")), (call, name)


def test_longer_ones_thin_ones_and_fp32_share_their_sums(chosen):
    calls = [("f16", 401, 70, 0, 0), ("f16", 401, 70, 1, 1), ("f16", 48, 7, 0, 0), ("f32", 64, 64, 0, 0), ("f32", 55, 83, 1, 0)]
    for call, name in zip(calls, chosen(calls)):
        assert name.startswith(("htiny", "stiny")), (call, name)
