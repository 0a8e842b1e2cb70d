"""Which kernel a batched call takes (csrc/select.hip), on the CPU: the kernels that keep whole instances in LDS (csrc/batched_lines.hip) only where
they were measured to gain."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_1705_05249_amd")

# dtype, m, n, k, A along k, B along the columns, instances, strided, beta (column-major); us on the tiles or register blocks / whole in LDS
SLOWER = [("f32", 24, 104, 48, 0, 1, 2855, 0, 1),        # 27 / 39
          ("f32", 32, 16, 40, 0, 1, 2982, 0, 0),         # 8.9 / 12.6
          ("f32", 32, 38, 37, 0, 0, 18592, 0, 0),        # 63 / 86
          ("f32", 30, 5, 48, 0, 0, 15418, 1, 0),         # 27.1 / 36.5
          ("f32", 25, 15, 67, 0, 1, 19791, 1, 0),        # 48 / 64
          ("f32", 7, 152, 6, 0, 0, 76, 0, 1),            # 4.6 / 6.1
          ("f32", 17, 104, 40, 0, 0, 4482, 0, 1),        # 40 / 52
          ("f32", 188, 60, 20, 1, 0, 1092, 0, 0),        # 20.8 / 26.6
          ("f16", 56, 56, 56, 1, 0, 16610, 0, 0),        # 63 / 86
          ("f16", 48, 48, 48, 0, 0, 9500, 0, 1),         # 1.23
          ("f16", 17, 17, 17, 0, 0, 8000, 0, 1)]         # 9.0 / 10.9
FASTER = [("f16", 68, 68, 68, 0, 0, 7141, 0, 1),         # 124 / 55
          ("f16", 36, 36, 36, 0, 1, 19400, 0, 0),        # 63 / 39
          ("f16", 13, 103, 8, 0, 0, 8456, 0, 1),         # 65 / 22
          ("f16", 45, 37, 16, 0, 0, 9600, 0, 1),         # 41 / 21.5
          ("f32", 71, 71, 71, 0, 0, 7608, 1, 1),         # 202 / 145
          ("f32", 22, 122, 9, 0, 0, 10300, 0, 1),        # 72 / 48
          ("f32", 152, 8, 8, 0, 0, 7118, 0, 0),          # 63 / 27
          ("f32", 38, 38, 38, 1, 0, 5415, 0, 1),         # 34.6 / 31.5
          ("f32", 35, 35, 35, 1, 1, 18139, 0, 1),        # 106 / 95
          ("f32", 39, 51, 52, 1, 0, 3199, 1, 1),         # 32.7 / 29.0
          ("f32", 34, 43, 40, 1, 1, 20000, 1, 1),        # 121 / 108
          ("f32", 63, 68, 68, 1, 0, 7331, 0, 1),         # 155 / 119
          ("f32", 54, 66, 67, 1, 0, 8072, 1, 0)]         # 140 / 116


@pytest.fixture(scope="module")
def chosen(tmp_path_factory):
    """kernel names of batched calls, from the built library's own rule and table"""
    from paper_1705_05249_amd import gemm as G
    G.lib()
    folder = tmp_path_factory.mktemp("batched")
    src, exe = folder / "choose.cpp", folder / "choose"
    src.write_text("""
        #include <cstdio>
        #include "select.h"
        int main()
        {
            std::vector<mg::KernelEntry> table;
            mg::register_batched(table);
            mg::register_batched_tile(table);
            mg::register_batched_lines(table);
            int f32, at, bt, strided, old;
            long long m, n, k, batch, pad;
            while (scanf("%d %lld %lld %lld %d %d %lld %d %d %lld", &f32, &m, &n, &k, &at, &bt, &batch, &strided, &old, &pad) == 10) {
                mg::BatchedProblem p{};
                p.dtype = f32 ? MG_F32 : MG_F16;
                p.m = m; p.n = n; p.k = k; p.batch = batch;
                p.a_trans = at; p.b_trans = bt; p.strided = strided;
                p.lda = (at ? k : m) + pad; p.ldb = (bt ? n : k) + pad; p.ldc = m + pad;
                p.alpha = 1.f; p.beta = old ? 0.5f : 0.f;
                p.stride_a = p.lda * (at ? m : k); p.stride_b = p.ldb * (bt ? k : n); p.stride_c = p.ldc * n;
                const int id = mg::select_batched(table, p);
                puts(id < 0 ? "none" : table[id].name);
            }
        }""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(PACKAGE, "csrc"), str(src),
                    os.path.join(PACKAGE, "libmg_gemm.so"), "-Wl,-rpath," + PACKAGE, "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-o", str(exe)],
                   check=True)

    def choose(calls, pad=0):
        lines = "".join(" ".join(str(int(v)) for v in ((c[0] == "f32",) + tuple(c[1:]) + (pad,))) + "\n" for c in calls)
        out = subprocess.run([str(exe)], input=lines, check=True, capture_output=True, text=True, timeout=60).stdout.split()
        assert len(out) == len(calls)
        return out
    return choose


def test_calls_that_whole_instances_slow_down_stay_on_the_other_kernels(chosen):
    for call, name in zip(SLOWER, chosen(SLOWER)):
        assert "lines" not in name, (call, name)


def test_calls_that_whole_instances_speed_up_take_them(chosen):
    for call, name in zip(FASTER, chosen(FASTER)):
        assert "lines" in name, (call, name)


def test_every_call_has_a_kernel(chosen):
    """extents at the edges of blocks, tiles and pieces, few and many instances, both forms"""
    calls = [(t, m, n, k, at, bt, batch, strided, 1) for t in ("f32", "f16") for m in (1, 16, 17, 33, 64, 160, 1100) for n in (1, 16, 32, 65, 300)
             for k in (0, 1, 17, 64, 200, 5000) for at in (0, 1) for bt in (0, 1) for batch, strided in ((1, 0), (300, 1), (30000, 0))]
    assert "none" not in chosen(calls) and "none" not in chosen(calls, pad=1)
