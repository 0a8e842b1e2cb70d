"""Which kernel a product with a triangle takes (csrc/select.hip), on the CPU: FP16 ones with a triangular operand and short sums stay on the macro tiles, SYRK off
16 bytes take the checked tiles where those were measured to be faster."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_1705_05249_amd")


@pytest.fixture(scope="module")
def chosen(tmp_path_factory):
    """kernel names of column-major products with a lower triangular op(A), m x m, and a dense op(B), m x n, or, where n is 0, of a triangle of an m x m C with sums of k terms,
    from the built library's own rule and table"""
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
            int f32, at, bt, upper, beta;
            long long m, n, k, pad;
            while (scanf("%d %lld %lld %d %d %lld %d %d %lld", &f32, &m, &n, &at, &bt, &k, &upper, &beta, &pad) == 9) {
                mg::Problem p{};
                p.dtype = f32 ? MG_F32 : MG_F16;
                p.m = p.k = m; p.n = n;
                p.a_trans = at; p.b_trans = bt;
                p.lda = m; p.ldb = bt ? n : m; p.ldc = m;
                p.alpha = 1.f;
                p.shape = mg::MG_SHAPE_A_LOWER;
                if (n == 0) {
                    p.n = m; p.k = k;
                    p.lda = p.ldb = (at ? k : m) + pad; p.ldc = m + pad;
                    p.beta = beta ? 0.5f : 0.f;
                    p.mask_c = true;
                    p.shape = upper ? mg::MG_SHAPE_C_UPPER : mg::MG_SHAPE_C_LOWER;
                }
                int32_t kernel = -1, split = 0;
                mg::select_config(table, p, 256, size_t(1) << 30, &kernel, &split);
                puts(kernel < 0 ? "none" : table[kernel].name);
            }
        }""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(PACKAGE, "csrc"), str(src),
                    os.path.join(PACKAGE, "libmg_gemm.so"), "-Wl,-rpath," + PACKAGE, "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-o", str(exe)],
                   check=True)

    def choose(calls):
        lines = "".join(f"{int(t == 'f32')} {m} {n} {at} {bt} {' '.join(str(int(v)) for v in rest or (0, 0, 0, 0))}\n" for t, m, n, at, bt, *rest in calls)
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


# (n, k, A along k, upper, beta, odd leading dimensions); us there / on the faster tiles
SLOW_256 = [(5409, 103, 1, 0, 1, 1),          # 63.1 / 34.2
            (5584, 267, 1, 1, 1, 1),          # 69.5 / 42.8
            (5435, 100, 0, 0, 0, 0),          # 34.7 / 23.8
            (5295, 19, 0, 1, 0, 1),           # 30.6 / 22.3
            (5551, 587, 0, 0, 1, 1),          # 88.5 / 57.1
            (4345, 463, 0, 0, 1, 0),          # 56.9 / 39.8
            (6959, 474, 1, 0, 1, 0)]          # 98.5 / 73.2
FAST_256 = [(5077, 3771, 1, 0, 0, 0),         # 116 / 181
            (4917, 2341, 0, 1, 0, 0),         # 79 / 117
            (4017, 5436, 1, 1, 0, 0)]         # 119 / 173
SLOW_128 = [(3865, 220, 1, 1, 0, 0),          # 24.1 / 17.7
            (3803, 13, 1, 1, 0, 1),           # 21.0 / 16.1
            (3748, 179, 1, 0, 0, 1)]          # 23.2 / 17.9


def _syrk(calls):
    return [("f16", n, 0, at, 1 - at, k, upper, beta, (1 - n % 2 if odd else 0)) for n, k, at, upper, beta, odd in calls]


def test_syrk_off_16_bytes_on_the_largest_checked_tile(chosen):
    for call, name in zip(SLOW_256, chosen(_syrk(SLOW_256))):
        assert "_256x256x" not in name, (call, name)
    for call, name in zip(FAST_256, chosen(_syrk(FAST_256))):
        assert name.startswith("hmfma_256x256x64"), (call, name)


def test_syrk_off_16_bytes_in_nearly_full_rounds(chosen):
    """two 128 x 128 tiles on each compute unit, 30 x 30 and 31 x 31 of them: some compute units get a third"""
    for call, name in zip(SLOW_128, chosen(_syrk(SLOW_128))):
        assert not name.startswith("hmfma_128x128x64"), (call, name)
