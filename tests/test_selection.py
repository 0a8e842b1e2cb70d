"""Host-only checks of the rules that choose a kernel (csrc/select.hip), through the selection query and the workspace queries."""
import os
import subprocess
import sys

import pytest

from paper_1705_05249_amd import gemm as G

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
C, N, T = G.MG_COL_MAJOR, G.MG_NO_TRANS, G.MG_TRANS


def matvec(dtype, outputs, length, ld):
    """(kernel name, slices) of a column-major matrix-vector product with all the workspace it asks for"""
    sel = G.mg_query_selected(dtype, C, N, N, outputs, 1, length, ld, length, outputs)
    need = G.mg_gemv_workspace_bytes(dtype, C, N, outputs, length, ld)
    assert need == (sel["split_k"] * outputs * 4 if sel["split_k"] > 1 else 0)
    return G.mg_kernel_name(sel["kernel_id"]), sel["split_k"]


@pytest.mark.parametrize("dtype,outputs,length,ld", [
    (G.MG_F32, 128, 200000, 1024), (G.MG_F32, 64, 400000, 1024), (G.MG_F32, 192, 140000, 1024), (G.MG_F32, 16, 2000000, 1024),
    (G.MG_F16, 256, 200000, 2048), (G.MG_F16, 128, 400000, 2048), (G.MG_F32, 128, 200000, 1025), (G.MG_F32, 128, 100000, 1024),
    (G.MG_F32, 100, 3000000, 1024)])
def test_few_outputs_and_a_long_sum_are_sliced(dtype, outputs, length, ld):
    """a handful of work-groups would otherwise read the whole matrix"""
    name, slices = matvec(dtype, outputs, length, ld)
    assert 64 <= slices <= 256, (name, slices)


@pytest.mark.parametrize("dtype,outputs,length,ld,panel", [
    (G.MG_F32, 8192, 8192, 8192, True), (G.MG_F32, 8192, 8200, 8192, False), (G.MG_F32, 8192, 6000, 8192, True),
    (G.MG_F32, 4096, 7168, 4096, False), (G.MG_F32, 2048, 16384, 2048, True), (G.MG_F32, 512, 97656, 1024, False),
    (G.MG_F32, 16384, 4096, 16384, False), (G.MG_F32, 8192, 8192, 8193, False), (G.MG_F32, 64, 400000, 1024, True),
    (G.MG_F32, 128, 200000, 1024, False), (G.MG_F32, 192, 260416, 1024, False), (G.MG_F32, 1024, 65536, 1024, False), (G.MG_F16, 256, 390625, 2048, True), (G.MG_F16, 1024, 97656, 2048, False),
    (G.MG_F16, 1500, 66666, 2048, True), (G.MG_F16, 16384, 4608, 16384, False), (G.MG_F32, 12288, 12288, 12288, False)])
def test_streamed_matrices_take_the_panel_kernel_where_it_gains(dtype, outputs, length, ld, panel):
    name, slices = matvec(dtype, outputs, length, ld)
    assert ("panel" in name) == panel and slices > 1, (name, slices)


@pytest.mark.parametrize("dtype,outputs,length,slices", [(G.MG_F32, 3072, 16384, 42), (G.MG_F32, 9000, 9000, 14), (G.MG_F16, 24576, 7680, 10),
                                                         (G.MG_F32, 8200, 8200, 15)])
def test_slices_of_a_streamed_matrix_fill_whole_turns(dtype, outputs, length, slices):
    """two work-groups per compute unit, none left over"""
    name, got = matvec(dtype, outputs, length, outputs)
    assert "axpy" in name and got == slices


@pytest.mark.parametrize("dtype,outputs,length,kernel", [
    (G.MG_F32, 60000, 64, "axpy"), (G.MG_F32, 65532, 16, "axpy"), (G.MG_F32, 60000, 128, "axpy"), (G.MG_F32, 40000, 64, "axpy"), (G.MG_F32, 1000, 4, "axpy"),
    (G.MG_F32, 65535, 5, "axpy"), (G.MG_F16, 60000, 32, "axpy"), (G.MG_F32, 65535, 32, "panel16"), (G.MG_F32, 32768, 64, "panel16"),
    (G.MG_F32, 1000, 64, "panel16"), (G.MG_F16, 60000, 64, "panel16"), (G.MG_F16, 65535, 128, "panel16"), (G.MG_F32, 40000, 512, "panel16"),
    (G.MG_F16, 60000, 512, "panel16"), (G.MG_F16, 65535, 512, "panel8"), (G.MG_F32, 32768, 512, "panel8"), (G.MG_F32, 20000, 256, "panel16"),
    (G.MG_F32, 20000, 700, "panel8"), (G.MG_F32, 1000, 1000, "panel4")])
def test_short_sums(dtype, outputs, length, kernel):
    name, slices = matvec(dtype, outputs, length, outputs)
    assert name.startswith(f"gemv_{kernel}_") and slices == 1, name


@pytest.mark.parametrize("dtype,outputs,length,ld", [
    (G.MG_F32, 1500, 12000, 1501), (G.MG_F32, 1500, 8192, 1500), (G.MG_F16, 3000, 12000, 3000), (G.MG_F16, 5000, 8192, 5000),
    (G.MG_F32, 4096, 4096, 4096), (G.MG_F32, 2048, 4096, 2049), (G.MG_F16, 4096, 4096, 4097), (G.MG_F16, 5000, 4000, 5000),
    (G.MG_F32, 9000, 2560, 9000), (G.MG_F32, 8192, 2560, 8192), (G.MG_F16, 18000, 2560, 18001)])
def test_panels_do_not_outnumber_the_compute_units(dtype, outputs, length, ld):
    """one compute unit with two of the sixteen-wavefront work-groups sets the time"""
    name, slices = matvec(dtype, outputs, length, ld)
    lanes, elems = int(name.split("_")[1][5:]), 4 if dtype == G.MG_F32 else 8
    assert -(-outputs // (lanes * elems)) * slices <= 256, (name, slices)
    assert slices > 1 or lanes == 4 or outputs > 3 * elems * 256, name


def test_tiles_of_a_triangle(tmp_path):
    """the closed form against the tiles counted one by one"""
    src, exe = tmp_path / "count.cpp", tmp_path / "count"
    src.write_text("""
        #include <cstdio>
        #include "tile_count.h"
        int main()
        {
            const int tiles[][2] = {{256, 256}, {256, 128}, {128, 128}, {128, 64}, {64, 64}};
            for (const auto &t : tiles)
                for (int64_t n = 1; n < 3000; n += n < 300 ? 1 : 61) {
                    const int64_t across_m = (n + t[0] - 1) / t[0], across_n = (n + t[1] - 1) / t[1];
                    int64_t lower = 0, upper = 0;
                    for (int64_t i = 0; i < across_m; ++i)
                        for (int64_t j = 0; j < across_n; ++j) {
                            lower += (i + 1) * t[0] > j * t[1];                    // the tile's last row reaches its first column
                            upper += (j + 1) * t[1] > i * t[0];
                        }
                    if (lower != mg::triangle_tiles(true, across_m, across_n, t[0], t[1]) ||
                        upper != mg::triangle_tiles(false, across_m, across_n, t[0], t[1]))
                        printf("%d x %d, n = %lld\\n", t[0], t[1], (long long)n);
                }
        }""")
    csrc = os.path.join(ROOT, "paper_1705_05249_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", csrc, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout == ""


def test_every_tile_of_a_triangle_has_one_work_group(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text("""
        #include <cstdio>
        #include <vector>
        #include "tile_count.h"
        int main()
        {
            for (int tiles = 1; tiles < 1200; tiles += tiles < 100 ? 1 : 97)
                for (int upper = 0; upper < 2; ++upper) {
                    std::vector<int> seen(tiles * tiles);
                    for (int id = 0; id < tiles * (tiles + 1) / 2; ++id) {
                        int tm = -1, tn = -1;
                        mg::triangle_tile(id, tiles, upper != 0, tm, tn);
                        if (tm < 0 || tn < 0 || tm >= tiles || tn >= tiles || (upper ? tn < tm : tn > tm) || seen[tm * tiles + tn]++)
                            printf("%d tiles, id %d: %d %d\\n", tiles, id, tm, tn);
                    }
                }
        }""")
    csrc = os.path.join(ROOT, "paper_1705_05249_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", csrc, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout == ""


def test_tiles_of_the_busiest_shader_engine(tmp_path):
    """against the kernels' walk (tile_coords_balanced) taken work-group by work-group, ids in turn over eight dies and their four engines"""
    src, exe = tmp_path / "engines.cpp", tmp_path / "engines"
    src.write_text("""
        #include <cstdio>
        #include "tile_count.h"
        int main()
        {
            const int tiles[][2] = {{256, 128}, {128, 128}};
            for (const auto &t : tiles)
                for (int upper = 0; upper < 2; ++upper)
                    for (int n = 1; n < 5000; n += 37) {
                        const int across_m = (n + t[0] - 1) / t[0], across_n = (n + t[1] - 1) / t[1];
                        int engine[32] = {0}, most = 0, slices = 1 + n % 3;
                        for (int id = 0; id < slices * across_m * across_n; ++id) {
                            const int wg = id % (across_m * across_n);
                            const int group = wg / (8 * across_n), first = 8 * group, size = across_m - first < 8 ? across_m - first : 8;
                            const int r = wg % (8 * across_n) % size, tn = wg % (8 * across_n) / size;
                            const int tm = first + ((group & 1 ? size - 1 - r : r) + tn + upper) % size;
                            engine[id % 32] += upper ? tm * t[0] < (tn + 1) * t[1] : tn * t[1] < (tm + 1) * t[0];
                        }
                        for (int d : engine) most = d > most ? d : most;
                        if (mg::busiest_engine_tiles(!upper, across_m, across_n, t[0], t[1], slices) != 32 * most)
                            printf("%d x %d, n = %d, upper %d\\n", t[0], t[1], n, upper);
                    }
            printf("%d %d\\n", (int)mg::busiest_engine_tiles(true, 15, 30, 256, 128, 1), (int)mg::busiest_engine_tiles(false, 21, 21, 128, 128, 1));
        }""")
    csrc = os.path.join(ROOT, "paper_1705_05249_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", csrc, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout == "320 288\n"


def test_selection_time_does_not_grow_with_the_matrix():
    """a rank-64 update of 2^20 x 2^20 is ranked in the time that one of 2048 x 2048 takes (no device: the launch fails)"""
    program = """
import sys, time
sys.path.insert(0, sys.argv[1])
import torch
assert torch.cuda.device_count() == 0
from paper_1705_05249_amd import gemm as G
P, call = 0x10000, G.lib().mg_hsyrk
def fastest(n):
    best = 1.0
    for _ in range(40):
        t = time.perf_counter()
        for _ in range(20):
            assert call(G.MG_COL_MAJOR, G.MG_LOWER, G.MG_NO_TRANS, n, 64, 1.0, P, n, 0.0, P, n, P, 1 << 50, None) == -12
        best = min(best, (time.perf_counter() - t) / 20)
    return best * 1e6
print(fastest(2048), fastest(2 ** 20))
"""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1")
    run = subprocess.run([sys.executable, "-c", program, ROOT], capture_output=True, text=True, timeout=300, env=env)
    assert run.returncode == 0, run.stderr
    small, large = map(float, run.stdout.split())
    assert large < 3.0 * small + 20.0, (small, large)                  # microseconds


def test_padded_copies_are_weighed_in_the_time_of_one_selection():
    """a ragged FP16 product that may take padded copies ranks the tiles for two or three paddings and for the direct route: not
    in several times what a product without that choice takes (no device: the launch fails)"""
    program = """
import sys, time
sys.path.insert(0, sys.argv[1])
import torch
assert torch.cuda.device_count() == 0
from paper_1705_05249_amd import gemm as G
P, call = 0x10000, G.lib().mg_hgemm
def fastest(n):
    need = G.mg_gemm_workspace_bytes(G.MG_F16, G.MG_COL_MAJOR, G.MG_NO_TRANS, G.MG_NO_TRANS, n, n, n, n, n, n)
    best = 1.0
    for _ in range(60):
        t = time.perf_counter()
        for _ in range(20):
            assert call(G.MG_COL_MAJOR, G.MG_NO_TRANS, G.MG_NO_TRANS, n, n, n, 1.0, P, n, P, n, 0.5, P, n, P, need, None) == -12
        best = min(best, (time.perf_counter() - t) / 20)
    return best * 1e6
print(fastest(900), fastest(1500), fastest(2050))
"""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1")
    run = subprocess.run([sys.executable, "-c", program, ROOT], capture_output=True, text=True, timeout=300, env=env)
    assert run.returncode == 0, run.stderr
    direct, *weighed = map(float, run.stdout.split())
    assert max(weighed) < 2.0 * direct, (direct, weighed)              # microseconds


def test_static_scratch_takes_what_the_fp32_pipes_take():
    """problems whose sums are sliced on the bf16 pipes alone are not refused for the room of the slices (no device: the launch fails)"""
    program = """
import sys
sys.path.insert(0, sys.argv[1])
import torch
assert torch.cuda.device_count() == 0
from paper_1705_05249_amd import gemm as G
N, T = G.MG_NO_TRANS, G.MG_TRANS
for m, n, k, ta, tb in ((1024, 896, 8448, T, N), (3200, 2752, 3840, T, N), (1443, 3497, 5168, T, N), (5248, 2176, 8640, N, T), (7968, 158, 3184, T, N),
                        (1536, 1024, 32768, N, N)):
    lda, ldb = (m if ta == N else k), (k if tb == N else n)
    print(G.lib().mg_sgemm_static(G.MG_COL_MAJOR, ta, tb, m, n, k, 1.0, 4096, lda, 4096, ldb, 0.0, 4096, m, None))
"""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1")
    run = subprocess.run([sys.executable, "-c", program, ROOT], capture_output=True, text=True, timeout=300, env=env)
    assert run.returncode == 0, run.stderr
    assert run.stdout.split() == ["-12"] * 5 + ["-10"]                 # the last one in eight slices on any pipes: 48 MB


def test_static_scratch_refuses_no_thin_product():
    """fewer than 16 rows or columns: with the slices that fit, however many the query names (no device: the launch fails)"""
    program = """
import sys
sys.path.insert(0, sys.argv[1])
import torch
assert torch.cuda.device_count() == 0
from paper_1705_05249_amd import gemm as G
for m, n, k in ((35500, 15, 4000), (15, 35500, 4000), (61424, 14, 426080), (2, 3000000, 9000)):
    assert m < 100 or G.mg_gemm_workspace_bytes(G.MG_F32, G.MG_COL_MAJOR, G.MG_NO_TRANS, G.MG_NO_TRANS, m, n, k, m, k, m) > G.MG_STATIC_SCRATCH_BYTES
    for layout, ld in ((G.MG_COL_MAJOR, (m, k, m)), (G.MG_ROW_MAJOR, (k, n, n))):
        print(G.lib().mg_sgemm_static(layout, G.MG_NO_TRANS, G.MG_NO_TRANS, m, n, k, 1.0, 4096, ld[0], 4096, ld[1], 0.0, 4096, ld[2], None))
"""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1")
    run = subprocess.run([sys.executable, "-c", program, ROOT], capture_output=True, text=True, timeout=300, env=env)
    assert run.returncode == 0, run.stderr
    assert run.stdout.split() == ["-12"] * 8


def test_the_workspace_query_covers_every_beta():
    """what the query returns holds the slices of the configuration that would be chosen with all the workspace there is"""
    import random
    T, rng = G.MG_TRANS, random.Random(3)
    shapes = [(704, 3072, 2560, N, T), (4544, 1920, 2432, N, N), (256, 1856, 4160, T, N)]
    shapes += [tuple(64 * rng.randint(1, 80) for _ in range(3)) + (rng.choice((N, T)), rng.choice((N, T))) for _ in range(3000)]
    shapes += [tuple(rng.randint(1, 5000) for _ in range(3)) + (rng.choice((N, T)), rng.choice((N, T))) for _ in range(1500)]
    for m, n, k, ta, tb in shapes:
        lda, ldb = (m if ta == N else k), (k if tb == N else n)
        room = G.mg_gemm_workspace_bytes(G.MG_F32, C, ta, tb, m, n, k, lda, ldb, m)
        for beta in (0.0, 1.0):
            slices = G.mg_query_selected(G.MG_F32, C, ta, tb, m, n, k, lda, ldb, m, 1.0, beta)["split_k"]
            assert slices == 1 or 4 * slices * m * n <= room, (m, n, k, ta, tb, beta)


@pytest.mark.parametrize("dtype,n,k,trans", [
    (G.MG_F16, 256, 2048, N), (G.MG_F16, 256, 3000, G.MG_TRANS), (G.MG_F16, 512, 2500, G.MG_TRANS), (G.MG_F16, 200, 2200, G.MG_TRANS),
    (G.MG_F32, 512, 1024, N), (G.MG_F32, 256, 768, G.MG_TRANS), (G.MG_F32, 200, 700, N)])
def test_syrk_query_has_room_for_slices(dtype, n, k, trans):
    """few tiles with a long sum: the product of the same size without a triangle takes a kernel that needs no workspace"""
    dense = -(-n * n * (4 if dtype == G.MG_F32 else 2) // 256) * 256
    for layout in (G.MG_COL_MAJOR, G.MG_ROW_MAJOR):
        assert G.mg_syrk_workspace_bytes(dtype, layout, trans, n, k) >= dense + 2 * 4 * n * n


def wanted_off_16_bytes(m, n, k, ta, tb):
    """(bytes that the query names, bytes of the slices that a tight FP16 call off 16 bytes prefers)"""
    args = (G.MG_F16, C, ta, tb, m, n, k, m if ta == N else k, k if tb == N else n, m)
    slices = [G.mg_query_selected(*args, 1.0, beta, alignment)["split_k"] for alignment in (8, 2) for beta in (0.0, 1.0)]
    return G.mg_gemm_workspace_bytes(*args), max(s * m * n * 4 if s > 1 else 0 for s in slices)


@pytest.mark.parametrize("m,n,k,ta,tb", [(424, 808, 2280, N, N), (1672, 560, 3264, N, T), (448, 608, 2744, T, T), (1000, 1000, 4096, N, N),
                                         (256, 2048, 4096, N, N), (1032, 976, 5896, T, N), (512, 1256, 5216, N, T), (304, 1368, 4160, T, T)])
def test_workspace_query_covers_operands_off_16_bytes(m, n, k, ta, tb):
    """us with the room that aligned operands ask for / with this: (1032, 976, 5896) 82.8 / 48.9, (304, 1368, 4160) 21.0 / 18.0"""
    room, wanted = wanted_off_16_bytes(m, n, k, ta, tb)
    assert room >= wanted > 0


def test_workspace_query_covers_most_operands_off_16_bytes():
    """the others gain less than a microsecond by their estimates"""
    import random
    rng = random.Random(1)
    sizes = [(rng.randrange(8, 188) * 8, rng.randrange(8, 188) * 8, rng.randrange(32, 1000) * 8, rng.choice((N, T)), rng.choice((N, T))) for _ in range(300)]
    assert sum(room < wanted for room, wanted in (wanted_off_16_bytes(*size) for size in sizes)) <= 30


@pytest.mark.parametrize("m,n,k,ta,tb,beta,slow", [
    (704, 128, 64, N, T, 0.5, "htiny"), (64, 128, 64, N, T, 0.0, "htiny"), (2432, 256, 64, N, N, 0.5, "hdma"), (2240, 1856, 64, N, N, 0.5, "hdma"),
    (896, 1024, 128, T, T, 0.0, "hdma16_"), (560, 6952, 64, T, N, 0.5, "hdma"), (232, 168, 16, T, N, 0.5, "hdma16r_128x128"),
    (136, 368, 40, T, T, 0.5, "hdma16r_128x128"), (128, 960, 320, N, T, 0.5, "htiny")])
def test_short_fp16_sums(m, n, k, ta, tb, beta, slow):
    """a few K-tiles of 64: not the kernels that a turn's first load and epilogue make slower there, by 1.14 to 1.34 times"""
    name = G.mg_query_selected(G.MG_F16, C, ta, tb, m, n, k, m if ta == N else k, k if tb == N else n, m, 1.0, beta)["name"]
    assert not name.startswith(slow), name


def test_long_and_few_fp16_sums_keep_their_kernels():
    for m, n, k, ta, tb, name in ((512, 196, 2304, N, N, "htiny"), (128, 128, 512, T, N, "htiny"), (64, 64, 256, T, N, "htiny"), (3000, 3000, 3000, N, N, "hdma16r_192x192"),
                                  (848, 496, 200, N, T, "hdma16r_64x64"), (40, 40, 48, N, N, "htiny")):
        chosen = G.mg_query_selected(G.MG_F16, C, ta, tb, m, n, k, m if ta == N else k, k if tb == N else n, m, 1.0, 0.0)["name"]
        assert chosen.startswith(name), (m, n, k, chosen)


@pytest.mark.parametrize("m,n,k,ta,tb", [(3280, 3600, 2600, T, N), (5416, 5112, 2456, N, N)])
def test_checked_256_tiles_where_192_leave_a_turn_empty(m, n, k, ta, tb):
    """us, 192 x 192 / 256 x 256: 86 / 68 and 159 / 142"""
    assert G.mg_query_selected(G.MG_F16, C, ta, tb, m, n, k, m if ta == N else k, k if tb == N else n, m, 1.0, 0.0)["name"].startswith("hmfma_256x256")


@pytest.mark.parametrize("channels,size,filters", [(164, 9, 40), (151, 8, 59), (150, 7, 51)])
def test_fp32_products_behind_the_unfold_pass_are_sliced(channels, size, filters):
    """few blocks, 1281 to 1536 terms: 14.0 us in slices, 15.8 on the kernel whose wavefronts share the sum; the query names the slices' room"""
    k, n = 9 * channels, size * size
    column = -(-4 * k * n // 256) * 256
    room = G.mg_conv2d_workspace_bytes(G.MG_F32, channels, size, size, (3, 3), (1, 1), (1, 1), (1, 1), filters) - column
    assert room >= 2 * 4 * n * filters
    alone = G.mg_query_selected(G.MG_F32, G.MG_ROW_MAJOR, N, N, filters, n, k, k, n, n)
    assert alone["name"].startswith("stiny")


@pytest.mark.parametrize("m,n,k,ta,tb,name,fringe", [
    (676, 323, 369, N, N, "stiny", 0), (129, 513, 1000, T, N, "stiny", 0), (65, 65, 300, N, T, "stiny", 0),      # 8.7 us, 13.9 with the fringe taken off
    (1025, 129, 1030, N, T, "s", 17), (450, 129, 1928, T, N, "s", 33), (1025, 1025, 600, N, N, "s", 17)])                                          # 15.3 us, 12.9 with it; more blocks than compute units
def test_fringe_of_fp32_products_whose_sum_is_shared(m, n, k, ta, tb, name, fringe):
    chosen = G.mg_query_selected(G.MG_F32, C, ta, tb, m, n, k, m if ta == N else k, k if tb == N else n, m)
    assert chosen["name"].startswith(name) and (chosen["fringe"] == 0) == (fringe == 0), chosen


@pytest.mark.parametrize("m,n,k,ta,tb,shared", [(56, 40, 72, N, T, False), (200, 72, 640, N, T, False), (56, 40, 648, N, T, True), (56, 40, 72, T, T, True), (57, 40, 72, N, T, True)])
def test_fp16_shared_sums_of_operands_along_their_rows(m, n, k, ta, tb, shared):
    """neither operand along k, rows on 16 bytes: up to 640 terms the tiles, 1.06 to 1.12 times as fast"""
    chosen = G.mg_query_selected(G.MG_F16, C, ta, tb, m, n, k, m if ta == N else k, k if tb == N else n, m)["name"]
    assert chosen.startswith("htiny") == shared, chosen


@pytest.mark.parametrize("m,n,k,tb,ldc", [(4391, 1435, 128, N, 4391), (5301, 5840, 40, N, 5301), (3767, 4576, 24, T, 3767), (5799, 1208, 16, N, 5800), (893, 5184, 64, N, 893)])
def test_short_fp16_sums_with_beta_whose_rows_of_c_end_inside_a_piece(m, n, k, tb, ldc):
    """us, 192 x 192 direct-to-LDS tiles / checked 64 x 64: 23.3 / 12.7, 66.6 / 36.8, 42.1 / 26.2, 20.3 / 13.0"""
    args = (G.MG_F16, C, T, tb, m, n, k, k, k if tb == N else n, ldc)
    assert G.mg_query_selected(*args, 1.0, 0.5)["name"].startswith("hmfma_64x64")


@pytest.mark.parametrize("ta,tb,m,n,k,beta", [(N, T, 7337, 2816, 10, 0.5), (N, N, 1137, 2758, 128, 0.7)])
def test_short_sums_off_16_bytes_on_large_grids(ta, tb, m, n, k, beta):
    """the register-staged tiles, several work-groups to a compute unit: (7337, 2816, 10) 28.3 us, 36.0 on the any-element tiles; (1137, 2758, 128) 9.2, 10.7"""
    sel = G.mg_query_selected(G.MG_F16, C, ta, tb, m, n, k, m if ta == N else k, k if tb == N else n, m, 1.0, beta, 2)
    assert G.mg_kernel_name(sel["kernel_id"]).startswith("hmfma_"), G.mg_kernel_name(sel["kernel_id"])


@pytest.mark.parametrize("ta,tb,m,n,k,kernel", [(N, N, 7, 9000, 700, "htiny_32x32"), (T, N, 7, 9000, 700, "htiny_32x32"), (N, N, 4, 30000, 400, "htiny_32x32"),
                                                (T, N, 60393, 7, 401, "hmfma_256x256"), (N, N, 7, 60000, 747, "htiny_32x32")])
def test_fewer_than_eight_rows_or_columns_of_fp16(ta, tb, m, n, k, kernel):
    """the largest tile only for both operands along k in grids that nearly fill the chip"""
    sel = G.mg_query_selected(G.MG_F16, C, ta, tb, m, n, k, m if ta == N else k, k if tb == N else n, m)
    assert G.mg_kernel_name(sel["kernel_id"]).startswith(kernel), G.mg_kernel_name(sel["kernel_id"])
