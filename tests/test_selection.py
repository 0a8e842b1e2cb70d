"""Host-only checks of the rules that choose a kernel (csrc/select.hip), through the selection query and the workspace queries."""
import pytest

from paper_1705_05249_amd import gemm as G

C, N = G.MG_COL_MAJOR, G.MG_NO_TRANS


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
