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
