"""Table memory of single-precision plans (host dry runs, no GPU)."""
import pytest


# Eight bytes an entry (two layouts of a float) whatever the field count: what
# few-field plans, whose GEMM reads plain floats, take.  T2799 is past the
# 96 GiB at which twelve bytes an entry would stop.
@pytest.mark.parametrize("n,grid,nlat,nl", [(63, "octahedral", 128, 0), (639, "octahedral", 1280, 0),
                                            (2699, "full", 4050, 8100), (2799, "full", 4200, 8400)])
def test_eight_bytes_an_entry(n, grid, nlat, nl):
    import paper_1908_06097_amd as shtx
    rc, few = shtx.plan_check(n, grid, nlat, 8, "fp32", nl)
    assert rc == 0
    for nf in (17, 33, 411):
        rc, info = shtx.plan_check(n, grid, nlat, nf, "fp32", nl)
        assert rc == 0 and info.table_bytes == few.table_bytes
