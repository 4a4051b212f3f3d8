"""dsv_plan_upload on the host: what it refuses (no device is needed, nothing is copied)."""
import ctypes

from paper_2607_28848_amd import dsv


def test_plan_upload_refuses_bad_arguments():
    lib = dsv.lib_handle()
    plan = dsv.segments_build([(0, 5, 0, 0), (5, 40, 1, 1)], 45, [8, 16], [1.0, 2.0], 16)
    fake = 1 << 20  # 256-byte aligned, never dereferenced by a refused call
    need = plan.meta_bytes
    assert lib.dsv_plan_upload(None, fake, need, None) == dsv.ERR_ARG
    assert lib.dsv_plan_upload(plan.handle, None, need, None) == dsv.ERR_ARG
    assert lib.dsv_plan_upload(plan.handle, fake + 16, need, None) == dsv.ERR_ARG
    assert lib.dsv_plan_upload(plan.handle, fake, need - 1, None) == dsv.ERR_SIZE
    assert ctypes.c_size_t(need).value >= 45 * 4
