"""The fused chunk's limit on one launch: its work-groups, whole blocks of 8
slices for the 8 XCDs, are counted as they are launched.  Refused on the host,
before anything is enqueued."""
import ctypes

import numpy as np
import pytest

from tests._util import note

pytestmark = pytest.mark.gpu


# 65535 rows x 32768 pairs of angles are 2^31 - 32768, in whole blocks 2^31
@pytest.mark.parametrize("rows,angles", [(65535, 65536), (65535, 65535), (65529, 65536)])
def test_too_many_work_groups_are_refused(rows, angles):
    import torch

    from paper_2209_08450_amd import tp
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    note(f"fbp limit {rows} x {angles}")
    plan = tp.Plan(np.arange(angles) * (np.pi / angles), 2, 1.0)
    buf = torch.zeros(256, dtype=torch.uint8, device="cuda")
    ptr, nul = ctypes.c_void_p(buf.data_ptr()), ctypes.c_void_p()
    ws = tp._fbp_ws(plan.handle, rows, tp.TP_F16)
    st = tp._fbp_chunk_out(plan.handle, ptr, 0, ptr, 1, ptr, 1, 0, rows, tp.TP_RAMP, tp.TP_F16, ptr, ws, tp.TP_F32, ptr,
                           nul, None)
    assert st == tp.TP_EINVAL and "too large for one call" in tp.last_error()
    plan.close()
