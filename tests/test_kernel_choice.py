"""The library's choice of kernels and grids on the host (no GPU)."""
import shutil

import pytest

from launch_record import ffn_part, record

OK = 0

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler for the recording runtime")


@pytest.mark.parametrize("device", [{"device": 5, "cus_status": 1}, {"device": 6, "cus": 7}, {"device": 64},
                                    {"device": 7, "device_status": 1}],
                         ids=["no-attribute", "seven-cus", "device-64", "no-device"])
def test_gemm_without_a_cu_count(device, tmp_path):
    """The large GEMMs run, unsplit, where the runtime gives no CU count or one
    below the XCD count: the persistent grid then has some other multiple of 8."""
    known, = record([ffn_part("down", 4, 4096, 8192, 4096, workspace=True, cus=304)], tmp_path)
    assert [g for _, g in known[1]] == [(304, 1, 1)] * 2  # (K long enough to be split: the GEMM and its fixup)
    calls = [ffn_part(p, 4, 4096, 8192, 4096, workspace=ws, **device) for p in ("up", "down") for ws in (False, True)]
    for status, launches in record(calls, tmp_path):
        assert status == OK
        (name, grid), = launches  # one GEMM, no fixup
        assert "grouped_gemm_dma_kernel" in name
        assert grid[0] >= 8 and grid[0] % 8 == 0 and grid[1:] == (1, 1)
