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


RING, REG = "skinny_dma_kernel", "skinny_reg_kernel"
SKINNY = [
    # (GEMM, segments, rows, d, d_ff, kernel): both sides of every line of the
    # rule, at sizes where the kernels were timed
    ("up", 15, 4, 2048, 1408, REG), ("up", 15, 8, 2048, 1408, REG), ("up", 60, 8, 2048, 1408, RING),
    ("up", 64, 6, 2048, 1408, RING), ("up", 8, 6, 4096, 1792, REG), ("up", 8, 12, 4096, 1792, RING),
    ("up", 60, 48, 2048, 352, REG), ("up", 60, 128, 2048, 352, RING), ("up", 15, 240, 2048, 176, REG),
    ("up", 15, 80, 2048, 352, REG), ("up", 15, 120, 2048, 352, RING),
    ("up", 15, 40, 2048, 1408, RING), ("up", 15, 48, 2048, 1408, REG), ("up", 15, 96, 2048, 1408, REG), ("up", 15, 160, 2048, 1408, RING),
    ("up", 8, 16, 4096, 3584, REG), ("up", 8, 48, 4096, 3584, REG), ("up", 8, 96, 4096, 3584, RING),
    ("up", 1, 16, 2048, 2816, REG), ("down", 1, 16, 2048, 2816, REG), ("down", 2, 32, 2048, 2816, REG),
    ("down", 15, 4, 2048, 1408, REG), ("down", 60, 96, 2048, 1408, REG), ("down", 60, 128, 2048, 1408, RING),
    ("down", 15, 96, 2048, 1408, REG), ("down", 15, 112, 2048, 1408, RING),
    ("down", 4, 12, 4096, 14336, REG), ("down", 8, 2, 4096, 14336, REG), ("down", 8, 4, 4096, 14336, RING),
    ("down", 8, 6, 4096, 3584, RING), ("down", 8, 16, 4096, 14336, REG),
    ("down", 8, 48, 4096, 14336, RING), ("down", 8, 64, 4096, 3584, RING), ("down", 8, 96, 4096, 1792, RING),
    ("down", 15, 240, 2048, 176, REG), ("down", 15, 241, 2048, 176, "skinny_gemm_kernel"),
]


def test_skinny_gemm_choice(tmp_path):
    """Decode-sized GEMMs: the 16-column kernel only where it is the faster one."""
    calls = [ffn_part(p, n, rows, d, f) for p, n, rows, d, f, _ in SKINNY]
    for case, (status, launches) in zip(SKINNY, record(calls, tmp_path)):
        assert status == OK
        (name, _), = launches
        assert case[-1] in name, (case, name)


def test_skinny_gemm_choice_follows_the_cu_count(tmp_path):
    """On half of the chip (128 CUs) the ring kernel is full twice as early."""
    calls = [ffn_part("up", 15, 4, 2048, f, cus=cus, device=1 + i)
             for i, (f, cus) in enumerate(((1408, 256), (1408, 128), (352, 128)))]
    assert [[k for k in (RING, REG) if k in launches[0][0]] for _, launches in record(calls, tmp_path)] == [[REG], [RING], [REG]]


TILES = [
    # (GEMM, segments, rows, d, d_ff, kernel): ragged K, where the register-staged
    # 128-row tiles are one round of workgroups at most, and past it
    ("down", 15, 1200, 2048, 176, "grouped_gemm_kernel<false, 128"), ("down", 15, 2000, 2048, 176, "grouped_gemm_kernel<false, 128"),
    ("down", 15, 2800, 2048, 176, "dma_kernel<false, true"), ("down", 15, 1200, 2048, 352, "dma_kernel<false, true"),
    ("down", 15, 1600, 2048, 352, "grouped_gemm_kernel<false, 128"), ("down", 15, 2000, 2048, 488, "dma_kernel<false, true"),
    ("down", 4, 1000, 2048, 616, "grouped_gemm_kernel<false, 128"), ("down", 4, 1000, 2048, 744, "dma_kernel<false, true"),
    ("down", 4, 1000, 2048, 192, "dma_kernel<false, true"),
    ("up", 4, 1000, 136, 1024, "grouped_gemm_kernel<true, 128"), ("up", 4, 1000, 392, 1024, "grouped_gemm_kernel<true, 128"),
    ("up", 4, 1000, 520, 1024, "dma_kernel<true, true"), ("up", 15, 1050, 200, 1024, "dma_kernel<true, true"),
    ("up", 15, 1950, 392, 1024, "dma_kernel<true, true"),
    # the half tiles' line in rows per segment, K whole
    ("up", 15, 15 * 768 - 1, 2048, 1408, "dma_kernel<true, true"), ("up", 15, 15 * 768, 2048, 1408, "dma_kernel<true, false"),
    # K too short for the copies; 256-row tiles where they are enough fewer rounds
    ("up", 4, 8000, 72, 4096, "grouped_gemm_kernel<true, 256"), ("up", 4, 5000, 72, 1024, "grouped_gemm_kernel<true, 256"),
    ("up", 4, 8000, 120, 120, "grouped_gemm_kernel<true, 128"),
    ("up", 8, 8184, 72, 4096, "grouped_gemm_kernel<true, 128"), ("up", 4, 8000, 136, 4096, "dma_kernel<true, true"),
    ("down", 4, 5000, 1024, 72, "grouped_gemm_kernel<false, 128"), ("down", 4, 8000, 1024, 72, "grouped_gemm_kernel<false, 256"),
    ("down", 4, 20000, 1024, 72, "grouped_gemm_kernel<false, 128"),
    ("up", 4, 1000, 72, 1024, "grouped_gemm_kernel<true, 128"), ("down", 4, 1000, 1024, 120, "grouped_gemm_kernel<false, 128"),
]


def test_large_gemm_choice(tmp_path):
    """Larger GEMMs: register-staged tiles where they are faster (or the only ones), else the persistent kernel."""
    calls = [ffn_part(p, n, rows, d, f) for p, n, rows, d, f, _ in TILES]
    for case, (status, launches) in zip(TILES, record(calls, tmp_path)):
        assert status == OK
        (name, _), = launches
        assert case[-1] in name, (case, name)
