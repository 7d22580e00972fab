"""Which form a just-in-time cast takes (host arithmetic, no GPU)."""
import pytest

from paper_2505_20524_amd import fog


@pytest.mark.parametrize("cus", [64, 256])
def test_one_launch_between_its_limits_in_elements(cus):
    low, high = (70 << 10) * cus // 16, (625 << 10) * cus // 16
    for chunks, want in ((low - 1, False), (low, True), (high, True), (high + 1, False)):
        assert fog.probe_cast_plan(chunks, 16, False, cus) == want
        assert fog.probe_cast_plan(16, chunks, False, cus) == want
    assert not fog.probe_cast_plan(16 * low + 1, 1, False, cus)


@pytest.mark.parametrize("rows,cols,want", [(4096, 8192, True), (8192, 14336, True), (4096, 4096, False), (16384, 16384, False),
                                            (1250000, 16, False), (16, 1250000, False), (5000000, 16, False), (640000, 64, False),   # an eighth, half filled
                                            (312512, 64, True), (64, 312512, True), (139008, 144, True),                            # ... but all held
                                            (1000000, 80, False), (144, 700000, False), (833344, 96, True), (400000, 272, True),
                                            (700000, 144, True), (176, 400000, True), (80, 500000, False)])
def test_transposing_form_by_tiles(rows, cols, want):
    """A workgroup's time goes by 128 x 128 tiles, filled or not: narrow tensors stay with the kernel that has a workgroup for each."""
    assert fog.probe_cast_plan(rows, cols, True, 256) == want
    assert fog.probe_cast_plan(rows, cols, False, 256) == ((70 << 10) * 256 <= rows * cols <= (625 << 10) * 256)
