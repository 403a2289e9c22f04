"""Registers of the FP64 value kernels on transposed tiles, from the build's record."""
import json
import os
import re

import pytest

PATH = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_04477_amd", "_build",
                    "kernel_resources.json")


@pytest.mark.skipif(not os.path.exists(PATH), reason="library not built")
def test_fp64_value_kernels_keep_their_tiles_in_registers():
    """bv_rows_kernel<7 .. 10, false> without tiles in scratch (a tile is 32 bytes per
    lane; G = 10 may keep an address or two there), and the general kernel at none of
    these sizes."""
    res = json.load(open(PATH))
    rows = {int(m.group(1)): r for n, r in res.items() if (m := re.search(r"bv_rows_kernelILi(\d+)ELb0E", n))}
    assert sorted(rows) == [7, 8, 9, 10]
    for g, r in rows.items():
        assert r["scratch"] <= (0 if g < 10 else 16), (g, r)
    general = {int(m.group(1)): r for n, r in res.items() if (m := re.search(r"bv_wave_kernelIdLi(\d+)ELi0ELb0E", n))}
    assert sorted(general) == [1, 2, 3, 4, 5, 6, 11]
    assert all(general[g]["scratch"] == 0 for g in range(1, 7))
