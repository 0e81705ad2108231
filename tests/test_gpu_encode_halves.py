"""hbfp_encode_packed by halves of 96 rows (few 192 x 192 regions) and by whole regions (more than 400): edges of halves, regions,
k-steps and panels, both rounding modes, vectors and tiles, bit for bit against hbfp_encode and hbfp_pack one by one."""
import numpy as np
import pytest
import torch

from tests.test_gpu_encode_packed import _check_against_separate_calls, _rand

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rounding", [0, 1])
@pytest.mark.parametrize("rows,cols", [(1, 4), (95, 96), (96, 192), (97, 196), (191, 188), (193, 100), (289, 388), (769, 772), (4000, 4004)])
@pytest.mark.parametrize("blocks", [((1, 24), (24, 1)), ((24, 24), (24, 24)), ((24, 24), (24, 1))])
def test_halves_and_regions(rows, cols, blocks, rounding):
    from paper_1804_01526_amd import hbfp
    print(f"[halves] {rows}x{cols} {blocks} rounding={rounding}", flush=True)
    x = _rand((rows, cols), rows + cols)
    _check_against_separate_calls(hbfp, x, [(*blocks[0], 8, rounding, 3, 1), (*blocks[1], 8, rounding, 9, 0)])
