"""Rows of a base block from 33 rows on: 64 in launches of at least 320 blocks of 64 rows whose rows
fill them, else 32 (both sides of the line were timed, see wide64_pays)."""
import pytest

import paper_2604_18655_amd as lib

LAYER = ((2048, 2048), (2048, 512), (2048, 512), (2048, 2048), (2048, 8192), (2048, 8192), (8192, 2048))


@pytest.mark.parametrize("shapes,M,int8_rows,rows", [
    ([(4096, 14336)], 64, False, 32),              # 112 blocks of 64 rows
    ([(4096, 14336)], 512, False, 64),             # 896
    ([(4096, 14336)], 1024, False, 64),            # 1792
    (LAYER, 128, False, 32),                       # 232
    (LAYER, 512, False, 64),                       # 928
    (LAYER * 4, 64, False, 64),                    # 464
    (LAYER * 16, 64, True, 64),                    # 1856, int8 rows
    ([(3072, 9216)] * 2, 72, False, 32),           # 288
    ([(3072, 9216)] * 4, 72, False, 32),           # 576, but 864 blocks of 32 rows do as much
    ([(3072, 9216)] * 4, 128, False, 64),          # 576 and 1152
    (LAYER * 16, 32, False, 32),                   # one chunk of 32 rows
    (LAYER * 16, 16, False, 16),                   # blocks of one column tile
    ([(2048, 2048)], 4, True, 32),                 # int8 rows: always blocks of four tiles
])
def test_rows_of_a_base_block(shapes, M, int8_rows, rows):
    projs = [lib.Proj(K, N, 32, None, None, None, 1.0) for K, N in shapes]
    assert lib.layer_step_block_rows(projs, M, int8_rows) == rows


def test_refused_shapes_have_no_block():
    assert lib.layer_step_block_rows([lib.Proj(100, 64, 32, None, None, None, 1.0)], 64) == 0
    assert lib.layer_step_block_rows([lib.Proj(128, 64, 32, None, None, None, 1.0)], 4097) == 0
