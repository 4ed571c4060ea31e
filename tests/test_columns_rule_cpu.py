"""Rules of the broadcasts in columns (csrc/columns_rule.h): what a block of 16 image rows needs of the bias tables, strides that
32-bit offsets cannot reach, and images that fill too little of a block, on both sides of the rule."""
import numpy as np
import pytest

from . import columns_rule


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return columns_rule.load(str(tmp_path_factory.mktemp("rules")))


def test_a_stage_holds_every_cell_row_a_block_touches(rules):
    """The kernel's own arithmetic (bilinear_coord, fp32) over all heights up to 300 and all block heights: a block that is served has room
    for each cell row from its first image row's lower neighbour to its last one's upper."""
    served = set()
    for cells in range(1, 66):
        for gh in range(1, 301):
            parts = rules.large_column_parts(1024, gh, cells)
            assert 0 <= parts <= 6 and (parts == 0 or cells <= 64)
            if parts == 0:
                continue
            served.add(parts)
            y = np.arange(gh, dtype=np.float32)
            s = np.maximum((y + np.float32(0.5)) * (np.float32(cells) / np.float32(gh)) - np.float32(0.5), np.float32(0))
            lo = np.minimum(np.floor(s).astype(int), cells - 1)
            hi = np.minimum(lo + 1, cells - 1)
            first = np.arange(0, gh, 16)
            need = hi[np.minimum(first + 16, gh) - 1] - lo[first] + 1
            assert need.max() <= parts, (cells, gh, need.max(), parts)
    assert served == {1, 2, 3, 4, 5, 6}
    assert rules.large_column_parts(1024, (1 << 31) // 4096, 7) == 0      # offsets in the row component
    assert rules.large_column_parts(1024, (1 << 31) // 4096 - 1, 7) == 3


@pytest.mark.parametrize("gw,stride,columns", [(600, 1 << 22, False), (512, 1 << 22, False), (511, 1 << 22, True), (600, 64, True), (1 << 20, 2048, False),
                                               (1 << 20, 2047, True), (4, 1 << 29, False), (56, 1 << 20, True), (17, 32, False), (22, 32, True)])
def test_output_offsets_of_the_small_kernel_fit_32_bits(rules, gw, stride, columns):
    assert bool(rules.small_columns(gw, stride)) == columns
    if columns:      # the last byte a lane of the last token's row can reach from the row's start
        assert (gw - 1) * stride * 2 + min(stride, 64) * 2 <= 1 << 32


# (units, grid, agents, d, cell rows): measured faster in rows / in columns
ROWS = [(128, (64, 8), 80, 64, 7), (128, (128, 4), 96, 64, 7), (408, (40, 4), 80, 64, 7), (48, (100, 12), 150, 64, 7), (48, (50, 24), 120, 64, 7),
        (96, (33, 20), 110, 64, 7), (88, (36, 20), 90, 64, 7), (128, (36, 80), 80, 64, 7), (192, (17, 8), 91, 64, 5), (256, (57, 4), 123, 32, 7), (384, (127, 4), 76, 128, 7)]
COLUMNS = [(8, (128, 128), 1024, 64, 7), (8, (64, 8), 128, 64, 7), (32, (67, 76), 322, 64, 7), (128, (64, 8), 80, 32, 7),
           (64, (64, 8), 80, 128, 7), (24, (100, 12), 150, 128, 7), (96, (33, 20), 110, 32, 7), (16, (96, 88), 252, 96, 7), (32, (113, 4), 152, 128, 7)]


@pytest.mark.parametrize("units,grid,n,d,cells", ROWS)
def test_narrow_images_stay_in_rows(rules, units, grid, n, d, cells):
    assert columns_rule.large_parts(rules, grid, n, d, units, cells) == 0


@pytest.mark.parametrize("units,grid,n,d,cells", COLUMNS)
def test_images_that_fill_the_blocks_go_in_columns(rules, units, grid, n, d, cells):
    assert columns_rule.large_parts(rules, grid, n, d, units, cells) > 0


# (grid, agents, d, cell rows): the aggregation in rows / in columns
@pytest.mark.parametrize("grid,n,d,cells,columns", [((128, 128), 1024, 64, 7, True), ((128, 128), 256, 64, 7, False), ((70, 48), 257, 32, 7, True),
                                                    ((69, 48), 257, 32, 7, False), ((7, 100), 90, 128, 7, True), ((3, 100), 90, 128, 1, False),
                                                    ((64, 12), 96, 128, 7, True), ((64, 20), 96, 128, 7, False), ((5, 16), 70, 96, 7, False),
                                                    ((40, 18), 96, 128, 4, False)])
def test_aggregation_in_columns(rules, grid, n, d, cells, columns):
    assert columns_rule.aggregate_columns(rules, grid, n, d, cells) == columns


def test_aggregation_offsets_fit_32_bits(rules):
    assert rules.large_aggregate_columns(128, 1 << 16, 64, 512, 7) and not rules.large_aggregate_columns(128, 1 << 16, 64, 512, 16)
    assert not rules.large_aggregate_columns(128, 1 << 20, 512, 16, 7) and rules.large_aggregate_columns(128, 1 << 20, 508, 16, 7)


def test_the_blocks_of_the_projections_are_those_their_tests_name(rules):
    """Every product of the edge cases runs on the blocks that its case says, and between them on every kernel that the rule can choose."""
    from .test_gpu_parity import PROJECTION_CASES
    named = set()
    for name, batch, heads, d, grid, _, _, _, blocks in PROJECTION_CASES:
        C = heads * d
        if blocks:
            assert [columns_rule.projection_blocks(rules, batch * grid[0] * grid[1], O, C) for O in (3 * C, C)] == blocks, name
            named.update(blocks)
    chosen = {columns_rule.projection_blocks(rules, M, O, C) for C in range(8, 1032, 8) for O in (3 * C, C)
              for M in (1, 784, 3136, 9216, 18000, 33496, 42008, 100352, 200704)}
    assert named == chosen and len(chosen) == 11


def test_the_shares_of_fp32_units_are_those_their_test_names(rules):
    """... and between them every number of 16-channel tiles a block can take, of one to four, and one block and several along the tokens."""
    from .test_gpu_fp32_shares import CASES
    assert [columns_rule.fused_f32_shares(rules, grid[0] * grid[1], d, units) for grid, _, d, units, _ in CASES] == [c[4] for c in CASES]
    builds = {((d + 15) // 16, 0 if split == (1, (d + 15) // 16) else split[1]) for _, _, d, _, split in CASES}
    assert builds >= {(dt, ct) for dt in (1, 2, 3, 4) for ct in range(1, dt + 1) if dt % ct == 0}
    assert [columns_rule.fused_f32_shares(rules, 196, 64, units) for units in (1, 64, 128, 256, 1000)] == [(4, 1), (4, 4), (2, 4), (1, 4), (1, 4)]
