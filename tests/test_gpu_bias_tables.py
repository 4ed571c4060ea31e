"""The half-resized bias tables (agent_attn_bias_tables for more than 64 agents) against the components' own formula, at the sizes
where their kernel branches: columns and image rows that end inside a block of 64 or of 16, narrow images whose waves take several
agents side by side, agents past the last whole 64 and off the 16-byte pieces, parameters off 16 bytes, block grids that wait in
LDS, whose cell rows come one a block, and that are too wide for LDS, components that are absent.

The layout (NA: agents rounded up to 64; entries times log2 e; he: cell rows, 1 without a block component; an absent row component has
no table), each table on a multiple of 256 bytes:
  B1  half[((i w / 4 + x / 4) NA + a) 4 + x % 4], rows[y NA + a]         per head
  B2  half[((i NA / 4 + a / 4) w + x) 4 + a % 4], rows[((a / 4) h + y) 4 + a % 4]
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
KEYS = ("b1_col", "b1_row", "b1_blk", "b2_col", "b2_row", "b2_blk")


@pytest.fixture(scope="module")
def aa():
    from paper_2312_08874_amd import binding
    binding.lib()
    return binding


def _shapes(H, n, grid, blk):
    h, w = grid
    return dict(b1_col=(H, n, w), b1_row=(H, n, h), b1_blk=(H, n) + blk, b2_col=(H, w, n), b2_row=(H, h, n), b2_blk=(H,) + blk + (n,))


def _along_x(blk, w):
    """[..., w0] -> [..., w], bilinear with half-pixel centres."""
    w0 = blk.shape[-1]
    s = np.maximum((np.arange(w) + 0.5) * w0 / w - 0.5, 0.0)
    i0 = np.minimum(s.astype(np.int64), w0 - 1)
    return blk[..., i0] * (1 - (s - i0)) + blk[..., np.minimum(i0 + 1, w0 - 1)] * (s - i0)


def _tables(p, H, n, grid, blk):
    """The expected tables in order, fp64, padded agents 0."""
    h, w = grid
    NA, log2e = (n + 63) // 64 * 64, np.log2(np.e)
    pad = ((0, 0), (0, NA - n))
    for kind in "12":
        col, row, b = (p.get("b%s_%s" % (kind, c)) for c in ("col", "row", "blk"))
        if col is None and row is None and b is None:
            continue
        first = kind == "1"
        he = 1 if b is None else blk[0]
        T = np.zeros((H, he, n, w))      # [head, cell row, agent, x]
        if col is not None:
            T += (col if first else col.transpose(0, 2, 1))[:, None]
        if b is not None:
            T += _along_x(b.transpose(0, 2, 1, 3) if first else b.transpose(0, 1, 3, 2), w)
        T = np.pad(T * log2e, ((0, 0),) + (pad[0], pad[1], (0, 0)))
        yield T.reshape(H, he, NA, w // 4, 4).transpose(0, 1, 3, 2, 4) if first else T.reshape(H, he, NA // 4, 4, w).transpose(0, 1, 2, 4, 3)
        if row is not None:
            R = np.pad((row if first else row.transpose(0, 2, 1)) * log2e, pad + ((0, 0),))
            yield R.transpose(0, 2, 1) if first else R.reshape(H, NA // 4, 4, h).transpose(0, 1, 3, 2)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("H,grid,n,blk,absent", [
    (1, (5, 4), 65, (2, 3), ()),                              # one quad of columns; agents past 64
    (2, (33, 8), 126, (7, 5), ()),                            # narrow: waves take eight quads of agents side by side
    (3, (3, 28), 200, (1, 1), ("b1_row",)),
    (2, (17, 36), 81, (4, 7), ("b2_col",)),
    (8, (64, 64), 256, (7, 7), ()),                           # runs of cell rows in LDS, a last run of one
    (8, (70, 128), 320, (7, 1), ()),                          # the widest pieces; cell rows of one sample
    (8, (20, 100), 512, (3, 150), ("b1_col", "b2_row")),      # two cell rows' samples do not fit LDS
    (4, (9, 132), 300, (20, 9), ()),                          # finer than the image; 128 + 4 columns
    (8, (130, 64), 1024, (12, 3), ("b2_blk",)),
    (1, (12, 12), 70, (5, 2), ("b1_blk", "b2_row"))])
def test_half_resized_tables(aa, H, grid, n, blk, absent, shift):
    """shift: floats by which every parameter's base is off 16 bytes.  Bound: a component, its interpolation and their sum are rounded
    about six times (2^-24 of the largest sum each); a place between two samples, up to w0, is rounded three times, and moves the
    interpolation by that times their difference."""
    gen = np.random.default_rng(H * n + grid[1])
    p = {k: gen.standard_normal(s).astype(np.float32) for k, s in _shapes(H, n, grid, blk).items() if k not in absent}
    dev = {}
    for k, v in p.items():
        room = torch.empty(v.size + 4, device="cuda")
        room[shift:shift + v.size] = torch.from_numpy(v.reshape(-1)).cuda()
        dev[k] = room[shift:shift + v.size].reshape(v.shape)
        assert dev[k].data_ptr() % 16 == 4 * shift
    tables = aa.agent_attn_bias_tables(dev, heads=H, N=grid[0] * grid[1], n=n, d=32, dtype=torch.bfloat16, grid=grid)
    place = 3 * 2.0 ** -24 * blk[1] * 2 * max(float(np.abs(p[k]).max()) for k in ("b1_blk", "b2_blk") if k in p) * np.log2(np.e)
    got, at = tables.view(torch.float32).cpu().numpy().astype(np.float64), 0
    for want in _tables({k: v.astype(np.float64) for k, v in p.items()}, H, n, grid, blk):
        assert np.abs(got[at:at + want.size] - want.reshape(-1)).max() <= 6 * 2.0 ** -24 * np.abs(want).max() + place
        at += (want.size + 63) // 64 * 64
    assert at == got.size
