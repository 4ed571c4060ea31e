"""fp32 units taken in one launch: a few units, whose blocks share out one unit's tiles of tokens and tiles of channels, against the
same unit among enough others to have a block for itself (the same sums in the same order: equal bits) and against the fp64 oracle."""
import numpy as np
import pytest
import torch

from . import util

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def aa():
    from paper_2312_08874_amd import binding
    binding.lib()
    return binding


# (blocks along the tokens, 16-channel tiles a block takes) by the rule (split_rules.h): whole units first and last (one block, its own
# code), then one tile of one to four, two of two and four, three of three, four of four, ragged last tiles and shares, channels that
# end inside a tile
CASES = [
    ((3, 5), (2, 2), 16, 1, (1, 1)),
    ((8, 8), (4, 4), 32, 1, (1, 1)),
    ((13, 5), (5, 3), 20, 3, (2, 1)),
    ((14, 14), (7, 7), 16, 4, (4, 1)),
    ((14, 14), (7, 7), 32, 1, (4, 1)),
    ((11, 13), (7, 7), 48, 2, (3, 1)),
    ((10, 10), (8, 8), 64, 1, (2, 1)),
    ((9, 9), (3, 3), 64, 30, (2, 1)),
    ((14, 14), (7, 7), 32, 100, (2, 2)),
    ((9, 9), (3, 3), 64, 40, (2, 2)),
    ((11, 13), (7, 7), 48, 100, (2, 3)),
    ((9, 9), (3, 3), 64, 100, (2, 4)),
    ((14, 14), (7, 7), 16, 200, (1, 1)),
]


@pytest.mark.parametrize("grid,agrid,d,units,split", CASES)
@pytest.mark.parametrize("module,given", [(False, False), (True, False), (False, True)])
def test_shares_equal_whole_units(aa, oracle, grid, agrid, d, units, split, module, given):
    rng = np.random.default_rng(units + d)
    N, n = grid[0] * grid[1], agrid[0] * agrid[1]
    q, k, v = (rng.standard_normal((units, 1, N, d)).astype(np.float32) for _ in range(3))
    params = {"dwc_w": rng.standard_normal((1, d, 3, 3)) / 3, "dwc_b": rng.standard_normal((1, d))} if module else {}
    agents = rng.standard_normal((units, 1, n, d)).astype(np.float32) if given else None
    dev = {name: torch.from_numpy(x).cuda() for name, x in {"Q": q, "K": k, "V": v, **({"A": agents} if given else {})}.items()}
    residual = 0.5 if module else 0.0
    kw = dict(grid=grid, agent_grid=agrid, params=util.params_to_device(params) if module else None, v_residual_k=residual)
    few = aa.agent_attn_fwd(**dev, **kw)
    times = -(-257 // units)
    many = aa.agent_attn_fwd(**{name: x.repeat(times, 1, 1, 1) for name, x in dev.items()}, **kw)
    assert torch.equal(many, few.repeat(times, 1, 1, 1))
    ref = oracle.agent_attn_fwd(q[:, 0], k[:, 0], v[:, 0], heads=1, grid=grid, agent_grid=agrid, A=None if agents is None else agents[:, 0],
                                v_residual_k=residual, **params)
    util.assert_parity(util.to_host64(few)[:, 0], ref, "f32", "shares of a unit")
