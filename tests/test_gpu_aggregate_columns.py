"""The aggregation that takes its tokens in columns (tiles of 16 image columns x 4 image rows down a strip): strips that reach
beside the image, strips that end inside a tile, tiles across two and more cell rows, strips longer than the 64 image rows whose
weights are held at a time, splits that begin inside a strip, absent components, masks, prepared tables.  Which kernel serves a
case is asked of the dispatch rule.  Reference: the fp64 oracle, with the forward's bars."""
import dataclasses

import numpy as np
import pytest

from paper_2312_08874_amd import inputs
from . import columns_rule, util
from .test_gpu_broadcast_columns import _layouts

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def aa():
    from paper_2312_08874_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return columns_rule.load(str(tmp_path_factory.mktemp("rules")))


def _forward(aa, oracle, rules, grid, agrid, blk, absent, dtype, d, *, mask=None, units=(2, 2), n_splits=0, tables=False):
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=units[0], heads=units[1], grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=24)
    assert columns_rule.aggregate_columns(rules, grid, wl.n, d, 1 if "b1_blk" in absent else blk[0])
    t = inputs.make_qkv(wl)
    params = {k: v for k, v in inputs.make_module_params(units[1], wl.n, d, grid, blk=blk, index=24).items() if k not in absent}
    ref_params = {k: v.copy() for k, v in params.items()}
    if mask:
        key, where, value = mask
        params[key][where], ref_params[key][where] = value, -1e4
    dev = {k: util.to_device(v, dtype, units + (wl.N, d)) for k, v in t.items()}
    kw = dict(grid=grid, agent_grid=agrid, params=util.params_to_device(params), v_residual_k=0.25)
    if n_splits:
        kw["n_splits"] = n_splits
    if tables:
        kw["params"]["bias_tables"] = aa.agent_attn_bias_tables(kw["params"], heads=units[1], N=wl.N, n=wl.n, d=d, dtype=dev["Q"].dtype, grid=grid)
    O = aa.agent_attn_fwd(dev["Q"], dev["K"], dev["V"], **kw)
    ref = util.oracle_forward_units(oracle, wl, t, list(range(units[0] * units[1])), params=ref_params, v_residual_k=0.25)
    util.assert_parity(util.to_host64(O).reshape(ref.shape), ref, dtype, "aggregation in columns",
                       max_abs=1e-2 * max(1.0, float(np.abs(ref).max())))


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 72)])
@pytest.mark.parametrize("grid,agrid,blk,absent", [
    ((8, 16), (8, 10), (1, 1), ("b1_row",)),           # two tiles, one cell row
    ((7, 44), (7, 10), (9, 7), ()),                    # a finer block grid than the image
    ((18, 48), (9, 8), (18, 3), ("b1_col",)),          # a cell row an image row
    ((23, 28), (11, 9), (7, 7), ()),                   # about three image rows a cell row, 16 + 12 columns
    ((66, 12), (11, 12), (4, 5), ("b1_row",)),         # past 64 image rows; one strip, 12 columns
    ((131, 32), (9, 15), (2, 9), ()),
    ((40, 60), (10, 13), (7, 7), ("b1_blk",)),         # no cell rows at all
    ((37, 64), (12, 22), (5, 2), ("b2_col", "b2_row", "b2_blk"))])
def test_aggregation_in_columns(aa, oracle, rules, grid, agrid, blk, absent, dtype, d):
    _forward(aa, oracle, rules, grid, agrid, blk, absent, dtype, d)


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f16", 32), ("f16", 40)])
@pytest.mark.parametrize("grid,agrid,blk,absent", [((70, 28), (20, 13), (7, 7), ()), ((83, 44), (20, 20), (5, 7), ("b1_row",)), ((41, 36), (17, 17), (3, 2), ("b1_col",))])
def test_aggregation_in_columns_of_many_agents(aa, oracle, rules, grid, agrid, blk, absent, dtype, d):
    _forward(aa, oracle, rules, grid, agrid, blk, absent, dtype, d)


@pytest.mark.parametrize("n_splits", [1, 2, 5, 11])
@pytest.mark.parametrize("grid,agrid,d", [((26, 44), (9, 8), 128), ((53, 28), (18, 15), 64)])
def test_aggregation_in_columns_splits(aa, oracle, rules, grid, agrid, d, n_splits):
    """Splits that begin inside a strip, and inside a cell row."""
    _forward(aa, oracle, rules, grid, agrid, (5, 3), (), "bf16", d, units=(1, 2), n_splits=n_splits, tables=n_splits == 5)


@pytest.mark.parametrize("dtype,d,grid,agrid", [("bf16", 64, (70, 28), (20, 13)), ("f16", 40, (83, 44), (20, 20)), ("f16", 32, (70, 28), (20, 13)),
                                                ("bf16", 24, (41, 36), (17, 17)), ("bf16", 128, (23, 28), (11, 9))])
def test_aggregation_in_columns_layouts(aa, rules, dtype, d, grid, agrid):
    """Token-major tensors, slices of a fused projection and padded outputs have the dense call's values, bit for bit."""
    import torch
    blk = (3, 2) if grid[0] == 41 else (7, 7)
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=2, heads=2, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=27)
    assert columns_rule.aggregate_columns(rules, grid, wl.n, d, blk[0])
    t = inputs.make_qkv(wl)
    kw = dict(grid=grid, agent_grid=agrid, v_residual_k=0.25,
              params=util.params_to_device(inputs.make_module_params(2, wl.n, d, grid, blk=blk, index=27)))
    dense = aa.agent_attn_fwd(*(util.to_device(t[k], dtype, (2, 2, wl.N, d)) for k in ("Q", "K", "V")), **kw)
    for name, q, k, v, out in _layouts(t, 2, 2, wl.N, d, dtype):
        aa.agent_attn_fwd(q, k, v, out=out, **kw)
        assert torch.equal(out, dense), name


@pytest.mark.parametrize("value", [-1e9, float(np.finfo(np.float32).min), -np.inf])
@pytest.mark.parametrize("key,where", [("b1_row", (slice(None), slice(0, 70), slice(0, 9))), ("b1_col", (slice(None), slice(3, None), slice(0, 17))),
                                       ("b1_blk", (slice(None), slice(0, 50), slice(0, 2))), ("b1_blk", (slice(None), 5, slice(None), 1))])
def test_aggregation_in_columns_masks(aa, oracle, rules, key, where, value):
    """Tokens masked for some agents, the first tiles of a strip and whole cell rows among them.  A masked weight is zero at any of
    these values, so the oracle's value at -1e4 is the reference for all."""
    _forward(aa, oracle, rules, (35, 28), (10, 9), (7, 7), (), "f16", 128, mask=(key, where, value))


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64)])
def test_aggregation_in_columns_infinite_corner(aa, rules, dtype, d):
    """An infinite value of a token reaches its own channels only: places beside the image read zeros, not the next image row."""
    import torch
    grid, agrid = (70, 28), (20, 14)
    n = agrid[0] * agrid[1]
    assert columns_rule.aggregate_columns(rules, grid, n, d, 7)
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=1, heads=1, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=25)
    t = inputs.make_qkv(wl)
    dev = {k: util.to_device(v, dtype, (1, 1, wl.N, d)) for k, v in t.items()}
    params = inputs.make_module_params(1, n, d, grid, blk=(7, 7), index=25)
    params = util.params_to_device({k: v for k, v in params.items() if k[:2] in ("b1", "b2")})
    clean = aa.agent_attn_fwd(dev["Q"], dev["K"], dev["V"], grid=grid, agent_grid=agrid, params=params)
    for tok in (grid[1] * 3, grid[1] * 4 - 1, wl.N - 1):
        v = dev["V"].clone()
        v[0, 0, tok, 5] = float("inf")
        O = aa.agent_attn_fwd(dev["Q"], dev["K"], v, grid=grid, agent_grid=agrid, params=params)
        assert not bool(torch.isfinite(O[..., 5]).any())
        rest = [c for c in range(d) if c != 5]
        assert torch.equal(O[..., rest], clean[..., rest])
