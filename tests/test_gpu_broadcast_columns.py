"""The broadcasts that take their tokens in columns.  Many agents (16 columns x 16 image rows a block, cell rows of the bias
tables beside the agents): edges of blocks and row pairs, the numbers of cell rows a stage holds and the first one past them,
components that are absent, masks, layouts, images that stay in rows.  Few agents with a convolution (a wave walks down image
rows): widths, every length of a walk, masks, layouts, an infinity.  Which kernel serves a case is asked of the dispatch rules
(columns_rule.h).  Reference: the fp64 oracle, with the forward's bars."""
import dataclasses

import numpy as np
import pytest

from paper_2312_08874_amd import inputs
from . import columns_rule, util

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def aa():
    from paper_2312_08874_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return columns_rule.load(str(tmp_path_factory.mktemp("rules")))


# grid, agent grid, block grid, components left out, cell rows in a stage (0: too many for one, taken in rows): rows 16 k + 1, + 15,
# a lone last row of a pair; columns 16 k + 4, + 12
CASES = [
    ((17, 20), (9, 8), (7, 7), (), 0),
    ((17, 20), (9, 8), (4, 7), (), 4),
    ((64, 16), (8, 9), (7, 7), (), 4),
    ((47, 36), (13, 10), (7, 5), ("b2_row",), 5),
    ((28, 20), (9, 8), (7, 7), (), 6),
    ((20, 12), (6, 12), (6, 7), ("b2_row",), 6),
    ((33, 28), (10, 10), (2, 3), ("b2_col",), 2),
    ((31, 12), (11, 6), (3, 2), ("b2_blk",), 1),
    ((16, 32), (8, 16), (4, 4), ("b1_col", "b1_row", "b1_blk"), 4),
    ((16, 24), (8, 12), (12, 7), (), 0),
    ((15, 64), (5, 14), (3, 7), ("dwc_w", "dwc_b"), 3),
]


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f16", 40), ("bf16", 24), ("f16", 128)])
@pytest.mark.parametrize("grid,agrid,blk,absent,parts", CASES)
def test_broadcast_in_columns(aa, oracle, rules, grid, agrid, blk, absent, parts, dtype, d):
    assert columns_rule.large_parts(rules, grid, agrid[0] * agrid[1], d, 4, 1 if "b2_blk" in absent else blk[0]) == parts
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=2, heads=2, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=14)
    t = inputs.make_qkv(wl)
    params = {k: v for k, v in inputs.make_module_params(2, wl.n, d, grid, blk=blk, index=14).items() if k not in absent}
    dev = {k: util.to_device(v, dtype, (2, 2, wl.N, d)) for k, v in t.items()}
    O = aa.agent_attn_fwd(dev["Q"], dev["K"], dev["V"], grid=grid, agent_grid=agrid, params=util.params_to_device(params),
                          v_residual_k=0.25)
    ref = util.oracle_forward_units(oracle, wl, t, list(range(4)), params=params, v_residual_k=0.25)
    util.assert_parity(util.to_host64(O).reshape(ref.shape), ref, dtype, "broadcast in columns",
                       max_abs=1e-2 * max(1.0, float(np.abs(ref).max())))


@pytest.mark.parametrize("mask", [-1e4, -1e9, float(np.finfo(np.float32).min), -np.inf])
@pytest.mark.parametrize("key,where", [("b2_row", (slice(None), slice(0, 5), slice(0, 70))), ("b2_col", (slice(None), slice(2, 9), slice(1, None))),
                                       ("b2_blk", (slice(None), slice(0, 2), slice(None), slice(0, 64)))])
def test_broadcast_in_columns_masks(aa, oracle, key, where, mask):
    """Agents masked for some tokens, the whole first chunk among them.  A masked weight is zero at any of these values, so
    the oracle's value at -1e4 is the reference for all."""
    grid, agrid, d, dtype = (35, 24), (9, 9), 64, "f16"
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=1, heads=2, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=14)
    t = inputs.make_qkv(wl)
    params = inputs.make_module_params(2, wl.n, d, grid, blk=(7, 7), index=14)
    ref_params = {k: v.copy() for k, v in params.items()}
    params[key][where] = mask
    ref_params[key][where] = -1e4
    dev = {k: util.to_device(v, dtype, (1, 2, wl.N, d)) for k, v in t.items()}
    O = aa.agent_attn_fwd(dev["Q"], dev["K"], dev["V"], grid=grid, agent_grid=agrid, params=util.params_to_device(params))
    ref = util.oracle_forward_units(oracle, wl, t, [0, 1], params=ref_params)
    util.assert_parity(util.to_host64(O).reshape(ref.shape), ref, dtype, "masked broadcast in columns",
                       max_abs=1e-2 * max(1.0, float(np.abs(ref).max())))


# many units of narrow images and of images with one row past a block: in rows and in columns by the rule (d, columns)
@pytest.mark.parametrize("d,dtype,columns", [(64, "bf16", False), (24, "f16", True), (128, "f16", True)])
@pytest.mark.parametrize("units,grid,agrid,blk", [(300, (17, 8), (9, 8), (4, 7)), (150, (36, 4), (18, 4), (5, 5)), (150, (29, 20), (13, 5), (7, 7))])
def test_broadcast_of_narrow_images(aa, oracle, rules, units, grid, agrid, blk, d, dtype, columns):
    """Units repeat with a period of six (three images, two heads): every one has the output of its first, bit for bit."""
    import torch
    assert bool(columns_rule.large_parts(rules, grid, agrid[0] * agrid[1], d, units, blk[0])) == columns
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=3, heads=2, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=17)
    t = inputs.make_qkv(wl)
    params = inputs.make_module_params(2, wl.n, d, grid, blk=blk, index=17)
    dev = {k: util.to_device(v, dtype, (3, 2, wl.N, d)).repeat(units // 6, 1, 1, 1) for k, v in t.items()}
    O = aa.agent_attn_fwd(dev["Q"], dev["K"], dev["V"], grid=grid, agent_grid=agrid, params=util.params_to_device(params))
    assert torch.equal(O, O[:3].repeat(units // 6, 1, 1, 1))
    ref = util.oracle_forward_units(oracle, wl, t, list(range(6)), params=params)
    util.assert_parity(util.to_host64(O[:3]).reshape(ref.shape), ref, dtype, "broadcast of narrow images",
                       max_abs=1e-2 * max(1.0, float(np.abs(ref).max())))


def _layouts(t, B, H, N, d, dtype):
    """(layout, Q, K, V, out): token-major, fused projection rows with a dense output, dense with padded rows of output."""
    import torch
    dense = [util.to_device(t[k], dtype, (B, H, N, d)) for k in ("Q", "K", "V")]
    yield ("token",) + tuple(x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in dense) + \
        (torch.full((B, N, H, d), float("nan"), dtype=dense[0].dtype, device="cuda").permute(0, 2, 1, 3),)
    qkv = torch.stack([x.permute(0, 2, 1, 3) for x in dense], dim=2).contiguous()
    yield ("qkv",) + tuple(qkv[:, :, i].permute(0, 2, 1, 3) for i in range(3)) + (torch.full_like(dense[0], float("nan")),)
    yield ("padded",) + tuple(dense) + (torch.full((B, H, N, d + 24), float("nan"), dtype=dense[0].dtype, device="cuda")[..., 8:8 + d],)


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f16", 40), ("bf16", 24), ("f16", 128)])
def test_broadcast_in_columns_layouts(aa, oracle, rules, dtype, d):
    """Token tensors and outputs in strides of their own have the dense call's values, bit for bit."""
    import torch
    grid, agrid = (35, 24), (9, 9)
    assert columns_rule.large_parts(rules, grid, 81, d, 4, 7)
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=2, heads=2, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=18)
    t = inputs.make_qkv(wl)
    params = inputs.make_module_params(2, wl.n, d, grid, blk=(7, 7), index=18)
    ref = util.oracle_forward_units(oracle, wl, t, list(range(4)), params=params, v_residual_k=0.25)
    kw = dict(grid=grid, agent_grid=agrid, params=util.params_to_device(params), v_residual_k=0.25)
    dense = aa.agent_attn_fwd(*(util.to_device(t[k], dtype, (2, 2, wl.N, d)) for k in ("Q", "K", "V")), **kw)
    util.assert_parity(util.to_host64(dense).reshape(ref.shape), ref, dtype, "dense", max_abs=1e-2 * max(1.0, float(np.abs(ref).max())))
    for name, q, k, v, out in _layouts(t, 2, 2, wl.N, d, dtype):
        aa.agent_attn_fwd(q, k, v, out=out, **kw)
        assert torch.equal(out, dense), name


# Half-resized tables of both kinds made in runs of cell rows, as many as leave a block per CU (kind 1 at widths padded to 32 and
# 128; at 64 its block component has another form)
@pytest.mark.parametrize("dtype,d", [("bf16", 32), ("f16", 96)])
@pytest.mark.parametrize("blk,runs", [((7, 7), 3), ((5, 3), 2)])
def test_half_resized_tables_in_runs(aa, oracle, blk, runs, dtype, d):
    grid, agrid, heads = (64, 64), (16, 16), 8
    blocks = heads * blk[0] * (256 // 64) * (64 // 16)      # of 64 agents x 16 columns of a cell row; kind 2: 64 columns x 16 agents
    assert blocks // 2 < 512 and blocks // 256 == runs and blk[0] % runs == 1      # (blocks of 32 would leave fewer than two a CU)
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=1, heads=heads, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=19)
    t = inputs.make_qkv(wl)
    params = inputs.make_module_params(heads, wl.n, d, grid, blk=blk, index=19)
    dev = {k: util.to_device(v, dtype, (1, heads, wl.N, d)) for k, v in t.items()}
    O = aa.agent_attn_fwd(dev["Q"], dev["K"], dev["V"], grid=grid, agent_grid=agrid, params=util.params_to_device(params))
    units, rows = [0, 3, 7], np.arange(0, wl.N, 37)
    ref = util.oracle_forward_units(oracle, wl, t, units, rows=rows, params=params)
    util.assert_parity(util.to_host64(O)[0][units][:, rows], ref, dtype, "tables in runs", max_abs=1e-2 * max(1.0, float(np.abs(ref).max())))


# the small-agent broadcast with a convolution: widths on both sides of whole sixteens and of the rule, a last segment of one
# image row, one image row in all, 1 .. 4 agent tiles
SMALL = [((31, 44), (7, 7)), ((33, 33), (4, 4)), ((16, 64), (3, 11)), ((65, 15), (8, 8)), ((22, 50), (5, 6)), ((1, 700), (1, 40)), ((64, 17), (7, 7))]


@pytest.mark.parametrize("dtype,d", [("bf16", 32), ("f16", 64)])
@pytest.mark.parametrize("absent", [(), ("b1_col", "b1_row", "b1_blk", "b2_col", "b2_row", "b2_blk"), ("dwc_b", "b2_row")])
@pytest.mark.parametrize("grid,agrid", SMALL)
def test_small_broadcast_in_columns(aa, oracle, rules, grid, agrid, absent, dtype, d):
    assert bool(rules.small_columns(grid[1], 2 * d)) == (grid != (64, 17))
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=2, heads=2, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=15)
    t = inputs.make_qkv(wl)
    params = {k: v for k, v in inputs.make_module_params(2, wl.n, d, grid, blk=(7, 7), index=15).items() if k not in absent}
    # token-major: the rows of one unit are not neighbours
    dev = {k: util.to_device(v, dtype, (2, 2, wl.N, d)).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for k, v in t.items()}
    vk = 0.25 if absent else 0.0
    O = aa.agent_attn_fwd(dev["Q"], dev["K"], dev["V"], grid=grid, agent_grid=agrid, params=util.params_to_device(params),
                          v_residual_k=vk)
    ref = util.oracle_forward_units(oracle, wl, t, list(range(4)), params=params, v_residual_k=vk)
    util.assert_parity(util.to_host64(O).reshape(ref.shape), ref, dtype, "small broadcast in columns",
                       max_abs=1e-2 * max(1.0, float(np.abs(ref).max())))


@pytest.mark.parametrize("dtype,d", [("f16", 64), ("bf16", 32)])
def test_small_broadcast_output_rows_past_4_gib(aa, oracle, dtype, d):
    """One image row of 600 tokens into a column slice of a buffer whose rows are 8 MiB: column 512 is 4 GiB past the first."""
    import torch
    grid, agrid = (1, 600), (1, 40)
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=1, heads=1, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=16)
    t = inputs.make_qkv(wl)
    params = {k: v for k, v in inputs.make_module_params(1, wl.n, d, grid, blk=(7, 7), index=16).items() if k in ("dwc_w", "dwc_b")}
    dev = {k: util.to_device(v, dtype, (1, 1, wl.N, d)) for k, v in t.items()}
    rows = torch.empty(600, 1 << 22, dtype=util.torch_dtype(dtype), device="cuda")
    out = rows[:, 8:8 + d].view(1, 1, 600, d)
    out.fill_(float("nan"))
    aa.agent_attn_fwd(dev["Q"], dev["K"], dev["V"], grid=grid, agent_grid=agrid, params=util.params_to_device(params), out=out)
    ref = util.oracle_forward_units(oracle, wl, t, [0], params=params)
    util.assert_parity(util.to_host64(out).reshape(ref.shape), ref, dtype, "output rows past 4 GiB",
                       max_abs=1e-2 * max(1.0, float(np.abs(ref).max())))


# units, grid, image rows a wave walks down: two swaps of its register sets and a third tile, the listed image's seven, an even number, a
# last walk shorter than the others, the whole height in one walk (even and odd)
WALKS = [(150, (35, 44), 5), (96, (56, 56), 7), (192, (40, 33), 8), (192, (31, 44), 7), (390, (40, 24), 10), (798, (22, 50), 22), (798, (23, 50), 23)]


@pytest.mark.parametrize("dtype,d", [("bf16", 32), ("f16", 64)])
@pytest.mark.parametrize("units,grid,rows", WALKS)
def test_small_broadcast_walks(aa, oracle, rules, units, grid, rows, dtype, d):
    """Walks of every length: with few units they are four image rows.  Units repeat with a period of six."""
    import torch
    assert rules.small_column_segment(units, *grid) == rows and rules.small_columns(grid[1], 2 * d)
    agrid = (7, 7)
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=3, heads=2, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=20)
    t = inputs.make_qkv(wl)
    params = inputs.make_module_params(2, wl.n, d, grid, blk=(7, 7), index=20)
    # token-major: the rows of one unit are not neighbours
    dev = {k: util.to_device(v, dtype, (3, 2, wl.N, d)).permute(0, 2, 1, 3).contiguous().repeat(units // 6, 1, 1, 1).permute(0, 2, 1, 3)
           for k, v in t.items()}
    O = aa.agent_attn_fwd(dev["Q"], dev["K"], dev["V"], grid=grid, agent_grid=agrid, params=util.params_to_device(params))
    assert torch.equal(O, O[:3].repeat(units // 6, 1, 1, 1))
    ref = util.oracle_forward_units(oracle, wl, t, list(range(6)), params=params)
    util.assert_parity(util.to_host64(O[:3]).reshape(ref.shape), ref, dtype, "small broadcast, walks",
                       max_abs=1e-2 * max(1.0, float(np.abs(ref).max())))


@pytest.mark.parametrize("dtype,d", [("bf16", 32), ("f16", 64)])
def test_small_broadcast_layouts(aa, oracle, rules, dtype, d):
    """Token tensors and outputs in strides of their own have the dense call's values, bit for bit."""
    import torch
    grid, agrid = (31, 44), (7, 7)
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=2, heads=3, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=21)
    t = inputs.make_qkv(wl)
    params = inputs.make_module_params(3, wl.n, d, grid, blk=(7, 7), index=21)
    ref = util.oracle_forward_units(oracle, wl, t, list(range(6)), params=params)
    kw = dict(grid=grid, agent_grid=agrid, params=util.params_to_device(params))
    dense = aa.agent_attn_fwd(*(util.to_device(t[k], dtype, (2, 3, wl.N, d)) for k in ("Q", "K", "V")), **kw)
    util.assert_parity(util.to_host64(dense).reshape(ref.shape), ref, dtype, "dense", max_abs=1e-2 * max(1.0, float(np.abs(ref).max())))
    for name, q, k, v, out in _layouts(t, 2, 3, wl.N, d, dtype):
        assert rules.small_columns(grid[1], out.stride(2))
        aa.agent_attn_fwd(q, k, v, out=out, **kw)
        assert torch.equal(out, dense), name


@pytest.mark.parametrize("key,where,mask", [
    (key, where, mask) for mask in (-1e4, -1e9, float(np.finfo(np.float32).min), -np.inf)
    for key, where in (("b2_row", (slice(None), slice(0, 5), slice(0, 20))), ("b2_col", (slice(None), slice(2, 9), slice(1, None))),
                       ("b2_blk", (slice(None), slice(0, 2), slice(None), slice(0, 16))))
    # (a dense table is evaluated with the formula as it stands: an infinite block value makes its interpolation NaN)
    if not (key == "b2_blk" and mask == -np.inf)])
def test_small_broadcast_masks(aa, oracle, key, where, mask):
    """Agents masked for some tokens, the whole first tile among them; reference as in test_broadcast_in_columns_masks."""
    grid, agrid, d, dtype = (31, 44), (7, 7), 32, "bf16"
    wl = dataclasses.replace(inputs.WORKLOADS["tiny"], batch=1, heads=2, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=22)
    t = inputs.make_qkv(wl)
    params = inputs.make_module_params(2, wl.n, d, grid, blk=(7, 7), index=22)
    ref_params = {k: v.copy() for k, v in params.items()}
    params[key][where] = mask
    ref_params[key][where] = -1e4
    dev = {k: util.to_device(v, dtype, (1, 2, wl.N, d)) for k, v in t.items()}
    O = aa.agent_attn_fwd(dev["Q"], dev["K"], dev["V"], grid=grid, agent_grid=agrid, params=util.params_to_device(params))
    ref = util.oracle_forward_units(oracle, wl, t, [0, 1], params=ref_params)
    util.assert_parity(util.to_host64(O).reshape(ref.shape), ref, dtype, "masked small broadcast",
                       max_abs=1e-2 * max(1.0, float(np.abs(ref).max())))


@pytest.mark.parametrize("dtype,d,agrid", [("bf16", 32, (7, 7)), ("f16", 64, (7, 7)), ("f16", 64, (9, 9))])
@pytest.mark.parametrize("corner", [(0, 0), (0, -1), (-1, 0), (-1, -1), (4, 15)])
def test_broadcast_in_columns_keeps_an_infinity_in_its_channel(aa, corner, dtype, d, agrid):
    """An infinity in one channel of V makes that channel of its unit infinite or NaN (every agent holds a share of it) and changes
    nothing else: neither other channels and units, nor through the convolution's clamped addresses the other side of the image."""
    import torch
    h, w = 35, 48
    gen = torch.Generator(device="cuda").manual_seed(23)
    q, k, v = (torch.randn(2, 2, h * w, d, generator=gen, device="cuda").to(util.torch_dtype(dtype)) for _ in range(3))
    params = util.params_to_device(inputs.make_module_params(2, agrid[0] * agrid[1], d, (h, w), blk=(7, 7), index=23))
    outs = []
    for value in (0.0, float("inf")):
        v.view(2, 2, h, w, d)[0, 1, corner[0], corner[1], 3] = value
        outs.append(aa.agent_attn_fwd(q, k, v, grid=(h, w), agent_grid=agrid, params=params))
    touched = torch.zeros_like(outs[0], dtype=torch.bool)
    touched[0, 1, :, 3] = True
    assert not torch.isfinite(outs[1][touched]).any()
    assert torch.isfinite(outs[0]).all() and torch.equal(outs[1][~touched], outs[0][~touched])
