"""Backward of units with at most 64 agents, whose agent kernels take the tokens' gradients as well, at the sizes where they
branch: agents at and beside the 16 of a wave and the 32 of a product step, tokens that end inside a tile of 32 or a column of
16, channels beside the padded width, one range and many (more than eight are added up first), given agents, the residual and the
convolution.  Reference and bars as in test_gpu_backward."""
import pytest

from paper_2312_08874_amd import inputs

from .test_gpu_backward import _run_case, _wl, aa  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
RESIDUAL = dict(v_residual_k=0.075)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("module", [False, True])
@pytest.mark.parametrize("grid,agrid,d", [((1, 1), (1, 1), 32), ((17, 19), (1, 15), 24), ((17, 19), (4, 4), 48), ((33, 16), (17, 1), 64),
                                          ((16, 31), (4, 8), 16), ((9, 34), (3, 11), 40), ((15, 47), (7, 9), 64), ((23, 17), (8, 8), 8),
                                          ((16, 16), (8, 8), 128), ((13, 33), (5, 13), 32), ((21, 9), (10, 6), 120)])
def test_both_sides_at_their_edges(aa, oracle, grid, agrid, d, module, dtype):  # noqa: F811
    _run_case(aa, oracle, _wl("both %s" % (agrid,), dtype, grid, agrid, d, batch=2, heads=2, index=61), module=module)


@pytest.mark.parametrize("dtype,d", [("f32", 32), ("bf16", 64), ("f16", 128)])
@pytest.mark.parametrize("module", [False, True])
@pytest.mark.parametrize("given", [False, True])
def test_both_sides_of_one_unit_in_many_ranges(aa, oracle, given, module, dtype, d):  # noqa: F811
    _run_case(aa, oracle, _wl("ranges", dtype, (61, 45), (7, 7), d, batch=1, heads=1, index=62), given=given, module=module,
              kw=RESIDUAL)


PLACES = [((17, 19), (4, 4), 32), ((14, 13), (4, 8), 64), ((12, 21), (5, 9), 48), ((16, 20), (8, 8), 40)]


def _tensors(grid, d, dtype, batch, heads, index):
    from . import util
    wl = _wl("places", dtype, grid, (1, 1), d, batch=batch, heads=heads, index=index)
    shape = (batch, heads, wl.N, d)
    t = [util.to_device(v, dtype, shape) for v in inputs.make_qkv(wl).values()]
    return t + [util.to_device(inputs.make_tensor((batch * heads, wl.N, d), stream=index * 16 + 12, dtype=dtype), dtype, shape)]


def _params(module, heads, n, d, grid):
    from . import util
    return dict(params=util.params_to_device(inputs.make_module_params(heads, n, d, grid, blk=(3, 2), index=66)) if module else None)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("module", [False, True])
@pytest.mark.parametrize("grid,agrid,d", PLACES)
def test_both_sides_of_strided_tensors(aa, grid, agrid, d, module, dtype):  # noqa: F811
    """Token-major tensors and slices of a fused projection have the dense call's gradients, bit for bit."""
    import torch
    dense = _tensors(grid, d, dtype, 2, 2, 66)
    kw = dict(grid=grid, agent_grid=agrid, v_residual_k=0.075, **_params(module, 2, agrid[0] * agrid[1], d, grid))
    ref = aa.agent_attn_bwd(*dense, **kw)
    major = [x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in dense]
    fused = torch.stack([x.permute(0, 2, 1, 3) for x in dense[:3]], dim=2).contiguous()
    for q, k, v, g in (major, [fused[:, :, i].permute(0, 2, 1, 3) for i in range(3)] + [major[3]], [fused[:, :, i].permute(0, 2, 1, 3) for i in range(3)] + [dense[3]]):
        got = aa.agent_attn_bwd(q, k, v, g, **kw)
        assert ref.keys() == got.keys() and all(torch.equal(got[key], ref[key]) for key in ref)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("module", [False, True])
@pytest.mark.parametrize("token_major", [False, True])
@pytest.mark.parametrize("window,agrid,d", PLACES)
def test_both_sides_of_windows(aa, window, agrid, d, token_major, module, dtype):  # noqa: F811
    """2 x 3 windows read where they lie have the gradients of window-major copies, bit for bit."""
    import torch
    (h, w), B, H = window, 2, 2
    image = _tensors((2 * h, 3 * w), d, dtype, B, H, 67)
    kw = dict(agent_grid=agrid, v_residual_k=0.075, **_params(module, H, agrid[0] * agrid[1], d, window))

    def part(x):
        return x.reshape(B, H, 2, h, 3, w, d).permute(0, 2, 4, 1, 3, 5, 6).reshape(B * 6, H, h * w, d).contiguous()
    ref = aa.agent_attn_bwd(*(part(x) for x in image), grid=window, **kw)
    if token_major:
        image = [x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in image]
    got = aa.agent_attn_bwd(*image, grid=(2 * h, 3 * w), window=window, **kw)
    assert ref.keys() == got.keys()
    for key in ref:
        assert torch.equal(part(got[key]) if key in ("dQ", "dK", "dV") else got[key], ref[key]), key


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("n,d", [(16, 32), (49, 64), (64, 48), (33, 128)])
def test_a_token_that_is_not_a_number_reaches_every_gradient_it_enters(aa, n, d, value, dtype):  # noqa: F811
    """Given agents: a query that is no finite number makes its weights NaN, hence dV_A = sum_t P2^T dO, and with it all of its
    unit's dK and dV; the gradients of the other queries, and of the other units, stay what they are."""
    import torch
    from . import util
    wl = _wl("nan", dtype, (13, 21), (1, n), d, batch=1, heads=2, index=63)
    t = {k: util.to_device(v, dtype, (1, 2, wl.N, d)) for k, v in inputs.make_qkv(wl).items()}
    rows = [util.to_device(inputs.make_tensor((2, r, d), stream=wl.index * 16 + 11 + i, dtype=dtype), dtype, (1, 2, r, d)) for i, r in ((0, n), (1, wl.N))]
    clean = aa.agent_attn_bwd(t["Q"], t["K"], t["V"], rows[1], rows[0])
    q = t["Q"].clone()
    q[0, 1, 37, 5] = value
    got = aa.agent_attn_bwd(q, t["K"], t["V"], rows[1], rows[0])
    for k in ("dK", "dV", "dA"):
        assert torch.isnan(got[k][0, 1]).all(), k
        assert torch.equal(got[k][0, 0], clean[k][0, 0]), k
    other = [i for i in range(wl.N) if i != 37]
    assert torch.isnan(got["dQ"][0, 1, 37]).all() and torch.equal(got["dQ"][0, 1, other], clean["dQ"][0, 1, other])
    assert torch.equal(got["dQ"][0, 0], clean["dQ"][0, 0])


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("grid,d", [((17, 19), 32), ((17, 20), 64), ((12, 16), 40)])
def test_a_residual_without_the_convolution_reads_its_own_token(aa, grid, d, dtype):  # noqa: F811
    """dV = P1^T dV_A + k dO: with an agent bias and no convolution an infinite dO adds to its own token's dV alone, so that the
    channel is as infinite as P1^T dV_A makes it everywhere (P1 > 0, the sign of dV_A's infinity is that of dO's).  Tokens of an
    image's last column also stand in for places beside it, with weights of 0, and are left out."""
    import torch
    from . import util
    wl = _wl("own", dtype, grid, (7, 7), d, batch=1, heads=2, index=64)
    t = {k: util.to_device(v, dtype, (1, 2, wl.N, d)) for k, v in inputs.make_qkv(wl).items()}
    dO = util.to_device(inputs.make_tensor((2, wl.N, d), stream=wl.index * 16 + 12, dtype=dtype), dtype, (1, 2, wl.N, d))
    params = {k: v for k, v in inputs.make_module_params(2, wl.n, d, grid, blk=(3, 2), index=64).items() if not k.startswith("dwc")}
    kw = dict(grid=grid, agent_grid=(7, 7), params=util.params_to_device(params), v_residual_k=0.3)
    clean = aa.agent_attn_bwd(t["Q"], t["K"], t["V"], dO, **kw)["dV"]
    for tok in (3, grid[1] + 2, wl.N - 2):
        g = dO.clone()
        g[0, 1, tok, 5] = float("inf")
        dV = aa.agent_attn_bwd(t["Q"], t["K"], t["V"], g, **kw)["dV"]
        assert torch.isposinf(dV[0, 1, :, 5]).all()
        rest = [c for c in range(d) if c != 5]
        assert torch.equal(dV[0, 0], clean[0, 0]) and torch.equal(dV[0, 1][:, rest], clean[0, 1][:, rest])


@pytest.mark.parametrize("grid,agrid,d", [((31, 43), (7, 9), 48), ((20, 33), (4, 8), 32), ((17, 50), (5, 5), 64)])
def test_fp32_value_gradient_rounds_no_more_than_nine_additions(aa, oracle, grid, agrid, d):  # noqa: F811
    """dV is nine weighted dO beside small products of the attention: added one after another onto the products, the partial sums
    grow evenly to the result, nine roundings that come to sqrt((1 + .. + 9) / 9) = sqrt(5) roundings of the result itself.  The bound
    leaves a twentieth for the products."""
    import numpy as np
    from . import util
    wl = _wl("rounding", "f32", grid, agrid, d, batch=1, heads=4, index=65)
    t = inputs.make_qkv(wl)
    dO = inputs.make_tensor((4, wl.N, d), stream=wl.index * 16 + 12, dtype="f32")
    params = inputs.make_module_params(4, wl.n, d, grid, blk=(3, 2), index=65)
    dev = {k: util.to_device(v, "f32", (1, 4, wl.N, d)) for k, v in t.items()}
    got = aa.agent_attn_bwd(dev["Q"], dev["K"], dev["V"], util.to_device(dO, "f32", (1, 4, wl.N, d)), grid=grid, agent_grid=agrid,
                            params=util.params_to_device(params))["dV"]
    B1, B2 = util.dense_biases(oracle, params, 4, wl.n, grid)
    ref = oracle.agent_attn_bwd(*(t[k].astype(np.float64) for k in ("Q", "K", "V")), dO.astype(np.float64), heads=4, grid=grid,
                                agent_grid=agrid, B1=B1, B2=B2, dwc_w=params["dwc_w"], dwc_b=params["dwc_b"])["dV"]
    one = np.linalg.norm(ref.astype(np.float32) - ref)
    err = np.linalg.norm(util.to_host64(got).reshape(ref.shape) - ref)
    print("dV error: %.3f roundings of the result" % (err / one))
    assert err <= 1.05 * np.sqrt(5) * one
