"""GPU parity of the backward pass (agent_attn_bwd through the C ABI) against the fp64 oracle's
gradients on the same seeded inputs.

Bar, per gradient tensor g with reference r: fp32 path max-abs <= 1e-4 * max(1, max|r|); fp16 / bf16
paths max-abs <= 1e-2 * max(1, max|r|) and relative L2 <= 5e-3, except bf16 problems with module terms, wider
than 128 or with the enlarged second scale of Appendix C.1 (see _check): 1e-2 (a gradient of theirs chains three
operands of relative error up to 2^-9; five unit roundoffs, as for the parameter gradients below; a near
one-hot broadcast softmax - the SD variant's scale d^-0.15 together with a bias - reaches 7e-3).  Up to 128
channels the kernels recompute their score tiles and round P and dS once, as operands
of the next product.  fp32 parameter gradients relative L2 <= 1e-4 (fp32 inputs), 5e-3 (fp16 inputs) or 1e-2
(bf16 inputs): the probabilities, V_A and dV_A that feed the MFMA products are rounded to the element
type, each with a relative error of up to one unit roundoff (2^-9 for bf16, 2^-11 for fp16), and a
parameter gradient chains three such operands; the bar is five unit roundoffs for bf16, and a
single small image (no averaging over a batch) reaches 5.4e-3.

With pooled agents the GPU rounds A to the element type as its forward does, and differentiates
through that rounding as if it were the identity.  For the 16-bit types the reference is therefore
assembled from oracle pieces fed with the GPU's pooled A: the gradient for given agents, plus the
pooling gradient of dA.
"""
import dataclasses

import numpy as np
import pytest

from paper_2312_08874_amd import inputs
from tests import util

pytestmark = pytest.mark.gpu
WL = inputs.WORKLOADS


@pytest.fixture(scope="module")
def aa():
    import torch
    assert torch.cuda.is_available()
    from paper_2312_08874_amd import binding
    binding.lib()
    return binding


def _stored(t, dtype, shape):
    import torch
    a = t.reshape(shape).cpu()
    if dtype == "bf16":
        return a.view(torch.int16).numpy().view(np.uint16)
    return a.numpy()


def _check(got, ref, dtype, what, pure=False):
    """pure: a problem without module terms and with the default scales, served by the kernels that keep P and dS
    in fp32 up to the one rounding that makes them matrix operands: the bf16 bar is the forward's 5e-3 there.
    With the enlarged second scale of Appendix C.1 (d^-0.15 instead of d^-0.5: scores four times larger at d = 64)
    the broadcast softmax is peaked, dS2 = P2 o (dP2 - D2) is a small difference of larger terms, and the 2^-9
    roundings behind dP2 = dO V_A^T show (V_A as an operand, P1 as the operand of the product that gives V_A:
    6e-3 .. 7e-3 each in an fp64 emulation with one rounding switched on at a time): dQ reaches 7.4e-3 on seeded
    random problems (two-term dS2 operands did not move it), so those keep the 1e-2 of the problems with module
    terms."""
    scale = max(1.0, float(np.abs(ref).max()))
    util.assert_parity(util.to_host64(got).reshape(ref.shape), ref, dtype, what,
                       max_abs=util.TOL[dtype]["max_abs"] * scale,
                       rel_l2=1e-2 if dtype == "bf16" and not pure else None)


def _check_param(got, ref, dtype, what, floor=0.0):
    """floor: the size a sum of the same terms with random signs would have (root of the summed squares).
    A parameter gradient whose terms cancel exactly (a bias component that is constant along the softmax
    axis, e.g. the column component of a one-column grid) has a reference of 0 and is measured against it."""
    err = float(np.linalg.norm(util.to_host64(got).reshape(ref.shape) - ref))
    rel = err / max(float(np.linalg.norm(ref)), floor, 1e-300)
    assert rel <= {"f32": 1e-4, "f16": 5e-3, "bf16": 1e-2}[dtype], "%s: rel_l2 %.3e" % (what, rel)


def _run_case(aa, oracle, wl, *, given=False, module=False, blk=(3, 2), kw=None, scale_qk=1.0, mask=None):
    """mask: (parameter, index, value, value for the reference)"""
    kw = kw or {}
    t = inputs.make_qkv(wl, scale_qk=scale_qk)
    dO = inputs.make_tensor((wl.units, wl.N, wl.d), stream=wl.index * 16 + 12, dtype=wl.dtype)
    shape = (wl.batch, wl.heads, wl.N, wl.d)
    dv = {k: util.to_device(v, wl.dtype, shape) for k, v in t.items()}
    dOd = util.to_device(dO, wl.dtype, shape)
    params = inputs.make_module_params(wl.heads, wl.n, wl.d, wl.grid, blk=blk, index=wl.index) if module else None
    if mask:
        params[mask[0]][mask[1]] = mask[2]
    pd = util.params_to_device(params) if module else None
    if mask:
        params[mask[0]][mask[1]] = mask[3]
    A_st = None
    if given:
        A_st = inputs.make_tensor((wl.units, wl.n, wl.d), stream=wl.index * 16 + 11, dtype=wl.dtype)
        Ad = util.to_device(A_st, wl.dtype, (wl.batch, wl.heads, wl.n, wl.d))
        got = aa.agent_attn_bwd(dv["Q"], dv["K"], dv["V"], dOd, Ad, grid=wl.grid if module else None, params=pd, **kw)
    else:
        got = aa.agent_attn_bwd(dv["Q"], dv["K"], dv["V"], dOd, grid=wl.grid, agent_grid=wl.agent_grid, params=pd, **kw)

    f64 = {k: inputs.to_float64(v, wl.dtype) for k, v in t.items()}
    B1 = B2 = None
    okw = dict(heads=wl.heads, grid=wl.grid, scale1=kw.get("scale1") or None, scale2=kw.get("scale2") or None,
               v_residual_k=kw.get("v_residual_k", 0.0))
    if module:
        B1, B2 = util.dense_biases(oracle, params, wl.heads, wl.n, wl.grid)
        okw.update(B1=B1, B2=B2, dwc_w=params["dwc_w"], dwc_b=params["dwc_b"])
    g64 = inputs.to_float64(dO, wl.dtype)
    if given:
        ref = oracle.agent_attn_bwd(f64["Q"], f64["K"], f64["V"], g64, A=inputs.to_float64(A_st, wl.dtype), **okw)
    elif wl.dtype == "f32":
        ref = oracle.agent_attn_bwd(f64["Q"], f64["K"], f64["V"], g64, agent_grid=wl.agent_grid, **okw)
    else:
        A_gpu = aa.agent_pool_fwd(dv["Q"], grid=wl.grid, agent_grid=wl.agent_grid)
        A64 = inputs.to_float64(_stored(A_gpu, wl.dtype, (wl.units, wl.n, wl.d)), wl.dtype)
        ref = oracle.agent_attn_bwd(f64["Q"], f64["K"], f64["V"], g64, A=A64, agent_grid=wl.agent_grid, **okw)
        ref["dQ"] = ref["dQ"] + oracle.pool_bwd(ref.pop("dA"), *wl.grid, *wl.agent_grid)
    for k in ("dQ", "dK", "dV") + (("dA",) if given else ()):
        _check(got[k], ref[k], wl.dtype, "%s %s" % (wl.name, k),
               pure=not module and not kw.get("scale2") and wl.d % 8 == 0 and wl.d <= 128)
    if module:
        h0, w0 = blk
        gh, gw = wl.grid
        for hd in range(wl.heads):
            c1, r1, b1 = oracle.bias1_components_bwd(ref["dB1"][hd], gh, gw, h0, w0)
            c2, r2, b2 = oracle.bias2_components_bwd(ref["dB2"][hd], gh, gw, h0, w0)
            sq = oracle.bias1_components_bwd(ref["dB1"][hd] ** 2, gh, gw, h0, w0) + \
                oracle.bias2_components_bwd(ref["dB2"][hd] ** 2, gh, gw, h0, w0)
            for (key, r), q in zip((("db1_col", c1), ("db1_row", r1), ("db1_blk", b1), ("db2_col", c2), ("db2_row", r2),
                                    ("db2_blk", b2)), sq):
                _check_param(got[key][hd], r, wl.dtype, "%s %s head %d" % (wl.name, key, hd),
                             floor=float(np.sqrt(np.abs(q).sum())))
        _check_param(got["ddwc_w"], ref["ddwc_w"], wl.dtype, wl.name + " ddwc_w")
        _check_param(got["ddwc_b"], ref["ddwc_b"], wl.dtype, wl.name + " ddwc_b")
    if mask and (wl.dtype == "f32" or wl.n > 64 or mask[0][3:] != "blk" or np.isfinite(mask[2])):
        # (a dense table is evaluated with the formula as it stands: an infinite block value makes its interpolation NaN)
        out = aa.agent_attn_fwd(dv["Q"], dv["K"], dv["V"], Ad, grid=wl.grid, params=pd, **kw)
        _check(out, oracle.agent_attn_fwd(f64["Q"], f64["K"], f64["V"], A=inputs.to_float64(A_st, wl.dtype), **okw), wl.dtype,
               wl.name + " out")
    return got


def _wl(name, dtype, grid, agrid, d, batch=2, heads=2, index=13):
    return dataclasses.replace(WL["tiny"], name=name, batch=batch, heads=heads, grid=grid, agent_grid=agrid, d=d,
                               dtype=dtype, index=index)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("grid,agrid,d", [((14, 14), (7, 7), 32), ((13, 11), (4, 3), 24), ((1, 1), (1, 1), 8),
                                          ((9, 70), (3, 9), 72), ((20, 20), (5, 5), 64)])
def test_backward_pure_pooled(aa, oracle, grid, agrid, d, dtype):
    _run_case(aa, oracle, _wl("pure", dtype, grid, agrid, d))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_backward_given_agents(aa, oracle, dtype):
    wl = _wl("given", dtype, (10, 13), (1, 20), 40)
    _run_case(aa, oracle, wl, given=True)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("grid,agrid,d", [((12, 10), (3, 5), 32), ((7, 9), (3, 3), 16)])
def test_backward_module_mode(aa, oracle, grid, agrid, d, dtype):
    _run_case(aa, oracle, _wl("module", dtype, grid, agrid, d), module=True)


@pytest.mark.parametrize("agrid,dtype,batch,heads,d", [((6, 5), "f32", 2, 1, 16), ((6, 5), "bf16", 2, 1, 16),
                                                       ((16, 16), "f16", 1, 2, 16), ((6, 5), "bf16", 2, 1, 136),
                                                       ((6, 5), "f32", 2, 1, 18), ((16, 16), "f16", 1, 1, 136)])
def test_backward_module_mode_many_tokens(aa, oracle, agrid, dtype, batch, heads, d):
    """Module terms on a 132 x 128 token grid.  16 channels: the recomputing kernels, token ranges of many columns.
    Wider than 128, or rows off the 16-byte grid: the kernels that keep the matrices in memory, where an agent's row of
    score gradients takes more than 64 KB of LDS in the kernel that sums the bias components (opt-in path), with a batch
    to add up first; with 256 agents a head's broadcast score gradients exceed the size up to which that kernel gathers
    them, so its three components take the one-pass-per-component kernels."""
    _run_case(aa, oracle, _wl("many_tokens", dtype, (132, 128), agrid, d, batch=batch, heads=heads, index=33),
              module=True, blk=(4, 3))


@pytest.mark.parametrize("grid,agrid,d,dtype,module", [((12, 10), (3, 5), 136, "bf16", True), ((7, 9), (3, 3), 160, "f16", True),
                                                       ((20, 21), (9, 10), 136, "f16", True), ((9, 70), (3, 9), 256, "bf16", False),
                                                       ((1, 1), (1, 1), 136, "f16", False)])
def test_backward_16_bit_wider_than_128(aa, oracle, grid, agrid, d, dtype, module):
    """16-bit heads that the recomputing kernels do not serve: matrix products with both attention matrices in memory,
    rows of up to and past 64 entries, with and without module terms."""
    _run_case(aa, oracle, _wl("wide", dtype, grid, agrid, d, index=35), module=module)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_backward_of_unaligned_tensors(aa, dtype):
    """Tensors one element off the 16-byte grid take the fp32 products with the matrices in memory (its workspace and the
    convolution's sums at the end of it): the gradients of the aligned call, which the tests above hold against the oracle,
    to the roundings of the two paths (16 bits: the bars of this file)."""
    import torch
    wl = _wl("unaligned", dtype, (13, 11), (4, 3), 24, index=36)
    shape = (wl.batch, wl.heads, wl.N, wl.d)
    dense = [util.to_device(inputs.make_tensor((wl.units, wl.N, wl.d), stream=960 + i, dtype=dtype), dtype, shape) for i in range(4)]
    A = util.to_device(inputs.make_tensor((wl.units, wl.n, wl.d), stream=964, dtype=dtype), dtype, (wl.batch, wl.heads, wl.n, wl.d))
    params = util.params_to_device(inputs.make_module_params(wl.heads, wl.n, wl.d, wl.grid, blk=(3, 2), index=wl.index))

    def off(t):
        v = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].reshape(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 16
        return v

    ref = aa.agent_attn_bwd(*dense, A, grid=wl.grid, params=params, v_residual_k=0.05)
    got = aa.agent_attn_bwd(*(off(t) for t in dense), A, grid=wl.grid, params=params, v_residual_k=0.05)
    assert set(got) == set(ref)
    for k in ref:
        a, b = got[k].double(), ref[k].double()
        assert bool(torch.isfinite(a).all()), k
        assert float((a - b).norm() / b.norm()) <= {"f32": 5e-6, "f16": 5e-3, "bf16": 1e-2}[dtype], k


@pytest.mark.parametrize("grid,agrid,d,dtype,blk,batch", [
    ((5, 37), (3, 4), 32, "f16", (7, 7), 2),        # more cell rows than image rows: some are never touched
    ((33, 16), (11, 12), 64, "bf16", (4, 5), 1),    # one x-tile: columns are segments; two agent blocks, the last ragged
    ((9, 70), (9, 15), 128, "bf16", (1, 3), 1),     # one cell row; odd number of x-tiles; agents past one LDS chunk
    ((40, 17), (8, 16), 40, "f16", (3, 17), 3),     # one token in the last x-tile; exactly one LDS chunk of agents
    ((4, 200), (2, 33), 16, "bf16", (3, 2), 2),     # many pairs of columns per range, one segment
    ((64, 3), (9, 3), 24, "f16", (9, 2), 1),        # three columns wide, the rest of the tile masked
    ((13, 33), (8, 8), 96, "f32", (5, 4), 1),       # fp32: exactly one LDS chunk of agents, one token column per wave
    ((21, 20), (5, 13), 128, "f32", (3, 3), 1), ((10, 47), (4, 4), 44, "f32", (2, 7), 2)])
def test_backward_agent_bias_off_the_tile_sizes(aa, oracle, grid, agrid, d, dtype, blk, batch):
    """The recomputing kernels with an agent bias walk down 16-token columns of the image: grids, cell grids and
    agent counts on and off their tiles, every gradient (bars as everywhere in this file)."""
    _run_case(aa, oracle, _wl("bias_tiles", dtype, grid, agrid, d, batch=batch, index=81), module=True, blk=blk)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_backward_block_grid_finer_than_the_image(aa, oracle, dtype):
    """Cell rows that no image row touches have gradients of exactly zero, whatever the workspace held (one image and
    one segment: the parts the kernels leave would serve as the sums)."""
    import torch
    ws = torch.full((32 << 20,), 0x41, dtype=torch.uint8, device="cuda")
    got = _run_case(aa, oracle, _wl("fine_blocks", dtype, (2, 9), (2, 3), 16, batch=1, index=21), module=True, blk=(7, 12),
                    kw={"workspace": ws})
    for g in (got["db1_blk"], got["db2_blk"].permute(0, 3, 1, 2)):
        assert bool((g[:, :, [0, 3, 6]] == 0).all())      # the image rows read cells 1, 2 and 4, 5


@pytest.mark.parametrize("keys", [("b1_col",), ("b1_row", "b2_blk"), ("b2_row", "dwc_w"), ("dwc_w",)])
def test_backward_single_module_terms(aa, oracle, keys):
    """One stage with a bias and the other without, single components, the convolution alone: the gradients against
    those of the fp32 path on the same values (itself held against the oracle above), at the bf16 bar."""
    import torch
    wl = _wl("terms", "bf16", (21, 30), (5, 6), 64, batch=2, heads=2, index=83)
    t = inputs.make_qkv(wl)
    t["dO"] = inputs.make_tensor((wl.units, wl.N, wl.d), stream=wl.index * 16 + 12, dtype=wl.dtype)
    shape = (wl.batch, wl.heads, wl.N, wl.d)
    dv = [util.to_device(t[k], wl.dtype, shape) for k in ("Q", "K", "V", "dO")]
    A = util.to_device(inputs.make_tensor((wl.units, wl.n, wl.d), stream=wl.index * 16 + 11, dtype=wl.dtype), wl.dtype,
                       (wl.batch, wl.heads, wl.n, wl.d))
    full = util.params_to_device(inputs.make_module_params(wl.heads, wl.n, wl.d, wl.grid, blk=(4, 3), index=wl.index))
    params = {k: full[k] for k in keys}
    got = aa.agent_attn_bwd(*dv, A, grid=wl.grid, params=params)
    ref = aa.agent_attn_bwd(*[x.float() for x in dv], A.float(), grid=wl.grid, params=params)
    assert set(got) == set(ref)
    for k in ref:
        a, b = got[k].double(), ref[k].double()
        assert bool(torch.isfinite(a).all()) and float((a - b).norm() / b.norm()) <= 1e-2, k


# places of a component that mask tokens of the aggregation (B1) or agents of the broadcast (B2), other tokens / agents staying
ALL = slice(None)
MASKED = {"b1_col": [(ALL, ALL, slice(0, 16)), (ALL, ALL, slice(17, None)), (ALL, 3, slice(2, 19))],
          "b1_row": [(ALL, ALL, slice(0, 3)), (ALL, ALL, slice(12, None)), (ALL, 3, slice(0, 15))],
          "b1_blk": [(ALL, ALL, 0), (ALL, ALL, ALL, 1), (ALL, 3, slice(0, 2))],
          "b2_col": [(ALL, ALL, 3), (ALL, slice(0, 3), slice(1, None)), (ALL, slice(0, 3), slice(0, -1))],
          "b2_row": [(ALL, ALL, slice(2, 5)), (ALL, slice(12, None), slice(0, 8)), (ALL, slice(12, None), slice(0, -1))],
          "b2_blk": [(ALL, ALL, ALL, 3), (ALL, 0, ALL, slice(1, None)), (ALL, 0, ALL, slice(0, -1))]}


@pytest.mark.parametrize("n,d", [(9, 32), (70, 64), (130, 32)])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("key", sorted(MASKED))
def test_masks_in_the_agent_bias(aa, oracle, key, dtype, n, d):
    """Components that mask whole rows, columns, cells or agents, in the first tiles of a walk and in later ones, with
    something left to attend to: the forward pass and every gradient at the usual bars (16 x 20 tokens, 1280 in all: the
    fp32 forward takes its streaming kernels; the 16-bit forward its small kernels, and past 64 agents its large ones with
    the block component in matrix and in table form)."""
    for place in MASKED[key]:
        for value in (-1e4, -1e9, float(np.finfo(np.float32).min), -np.inf):
            wl = _wl("mask %s %s %g" % (key, place, value), dtype, (16, 20), (1, n), d, index=85)
            _run_case(aa, oracle, wl, given=True, module=True, mask=(key, place, value, max(value, -1e9)))


# places that mask a whole softmax row: every token of an agent (B1), every agent of a token (B2)
ROWS = {"b1_col": (ALL, 3), "b1_row": (ALL, 3), "b1_blk": (ALL, 3), "b2_col": (ALL, slice(17, None)),
        "b2_row": (ALL, slice(0, 3)), "b2_blk": (ALL, 0)}


def _masked_rows(aa, oracle, key, dtype, n, d, value):
    """dQ, dK, dV, dA with the rows of ROWS[key] at `value`, the reference, dO"""
    wl = _wl("rows", dtype, (16, 20), (1, n), d, index=86)
    t = inputs.make_qkv(wl)
    t["dO"] = inputs.make_tensor((wl.units, wl.N, d), stream=wl.index * 16 + 12, dtype=dtype)
    t["A"] = inputs.make_tensor((wl.units, n, d), stream=wl.index * 16 + 11, dtype=dtype)
    dv = [util.to_device(t[k], dtype, (wl.batch, wl.heads) + t[k].shape[1:]) for k in ("Q", "K", "V", "dO", "A")]
    params = inputs.make_module_params(wl.heads, n, d, wl.grid, blk=(3, 2), index=wl.index)
    params = {k: params[k] for k in ROWS}
    params[key][ROWS[key]] = value
    got = aa.agent_attn_bwd(*dv, grid=wl.grid, params=util.params_to_device(params))
    f64 = {k: inputs.to_float64(v, dtype) for k, v in t.items()}
    B1, B2 = util.dense_biases(oracle, params, wl.heads, n, wl.grid)
    ref = oracle.agent_attn_bwd(f64["Q"], f64["K"], f64["V"], f64["dO"], A=f64["A"], heads=wl.heads, grid=wl.grid, B1=B1, B2=B2)
    return {k: util.to_host64(got[k]).reshape(ref[k].shape) for k in ("dQ", "dK", "dV", "dA")}, ref, f64["dO"]


@pytest.mark.parametrize("n,d", [(9, 32), (70, 24), (70, 64), (40, 128)])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("key", sorted(ROWS))
def test_backward_softmax_rows_masked_throughout(aa, oracle, key, dtype, n, d):
    """Rows in which every entry is masked stay softmax rows.  At -1e4 an fp32 score is a multiple of 2^-10, weights are
    good to 7e-4.  At -1e9 it is one of 64 and the weights are what the rounding leaves, but they add up to one: then
    sum_t dV = sum_a dV_A = sum_t dO, to the roundings of P1, P2, dV_A and dV (a few 2^-9, 2^-12 of dO in 16 bits)."""
    got, ref, _ = _masked_rows(aa, oracle, key, dtype, n, d, -1e4)
    for k in ref.keys() & got.keys():
        util.assert_parity(got[k], ref[k], dtype, "%s %s" % (key, k), max_abs=np.inf, rel_l2={"f32": 1e-3, "f16": 5e-3, "bf16": 1e-2}[dtype])
    got, ref, dO = _masked_rows(aa, oracle, key, dtype, n, d, -1e9)
    assert all(np.isfinite(v).all() for v in got.values())
    err = np.linalg.norm(got["dV"].sum(1) - dO.sum(1)) / np.linalg.norm(dO)
    assert err <= {"f32": 2e-6, "f16": 1e-3, "bf16": 8e-3}[dtype], err
    # at the lowest float nothing of the scores is left, in 64 bits neither: the weights are equal
    got, ref, _ = _masked_rows(aa, oracle, key, dtype, n, d, float(np.finfo(np.float32).min))
    for k in ref.keys() & got.keys():
        util.assert_parity(got[k], ref[k], dtype, "%s %s lowest" % (key, k), max_abs=np.inf, rel_l2={"f32": 1e-5, "f16": 5e-3, "bf16": 1e-2}[dtype])


@pytest.mark.parametrize("blk", [True, False])
def test_backward_f32_holds_the_weights_of_its_rows(aa, oracle, blk):
    """fp32 gradients with and without an agent bias, relative error below 6e-7 (3e-7 to 4e-7 measured): a weight taken
    from one fp32 log-sum-exp is off by up to 2^-24 of that, which made them 7e-7 to 1.1e-6 with a bias."""
    wl = _wl("f32 rows", "f32", (30, 41), (5, 7), 48, index=87)
    t = inputs.make_qkv(wl)
    t["dO"] = inputs.make_tensor((wl.units, wl.N, wl.d), stream=wl.index * 16 + 12, dtype="f32")
    t["A"] = inputs.make_tensor((wl.units, wl.n, wl.d), stream=wl.index * 16 + 11, dtype="f32")
    dv = [util.to_device(t[k], "f32", (wl.batch, wl.heads) + t[k].shape[1:]) for k in ("Q", "K", "V", "dO", "A")]
    params = inputs.make_module_params(wl.heads, wl.n, wl.d, wl.grid, blk=(3, 2), index=wl.index)
    params = {k: params[k] for k in ROWS} if blk else {}
    got = aa.agent_attn_bwd(*dv, grid=wl.grid, params=util.params_to_device(params) if blk else None)
    f64 = {k: inputs.to_float64(v, "f32") for k, v in t.items()}
    B1, B2 = util.dense_biases(oracle, params, wl.heads, wl.n, wl.grid)
    ref = oracle.agent_attn_bwd(f64["Q"], f64["K"], f64["V"], f64["dO"], A=f64["A"], heads=wl.heads, grid=wl.grid, B1=B1, B2=B2)
    for k in ("dQ", "dK", "dV", "dA"):
        util.assert_parity(util.to_host64(got[k]).reshape(ref[k].shape), ref[k], "f32", k, rel_l2=6e-7)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("only", [("ddwc_b",), ("ddwc_w",), ("db1_row", "ddwc_b")])
def test_backward_single_parameter_gradients(aa, only, offset):
    """A caller may ask for any of the parameter gradients: each has the bits it has when all are asked for, also the
    convolution's bias without its weights.  offset 1: tensors that are not 16-byte aligned, the path that keeps the
    matrices in memory."""
    import ctypes
    import torch
    wl = _wl("single", "f32", (9, 10), (3, 2), 12, index=88)
    params = util.params_to_device(inputs.make_module_params(wl.heads, wl.n, wl.d, wl.grid, blk=(3, 2), index=wl.index))
    count = wl.units * wl.N * wl.d

    def placed(i):
        t = torch.zeros(count + 4, device="cuda")
        v = t[offset:offset + count].reshape(wl.batch, wl.heads, wl.N, wl.d)
        v.copy_(util.to_device(inputs.make_tensor((wl.units, wl.N, wl.d), stream=950 + i), "f32", v.shape))
        return v

    q, k, v, dO = (placed(i) for i in range(4))
    A = util.to_device(inputs.make_tensor((wl.units, wl.n, wl.d), stream=954), "f32", (wl.batch, wl.heads, wl.n, wl.d))
    full = aa.agent_attn_bwd(q, k, v, dO, A, grid=wl.grid, params=params)
    desc, p = aa.make_desc(wl.batch, wl.heads, wl.N, wl.n, wl.d, 0, wl.grid), aa.make_params(params)
    ws = torch.empty(int(aa.lib().agent_attn_bwd_workspace_bytes(ctypes.byref(desc), aa._pp(p))), dtype=torch.uint8, device="cuda")
    outs = [torch.empty_like(full[x]) for x in ("dQ", "dK", "dV", "dA")]
    grads, g = {x: torch.full_like(full[x], float("nan")) for x in only}, aa.aa_param_grads()
    for x, t in grads.items():
        setattr(g, x, t.data_ptr())
    st = aa.lib().agent_attn_bwd(ctypes.byref(desc), q.data_ptr(), k.data_ptr(), v.data_ptr(), A.data_ptr(), aa._pp(p), dO.data_ptr(),
                                 ws.data_ptr(), ws.numel(), *(t.data_ptr() for t in outs), ctypes.byref(g), None)
    torch.cuda.synchronize()
    assert st == 0
    for x, t in grads.items():
        assert torch.equal(t, full[x]), x


def test_backward_of_a_unit_past_2_30_elements(aa):
    """A pure 16-bit unit of 2^24 + 77 tokens, 64 channels: every gradient against plain fp32 products (bf16 bar of this file)."""
    import torch
    N, n, d = (1 << 24) + 77, 4, 64
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v, g = (torch.randn(N, d, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(4))
    a = torch.randn(n, d, generator=gen, device="cuda", dtype=torch.bfloat16)
    got = aa.agent_attn_bwd(*(x[None, None] for x in (q, k, v, g)), a[None, None])
    c, A = d ** -0.5, a.float()
    P1 = torch.softmax(c * (A @ k.float().t()), 1)
    VA = P1 @ v.float()
    P2 = torch.softmax(c * (q.float() @ A.t()), 1)
    dVA = P2.t() @ g.float()
    dP2 = g.float() @ VA.t()
    dS2 = P2 * (dP2 - (P2 * dP2).sum(1, keepdim=True))
    dP1 = dVA @ v.float().t()
    dS1 = P1 * (dP1 - (P1 * dP1).sum(1, keepdim=True))
    ref = {"dQ": c * (dS2 @ A), "dK": c * (dS1.t() @ A), "dV": P1.t() @ dVA, "dA": c * (dS2.t() @ q.float() + dS1 @ k.float())}
    for name, r in ref.items():
        x = got[name][0, 0].float()
        assert bool(torch.isfinite(x).all()), name
        for part in (slice(0, None), slice(-1000, None)):      # all, and the end by itself
            err = float((x[part] - r[part]).norm() / r[part].norm())
            assert err <= 1e-2, (name, err)


def test_backward_module_given_agents_and_residual(aa, oracle):
    wl = _wl("module-given", "f32", (8, 8), (2, 8), 24)
    _run_case(aa, oracle, wl, given=True, module=True, kw=dict(v_residual_k=0.075, scale2=24 ** -0.15))


def test_backward_deit_shape(aa, oracle):
    """The DeiT-T shape of the benchmark, two batch elements."""
    wl = dataclasses.replace(WL["deit_t"], batch=2)
    _run_case(aa, oracle, wl)


@pytest.mark.parametrize("name,batch,heads", [("swin_t_s1", 1, 3), ("sd_latent", 1, 2), ("highres", 1, 1)])
def test_backward_workload_shapes(aa, oracle, name, batch, heads):
    """The other benchmark shapes at their real N, n and d (fewer units, so that the oracle's dense n x N matrices
    stay within seconds): every gradient element against the oracle."""
    wl = dataclasses.replace(WL[name], batch=batch, heads=heads)
    _run_case(aa, oracle, wl)


@pytest.mark.parametrize("grid,agrid,d,dtype,given", [((40, 37), (15, 10), 64, "bf16", False),
                                                      ((33, 31), (13, 21), 128, "f16", True),
                                                      ((50, 41), (9, 15), 40, "bf16", True),
                                                      ((26, 20), (14, 19), 104, "f16", False),
                                                      ((64, 48), (3, 2), 16, "bf16", False)])
def test_backward_many_agents_ragged(aa, oracle, grid, agrid, d, dtype, given):
    """Pure 16-bit problems off every tile size of the recomputing kernels: agent counts past one LDS chunk
    (128) with a ragged last chunk and a ragged last block of agents, token counts that end inside a tile
    and are cut into several ranges, head widths 16 .. 128, pooled (ragged windows) and given agents."""
    _run_case(aa, oracle, _wl("ragged", dtype, grid, agrid, d, batch=1, heads=2, index=29), given=given)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("scale_qk,given", [(4.0, True), (4.0, False), (8.0, True)])
def test_backward_peaky_softmaxes(aa, oracle, scale_qk, given, dtype):
    """Q and K four and eight times larger: both softmaxes close to one-hot, weights spread over many orders of
    magnitude, score gradients dominated by a few pairs.  Same bars."""
    _run_case(aa, oracle, _wl("peaky", dtype, (20, 18), (6, 5), 32, batch=1, heads=2, index=37), given=given,
              scale_qk=scale_qk)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("n,d,units,dwc", [(49, 64, 2, False), (63, 32, 1, True), (17, 128, 1, False), (64, 48, 1, False),
                                           (131, 16, 520, False)])
def test_backward_scores_far_below_zero(aa, oracle, n, d, units, dwc, dtype):
    """A token whose scores all lie near -128: exp(-log-sum-exp) overflows, which the rows that fill the last tile of
    agents must not see (agent counts off the tile of 32; the last case has units enough for the kernel with four token
    columns per wave).  Channel 0 holds the common part of agents and token: there dQ is the sum of the token's score
    gradients, zero but for their roundings, times 16, and dA takes 8 times the error of one token's score gradients
    where other channels take an average over tokens, so these two are asked to be finite only; the bars elsewhere as
    usual."""
    wl = _wl("far_below", dtype, (5, 8), (1, n), d, batch=1, heads=units, index=61)
    t = inputs.make_qkv(wl)
    t["dO"] = inputs.make_tensor((units, wl.N, d), stream=wl.index * 16 + 12, dtype=dtype)
    t["A"] = inputs.make_tensor((units, n, d), stream=wl.index * 16 + 11, dtype=dtype)
    f64 = {k: inputs.to_float64(v, dtype).copy() for k, v in t.items()}
    f64["A"][:, :, 0] = 16.0
    f64["Q"][:, :, 0] = 0.0
    f64["Q"][:, 3, 0] = -8.0 * d ** 0.5
    dv = [util.to_device(inputs.to_storage(f64[k], dtype), dtype, (1, units) + f64[k].shape[1:]) for k in ("Q", "K", "V", "dO", "A")]
    f64 = {k: util.to_host64(x).reshape(f64[k].shape) for k, x in zip(("Q", "K", "V", "dO", "A"), dv)}      # as rounded
    w = np.zeros((units, d, 3, 3), np.float32)
    kw = dict(grid=wl.grid, params={"dwc_w": util.params_to_device({"w": w})["w"]}) if dwc else {}
    got = aa.agent_attn_bwd(*dv, **kw)
    ref = oracle.agent_attn_bwd(f64["Q"], f64["K"], f64["V"], f64["dO"], A=f64["A"], heads=units, grid=wl.grid)
    for k in ("dQ", "dK", "dV", "dA"):
        x = util.to_host64(got[k]).reshape(ref[k].shape)
        assert np.isfinite(x).all(), k
        first = 1 if k in ("dQ", "dA") else 0
        _check(got[k][..., first:], ref[k][..., first:], dtype, k)


@pytest.mark.parametrize("grid,agrid,d,masked", [((12, 12), (4, 4), 32, None), ((40, 40), (12, 12), 64, None),
                                                  ((21, 18), (5, 4), 32, False), ((21, 18), (5, 4), 32, True)])
def test_backward_is_deterministic_and_ignores_workspace(aa, grid, agrid, d, masked):
    """masked: None: no module terms; True: a token and an agent masked throughout in one of the heads, so that the blocks of
    its units are told by their flags to take the form for large references"""
    import torch
    wl = _wl("det", "bf16", grid, agrid, d)
    params = None
    if masked is not None:
        params = inputs.make_module_params(wl.heads, wl.n, d, grid, blk=(3, 2), index=wl.index)
        if masked:
            params["b1_row"][1, 2] = params["b2_row"][1, 3] = -1e9
        params = util.params_to_device(params)
    kw = dict(grid=wl.grid, agent_grid=wl.agent_grid, params=params)
    t = inputs.make_qkv(wl)
    shape = (wl.batch, wl.heads, wl.N, wl.d)
    dv = {k: util.to_device(v, wl.dtype, shape) for k, v in t.items()}
    dO = util.to_device(inputs.make_tensor((wl.units, wl.N, wl.d), stream=300, dtype=wl.dtype), wl.dtype, shape)
    a = aa.agent_attn_bwd(dv["Q"], dv["K"], dv["V"], dO, **kw)
    desc = aa.make_desc(wl.batch, wl.heads, wl.N, wl.n, wl.d, 2, wl.grid, wl.agent_grid)
    import ctypes
    need = int(aa.lib().agent_attn_bwd_workspace_bytes(ctypes.byref(desc), aa._pp(aa.make_params(params))))
    for fill in (0xFF, 0x41):
        ws = torch.full((need,), fill, dtype=torch.uint8, device="cuda")
        b = aa.agent_attn_bwd(dv["Q"], dv["K"], dv["V"], dO, workspace=ws, **kw)
        for k in a:
            assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("dtype,d", [("f32", 24), ("bf16", 32), ("f32", 21), ("bf16", 20), ("f16", 136)])
def test_backward_windows_in_descriptor(aa, dtype, d):
    """Windows named in the descriptor (Sec. 5.5): the gradients of the image tensors are, bit for bit, those
    of the same windows handed over as a batch (a case the tests above hold against the oracle).  The first two widths are
    read in place, the others staged through window-major copies."""
    import torch
    batch, heads, image, window, agrid = 2, 2, (12, 18), (6, 6), (3, 3)
    (Y, X), (wh, ww) = image, window
    nwin = (Y // wh) * (X // ww)
    params = util.params_to_device(inputs.make_module_params(heads, 9, d, window, blk=(3, 2), index=21))

    def part(x):      # [B,H,Y*X,d] -> [B*windows,H,wh*ww,d]
        v = x.reshape(batch, heads, Y // wh, wh, X // ww, ww, d)
        return v.permute(0, 2, 4, 1, 3, 5, 6).reshape(batch * nwin, heads, wh * ww, d).contiguous()

    def unpart(x):
        v = x.reshape(batch, Y // wh, X // ww, heads, wh, ww, d)
        return v.permute(0, 3, 1, 4, 2, 5, 6).reshape(batch, heads, Y * X, d).contiguous()

    img = [util.to_device(inputs.make_tensor((batch * heads, Y * X, d), stream=700 + i, dtype=dtype), dtype,
                          (batch, heads, Y * X, d)) for i in range(4)]
    a = aa.agent_attn_bwd(*img, grid=image, window=window, agent_grid=agrid, params=params, v_residual_k=0.05)
    b = aa.agent_attn_bwd(*[part(x) for x in img], grid=window, agent_grid=agrid, params=params, v_residual_k=0.05)
    for k in ("dQ", "dK", "dV"):
        assert torch.equal(a[k], unpart(b[k])), k
    for k in a:
        if k not in ("dQ", "dK", "dV"):
            assert torch.equal(a[k], b[k]), k
    assert float(a["dQ"].float().abs().max()) > 0


@pytest.mark.parametrize("seed", range(36))
def test_backward_random_problems(aa, oracle, seed):
    """Seeded random shapes: both product paths (fp32 vector and MFMA, with padded score rows and ragged
    tiles), pooled and given agents, with and without the module terms and the SD-variant scalars."""
    rng = np.random.default_rng(500 + seed)
    dtype = ["f32", "f16", "bf16"][seed % 3]
    module = bool(rng.random() < 0.5)
    gh, gw = int(rng.integers(1, 25)), int(rng.integers(1, 25))
    if module and dtype != "f32":
        # a parameter gradient sums one term per token; the rounding of the 16-bit MFMA operands (relative
        # to the size of P * dP, not of the much smaller dS) only averages out over enough of them
        gh, gw = max(gh, 8), max(gw, 8)
    ah, aw = int(rng.integers(1, min(gh, 10) + 1)), int(rng.integers(1, min(gw, 10) + 1))
    d = int(rng.integers(1, 70)) if (dtype == "f32" and seed % 2) else int(rng.choice([8, 16, 24, 32, 40, 64, 72, 128]))
    wl = _wl("random%d" % seed, dtype, (gh, gw), (ah, aw), d, batch=int(rng.integers(1, 3)),
             heads=int(rng.integers(1, 4)), index=40 + seed)
    kw = dict(v_residual_k=0.075, scale2=float(d) ** -0.15) if rng.random() < 0.3 else None
    _run_case(aa, oracle, wl, given=bool(rng.random() < 0.3), module=module,
              blk=(int(rng.integers(1, 6)), int(rng.integers(1, 6))), kw=kw)


@pytest.mark.parametrize("module,d", [(False, 32), (True, 32), (True, 136)])
def test_backward_replayed_from_a_graph(aa, module, d):
    """The backward pass allocates nothing and clears nothing with memsets: captured once, every replay gives the
    bits of the eager call on the inputs of the moment (the recomputing kernels, pure and with module terms; wider than
    128 the kernels that keep the matrices in memory; with their parameter gradients)."""
    import ctypes
    import torch
    wl = _wl("graph", "bf16", (24, 20), (6, 5), d, batch=2, heads=2, index=41)
    shape = (wl.batch, wl.heads, wl.N, wl.d)
    t = [util.to_device(inputs.make_tensor((wl.units, wl.N, wl.d), stream=900 + i, dtype=wl.dtype), wl.dtype, shape)
         for i in range(4)]
    params = util.params_to_device(inputs.make_module_params(wl.heads, wl.n, wl.d, wl.grid, blk=(3, 2), index=wl.index)) \
        if module else None
    kw = dict(grid=wl.grid, agent_grid=wl.agent_grid, params=params)
    desc = aa.make_desc(wl.batch, wl.heads, wl.N, wl.n, wl.d, 2, wl.grid, wl.agent_grid)
    need = int(aa.lib().agent_attn_bwd_workspace_bytes(ctypes.byref(desc), aa._pp(aa.make_params(params))))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        aa.agent_attn_bwd(*t, workspace=ws, stream=side, **kw)      # first call outside the capture (one-time set-up)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            got = aa.agent_attn_bwd(*t, workspace=ws, stream=side, **kw)
    torch.cuda.synchronize()
    for rep in range(3):
        for x in t:
            x.copy_(torch.roll(x, shifts=rep + 1, dims=2))
        ws.fill_(rep)
        for v in got.values():
            v.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        eager = aa.agent_attn_bwd(*t, **kw)
        for k in eager:
            assert torch.equal(got[k], eager[k]), "replay %d: %s differs from the eager call" % (rep, k)


@pytest.mark.parametrize("dtype,d", [("f32", 20), ("bf16", 32), ("f32", 21), ("f16", 20), ("bf16", 136)])
@pytest.mark.parametrize("layout", ["token_major", "fused_qkv"])
def test_backward_strided_layouts(aa, dtype, d, layout):
    """Token-major [B,N,H,d] tensors and the q / k / v slices of a fused projection [B,N,3,H,d]: read in place (the first
    two widths) or staged through dense copies, every gradient has the bits of the dense call and lands with the strides
    of its tensor."""
    import torch
    wl = _wl("strided", dtype, (9, 8), (3, 4), d, batch=2, heads=3, index=71)
    t = inputs.make_qkv(wl)
    dO = inputs.make_tensor((wl.units, wl.N, wl.d), stream=wl.index * 16 + 12, dtype=wl.dtype)
    shape = (wl.batch, wl.heads, wl.N, wl.d)
    dense = {k: util.to_device(v, wl.dtype, shape) for k, v in t.items()}
    dense["dO"] = util.to_device(dO, wl.dtype, shape)
    params = util.params_to_device(inputs.make_module_params(wl.heads, wl.n, wl.d, wl.grid, blk=(3, 2), index=wl.index))
    kw = dict(grid=wl.grid, agent_grid=wl.agent_grid, params=params)
    ref = aa.agent_attn_bwd(dense["Q"], dense["K"], dense["V"], dense["dO"], **kw)
    if layout == "token_major":
        view = {k: v.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for k, v in dense.items()}
    else:
        fused = torch.stack([dense[k].permute(0, 2, 1, 3) for k in ("Q", "K", "V")], dim=2).contiguous()   # [B,N,3,H,d]
        view = {k: fused[:, :, i].permute(0, 2, 1, 3) for i, k in enumerate(("Q", "K", "V"))}
        view["dO"] = dense["dO"].permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    assert not view["Q"].is_contiguous()
    got = aa.agent_attn_bwd(view["Q"], view["K"], view["V"], view["dO"], **kw)
    for k in ("dQ", "dK", "dV"):
        assert got[k].stride() == view["Q"].stride()
        assert torch.equal(got[k], ref[k]), k
    for k in ref:
        if k not in ("dQ", "dK", "dV"):
            assert torch.equal(got[k], ref[k]), k

