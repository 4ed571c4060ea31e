"""agent_attn_fwd_static: the forward pass on the library's own static workspace (for callers that cannot
allocate) must give the bits of agent_attn_fwd, on consecutive calls that share the array, the second one
on a smaller problem."""
import dataclasses

import pytest

from paper_2312_08874_amd import inputs
from tests import util

pytestmark = pytest.mark.gpu

WL = inputs.WORKLOADS

# (first problem, second and smaller problem): split small-agent path, large-agent path, reference path
PAIRS = [
    ("split", dataclasses.replace(WL["swin_t_s1"], batch=2), dataclasses.replace(WL["swin_t_s1"], batch=1, grid=(40, 40))),
    ("large", dataclasses.replace(WL["sd_latent"], batch=1), dataclasses.replace(WL["sd_latent"], batch=1, heads=3,
                                                                                 grid=(24, 32), agent_grid=(9, 9))),
    ("reference", dataclasses.replace(WL["tiny"], batch=2, heads=2, grid=(30, 30)), WL["tiny"]),
]


def _dev(wl):
    t = inputs.make_qkv(wl)
    return {k: util.to_device(v, wl.dtype, (wl.batch, wl.heads, wl.N, wl.d)) for k, v in t.items()}


@pytest.mark.parametrize("name,first,second", PAIRS, ids=[p[0] for p in PAIRS])
@pytest.mark.parametrize("module", [False, True])
def test_static_workspace_matches_caller_workspace(name, first, second, module):
    import torch
    from paper_2312_08874_amd import binding as aa
    aa.lib()
    assert aa.static_scratch_bytes() == 64 << 20
    outs = []
    for wl in (first, second):          # two calls in a row on the shared array, the second one smaller
        dv = _dev(wl)
        params = util.params_to_device(inputs.make_module_params(wl.heads, wl.n, wl.d, wl.grid, index=wl.index)) \
            if module else None
        kw = dict(grid=wl.grid, agent_grid=wl.agent_grid, params=params)
        out = torch.full_like(dv["Q"], 3.0)
        aa.agent_attn_fwd_static(dv["Q"], dv["K"], dv["V"], out=out, **kw)
        outs.append((out, dv, kw))
    torch.cuda.synchronize()
    for out, dv, kw in outs:
        ref = aa.agent_attn_fwd(dv["Q"], dv["K"], dv["V"], **kw)
        assert bool(torch.isfinite(out.float()).all())
        assert torch.equal(out, ref)


@pytest.mark.parametrize("dtype,d,grid,agrid", [("bf16", 64, (128, 128), (28, 28)), ("f16", 40, (96, 128), (30, 30))])
def test_static_workspace_takes_the_tables_of_the_biases_in_turn(dtype, d, grid, agrid):
    """Many agents, whose tables do not fit the array at once."""
    import torch
    from paper_2312_08874_amd import binding as aa
    wl = dataclasses.replace(WL["tiny"], batch=1, heads=8, grid=grid, agent_grid=agrid, d=d, dtype=dtype, index=26)
    dv = _dev(wl)
    host = inputs.make_module_params(wl.heads, wl.n, d, grid, blk=(7, 7), index=26)
    params = util.params_to_device(host)
    desc = aa.make_desc(1, wl.heads, wl.N, wl.n, d, aa._dtype_code(dv["Q"]), grid, agrid)
    assert aa.workspace_bytes(desc, aa.make_params(params)) > aa.static_scratch_bytes()
    kw = dict(grid=grid, agent_grid=agrid, params=params)
    ref = aa.agent_attn_fwd(dv["Q"], dv["K"], dv["V"], **kw)
    out = torch.full_like(dv["Q"], 3.0)
    for _ in range(2):
        aa.agent_attn_fwd_static(dv["Q"], dv["K"], dv["V"], out=out, **kw)
        assert torch.equal(out, ref)


def test_static_workspace_rejects_oversized_problems():
    import torch
    from paper_2312_08874_amd import binding as aa
    wl = dataclasses.replace(WL["highres"], batch=16)      # V_A and the pooled agents alone exceed 64 MiB
    desc = aa.make_desc(wl.batch, wl.heads, wl.N, wl.n, wl.d, aa.AA_BF16, wl.grid, wl.agent_grid)
    assert aa.workspace_bytes(desc) > aa.static_scratch_bytes()
    fake = torch.empty(16, dtype=torch.bfloat16, device="cuda")
    st = aa.lib().agent_attn_fwd_static(__import__("ctypes").byref(desc), fake.data_ptr(), fake.data_ptr(),
                                        fake.data_ptr(), None, None, fake.data_ptr(), None)
    assert st == -5      # AA_ERR_WORKSPACE, decided on the host before any launch
