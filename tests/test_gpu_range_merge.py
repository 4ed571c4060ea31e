"""Merge of the aggregation's token ranges (fp32 forward in several launches): values at the ends of the type's range, in the last
range, which stands in for the ranges that a trip of eight asks for past the last one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def aa():
    from paper_2312_08874_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("grid,agrid,d", [((17, 20), (4, 8), 64), ((40, 33), (8, 8), 128), ((16, 16), (7, 9), 40), ((56, 56), (7, 7), 32)])
@pytest.mark.parametrize("value", [float("inf"), float("-inf")])
def test_an_infinite_value_stays_infinite(aa, grid, agrid, d, value):
    """Every weight is positive: an infinite value of the last token makes its channel of its unit infinite, and nothing else changes."""
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(1, 2, grid[0] * grid[1], d, generator=gen, device="cuda") for _ in range(3))
    clean = aa.agent_attn_fwd(q, k, v, grid=grid, agent_grid=agrid)
    v[0, 1, -1, 5] = value
    out = aa.agent_attn_fwd(q, k, v, grid=grid, agent_grid=agrid)
    assert (out[0, 1, :, 5] == value).all()
    rest = [c for c in range(d) if c != 5]
    assert torch.equal(out[0, 0], clean[0, 0]) and torch.equal(out[0, 1][:, rest], clean[0, 1][:, rest])


@pytest.mark.parametrize("value", [4e35, -8e35])
def test_sums_of_the_ranges_that_pass_the_type_do_not(aa, value):
    """3136 equal scores: the sum over a range of at most 400 tokens fits fp32, over all of them it does not.  Their mean is the value
    itself, to a rounding (2^-24) for each term of a range and a few more."""
    q = torch.zeros(1, 64, 3136, 32, device="cuda")
    v = torch.full_like(q, value)
    out = aa.agent_attn_fwd(q, q, v, grid=(56, 56), agent_grid=(7, 7)).double()
    assert (out / value - 1).abs().max() <= 400 * 2.0 ** -24
