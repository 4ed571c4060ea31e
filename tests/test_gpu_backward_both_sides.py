"""Backward of units with at most 64 agents, whose agent kernels take the tokens' gradients as well, at the sizes where they
branch: agents at and beside the 16 of a wave and the 32 of a product step, tokens that end inside a tile of 32 or a column of
16, channels beside the padded width, one range and many (more than eight are added up first), given agents, the residual and the
convolution.  Reference and bars as in test_gpu_backward."""
import pytest

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
