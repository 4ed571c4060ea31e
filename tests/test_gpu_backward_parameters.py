"""Parameter gradients of the backward pass at the sizes where their kernels branch: batches shared out over the waves of a
block (eight images and more: groups of two, of whole eights with a remainder, an odd last one), image columns of one, two and
three rows and one and two columns (the convolution's window reaches past the image on both sides), every number of 16-byte
pieces per token, an infinity beside the image border, cell rows of the bias tables in runs.  Reference and bars as in test_gpu_backward."""
import pytest
import torch

from .test_gpu_backward import _run_case, _wl, aa  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("batch", [7, 8, 9, 21, 35, 64])
def test_backward_module_batches(aa, oracle, batch, dtype):  # noqa: F811
    _run_case(aa, oracle, _wl("batch %d" % batch, dtype, (9, 11), (3, 3), 32, batch=batch, heads=1, index=41), module=True)


@pytest.mark.parametrize("dtype,d", [("f16", 8), ("bf16", 24), ("f16", 40), ("bf16", 80), ("f32", 12), ("f32", 128)])
@pytest.mark.parametrize("grid,agrid", [((1, 9), (1, 3)), ((2, 5), (1, 2)), ((3, 2), (1, 1)), ((11, 1), (3, 1)), ((13, 17), (2, 3))])
def test_backward_convolution_edges(aa, oracle, grid, agrid, dtype, d):  # noqa: F811
    _run_case(aa, oracle, _wl("dwc %s" % (grid,), dtype, grid, agrid, d, batch=3, heads=3, index=42), module=True)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("blk", [(7, 7), (5, 3), (1, 9)])
def test_backward_tables_in_runs_of_cell_rows(aa, oracle, blk, dtype):  # noqa: F811
    """Enough columns of tables that a block makes three or two cell rows, with a remainder, and one."""
    _run_case(aa, oracle, _wl("runs %s" % (blk,), dtype, (28, 100), (8, 12), 16, batch=1, heads=40, index=43), module=True, blk=blk)


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 32), (torch.float32, 20)])
@pytest.mark.parametrize("corner", [(0, 0), (0, -1), (-1, 0), (-1, -1)])
def test_backward_convolution_infinite_corner(aa, corner, dtype, d):  # noqa: F811
    """An infinity in a corner pixel of V reaches the four taps that meet the pixel inside the image and no other."""
    h, w = 10, 13
    gen = torch.Generator(device="cuda").manual_seed(44)
    q, k, v, g = (torch.randn(2, 2, h * w, d, generator=gen, device="cuda").to(dtype) for _ in range(4))
    params = {"dwc_w": torch.randn(2, d, 3, 3, generator=gen, device="cuda"), "dwc_b": torch.zeros(2, d, device="cuda")}
    grads = []
    for value in (0.0, float("inf")):
        v.view(2, 2, h, w, d)[0, 1, corner[0], corner[1], 3] = value
        grads.append(aa.agent_attn_bwd(q, k, v, g, grid=(h, w), agent_grid=(3, 4), params=params)["ddwc_w"])
    met = torch.zeros(2, d, 3, 3, dtype=torch.bool, device="cuda")      # tap (ky, kx) meets pixel (0, 0) from (1 - ky, 1 - kx)
    met[1, 3, (slice(0, 2) if corner[0] == 0 else slice(1, 3)), (slice(0, 2) if corner[1] == 0 else slice(1, 3))] = True
    assert torch.isinf(grads[1][met]).all()
    assert torch.equal(grads[1][~met], grads[0][~met])
