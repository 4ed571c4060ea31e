"""Performance cases of the agent-attention library: the calls that programs using it make.

Three kinds of call, all through paper_2312_08874_amd.binding:

  forward   inference with the operator alone: a call prepared once on fixed buffers (prepare_fwd), or agent_attn_fwd
            when the attention runs inside windows
  module    inference with the projections around the operator (agent_attn_module_fwd)
  train     a training step of the operator: agent_attn_fwd, then agent_attn_bwd for an upstream gradient; returns the
            output and every gradient

A case is a flat dict: kind; batch, heads, the token grid, head width d and agent grid; the window (0 x 0: the whole
grid); dtype ("f32", "f16", "bf16"); terms ("none": the pure operator, "module": agent bias with a 7 x 7 block component
and the depthwise convolution, "residual": the Stable-Diffusion variant, k = 0.075 and an enlarged second scale);
tables (True: agent-bias tables built ahead, as inference with fixed parameters does); layout of the token tensors
("dense" [B,H,N,d], "token" [B,N,H,d], "qkv": slices of a fused projection [B,N,3,H,d] with a token-major gradient).
"""
import math

import torch

from paper_2312_08874_amd import binding, inputs

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BLOCK = (7, 7)
RESIDUAL_K = 0.075


def _case(name, kind, batch, heads, grid, d, agents, dtype, terms, *, window=(0, 0), tables=False, layout="dense"):
    c = {"kind": kind, "batch": batch, "heads": heads, "grid_h": grid[0], "grid_w": grid[1], "d": d,
         "agent_h": agents[0], "agent_w": agents[1], "window_h": window[0], "window_w": window[1], "dtype": dtype,
         "terms": terms, "tables": tables, "layout": layout}
    return dict(name=name, **c) if name else c


def _workload(name, kind, workload, terms, **kw):
    w = inputs.WORKLOADS[workload]
    return _case(name, kind, w.batch, w.heads, w.grid, w.d, w.agent_grid, w.dtype, terms, **kw)


def listed():
    return [
        # one small image, one head, fp32: nothing but latency
        _workload("tiny_f32", "forward", "tiny", "none"),
        # a block of a small vision transformer at 224 x 224 pixels, inference on a batch
        _workload("deit_t", "forward", "deit_t", "none"),
        # the high-resolution first stage of a hierarchical backbone, inference with its fixed bias parameters
        _workload("swin_t_s1_tables", "forward", "swin_t_s1", "module", tables=True),
        # self-attention of a latent-diffusion model at 512 x 512 pixels, training-free variant, one guided sample
        _workload("sd_latent_residual", "forward", "sd_latent", "residual"),
        # one image of 128 x 128 tokens with 1024 agents: the largest forward problem
        _workload("highres", "forward", "highres", "none"),
        # the same image through the whole module: projections, agent bias, convolution
        _workload("highres_projected", "module", "highres", "module"),
        # the module inside 28 x 28 windows of the first-stage image (the window-size ablation)
        _workload("swin_windows_projected", "module", "swin_t_s1", "module", window=(28, 28)),
        # training steps with every module term: the small transformer block ...
        _workload("deit_t_train", "train", "deit_t", "module"),
        # ... the first stage, reading q, k, v where a fused projection wrote them ...
        _workload("swin_t_s1_train", "train", "swin_t_s1", "module", layout="qkv"),
        # ... and fine-tuning at high resolution
        _workload("highres_train", "train", "highres", "module"),
        # fine-tuning the pure operator on an image whose sides divide by nothing
        _case("ragged_train_f16", "train", 2, 5, (37, 59), 64, (11, 17), "f16", "none"),
        # training in fp32 on another such image
        _case("ragged_train_f32", "train", 8, 6, (31, 43), 48, (7, 9), "f32", "module"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more problem of the ranges the listed ones span: sides 7 .. 128 tokens, agents up to a quarter of the
    tokens and 32 a side, widths 16 .. 128, 1 .. 192 units, no more work than the largest listed problem (fp32: than
    about twice the fp32 training step, its arithmetic rate being so much lower)."""
    kind = rng.choice(("forward", "forward", "train", "train", "module"))
    dtype = rng.choice(("bf16", "bf16", "f16", "f16", "f32"))
    pairs, rows = (4.5e8, 3e7) if dtype == "f32" else (8 * 1024 * 16384 * 64, 3.3e7)
    while True:
        d = rng.choice((16, 24, 32, 32, 40, 48, 64, 64, 80, 96, 128))
        batch, heads = _log_int(rng, 1, 64), rng.choice((1, 2, 3, 3, 4, 5, 6, 8, 8))
        grid = (_log_int(rng, 7, 128), _log_int(rng, 7, 128))
        window = (0, 0)
        if kind != "train" and rng.random() < 0.25:
            window = (_log_int(rng, 7, 28), _log_int(rng, 7, 28))
            grid = (window[0] * rng.randint(1, 4), window[1] * rng.randint(1, 4))
        inner = window if window[0] else grid
        agents = tuple(_log_int(rng, 3, max(3, min(32, s // 2))) for s in inner)
        tokens, n = grid[0] * grid[1], agents[0] * agents[1]
        if batch * heads > 192 or 8 * max(inner) < max(grid) or max(inner) > 8 * min(inner):
            continue
        if batch * heads * tokens * n * d > pairs or batch * heads * tokens * d > rows:
            continue
        if kind == "module" and batch * tokens * 4 * (heads * d) ** 2 > 2e10:
            continue
        break
    terms = rng.choice(("none", "module", "module", "residual"))
    tables = kind == "forward" and terms == "module" and not window[0] and dtype != "f32" and rng.random() < 0.5
    layout = rng.choice(("dense", "token", "qkv")) if kind != "module" else "dense"
    return _case(None, kind, batch, heads, grid, d, agents, dtype, terms, window=window, tables=tables, layout=layout)


def _token_tensors(case, gen, dtype, count):
    """`count` tensors of standard normal values shaped [B,H,T,d] in the case's layout."""
    B, H, T, d = case["batch"], case["heads"], case["grid_h"] * case["grid_w"], case["d"]

    def rnd(*shape):
        return torch.randn(*shape, generator=gen, device="cuda").to(dtype)

    if case["layout"] == "dense":
        return [rnd(B, H, T, d) for _ in range(count)]
    if case["layout"] == "token":
        return [rnd(B, T, H, d).permute(0, 2, 1, 3) for _ in range(count)]
    fused = rnd(B, T, 3, H, d)
    return [fused[:, :, i].permute(0, 2, 1, 3) for i in range(3)] + \
        [rnd(B, T, H, d).permute(0, 2, 1, 3) for _ in range(count - 3)]


def _module_params(case, gen):
    H, d, n = case["heads"], case["d"], case["agent_h"] * case["agent_w"]
    h, w = (case["window_h"], case["window_w"]) if case["window_h"] else (case["grid_h"], case["grid_w"])

    def rnd(std, *shape):
        return std * torch.randn(*shape, generator=gen, device="cuda")

    return {"b1_col": rnd(0.5, H, n, w), "b1_row": rnd(0.5, H, n, h), "b1_blk": rnd(0.5, H, n, *BLOCK),
            "b2_col": rnd(0.5, H, w, n), "b2_row": rnd(0.5, H, h, n), "b2_blk": rnd(0.5, H, *BLOCK, n),
            "dwc_w": (2 * torch.rand(H, d, 3, 3, generator=gen, device="cuda") - 1) / 3, "dwc_b": rnd(0.1, H, d)}


def prepare(case, seed):
    """Inputs and parameters on the GPU, the buffers of an inference loop, its prepared call."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype = DTYPES[case["dtype"]]
    H, d, grid = case["heads"], case["d"], (case["grid_h"], case["grid_w"])
    kw = {"grid": grid, "agent_grid": (case["agent_h"], case["agent_w"])}
    if case["window_h"]:
        kw["window"] = (case["window_h"], case["window_w"])
    if case["terms"] == "module":
        kw["params"] = _module_params(case, gen)
    elif case["terms"] == "residual":
        kw.update(v_residual_k=RESIDUAL_K, scale2=float(d) ** -0.15)
    if case["tables"]:
        kw["params"]["bias_tables"] = binding.agent_attn_bias_tables(
            kw["params"], heads=H, N=grid[0] * grid[1], n=case["agent_h"] * case["agent_w"], d=d, dtype=dtype, grid=grid)
    state = {"case": case, "kw": kw}
    if case["kind"] == "module":
        C = H * d

        def rnd(std, *shape):
            return (std * torch.randn(*shape, generator=gen, device="cuda")).to(dtype)

        x = rnd(1.0, case["batch"], grid[0] * grid[1], C)
        weights = (rnd(C ** -0.5, 3 * C, C), rnd(0.1, 3 * C), rnd(C ** -0.5, C, C), rnd(0.1, C))
        state.update(args=(x,) + weights, out=torch.empty_like(x))
    else:
        state["args"] = _token_tensors(case, gen, dtype, 4 if case["kind"] == "train" else 3)
        if case["kind"] == "forward":
            state["out"] = torch.empty_like(state["args"][0])
            if not case["window_h"]:
                state["call"] = binding.prepare_fwd(*state["args"], out=state["out"], **kw)
    return state


def run(state):
    kind, kw = state["case"]["kind"], state["kw"]
    if kind == "module":
        return binding.agent_attn_module_fwd(*state["args"], heads=state["case"]["heads"], out=state["out"], **kw)
    if kind == "forward":
        if "call" in state:
            state["call"]()
            return state["out"]
        return binding.agent_attn_fwd(*state["args"], out=state["out"], **kw)
    q, k, v, grad = state["args"]
    return {"out": binding.agent_attn_fwd(q, k, v, **kw), **binding.agent_attn_bwd(q, k, v, grad, **kw)}


def work(case):
    """Two n x N products each for aggregation and broadcast (8 N n d), five more for each in the backward pass
    (20 N n d), 8 T C^2 for the projections; every token tensor and parameter moved once."""
    es = 4 if case["dtype"] == "f32" else 2
    B, H, d, T = case["batch"], case["heads"], case["d"], case["grid_h"] * case["grid_w"]
    n, C = case["agent_h"] * case["agent_w"], case["heads"] * case["d"]
    pairs = B * H * T * n * d
    flops = (28 if case["kind"] == "train" else 8) * pairs
    count = {"forward": 4, "module": 2, "train": 8}[case["kind"]]
    nbytes = count * B * T * C * es
    if case["kind"] == "module":
        flops += 8 * B * T * C * C
        nbytes += 4 * C * (C + 1) * es
    if case["terms"] == "module":
        h, w = (case["window_h"], case["window_w"]) if case["window_h"] else (case["grid_h"], case["grid_w"])
        param = 4 * (2 * H * n * (h + w + BLOCK[0] * BLOCK[1]) + 10 * C)
        nbytes += (2 if case["kind"] == "train" else 1) * param
        flops += (54 if case["kind"] == "train" else 18) * B * T * C
    return {"bytes": nbytes, "flops": flops}


# Relative error allowed, about four times what comparing every kind of call with itself in 64 bits showed: a single
# pass rounds its output and the probabilities once (1.7e-3 in bf16, 2.1e-4 in fp16); the projections add a rounding of
# q, k, v and of the attention's output (4.1e-3, 5.5e-4); a gradient chains three rounded operands (4.2e-3, with the
# enlarged second scale up to 7e-3; 5e-4).  fp32: sums in another order (2e-7; gradients, differences of larger
# terms, 1.5e-6).
RELATIVE = {"forward": {"bf16": 7e-3, "f16": 9e-4, "f32": 1e-6},
            "module": {"bf16": 1.6e-2, "f16": 2.2e-3, "f32": 2e-6},
            "train": {"bf16": 2e-2, "f16": 2.5e-3, "f32": 1e-5}}


def tolerance(case):
    return {"rel": RELATIVE[case["kind"]][case["dtype"]]}
