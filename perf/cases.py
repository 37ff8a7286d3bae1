"""Timed cases of the SDP path: what a training program has this library do, through its public entry points.

A case is one pass of one of these kinds:

  mlp     one step of the neuron-masked SwiGLU MLP for K workers back to back: mask -> index compaction, every worker's
          forward and backward with its weight gradients scattered into that worker's full-size buffer, and the
          coverage-normalised average of the K buffers
  attn    one worker's head-masked attention block, forward and backward
  block   a stack of residual blocks under block-level masking, forward through all and backward through all
  avg     the coverage-normalised average of K gradient buffers, alone
  update  gradient clipping and AdamW from the K buffers: squared norms, clipping coefficient, fused average + update

Index tables, weights, outputs and workspaces are made once, in prepare(), as a training loop keeps them from step to
step; the values are those of the seeded workloads (X, dY ~ N(0, 1), weights ~ N(0, 0.02^2), gradients ~ N(0, 1e-3^2)).
"""
import torch

import paper_2507_09029_amd as sdp

_DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # The small fp32 workload of the benchmark (correctness runs, unit-sized models): four workers of 256 tokens,
        # where the time is launches and latency.
        dict(name="mlp_f32_small", kind="mlp", dtype="f32", mode="fm", T=256, d=256, F=1024, p=512, K=4),
        # An fp32 residual block of modest width: the full-precision run a bf16 one is compared with.
        dict(name="block_f32", kind="block", dtype="f32", mode="fm", bits="1", Bt=2, S=256, d=512, H=8, hd=64, F=1376),
        # A small bf16 MLP at the paper's smallest width (hidden 768): short micro-batches, a few dozen tiles a launch.
        dict(name="mlp_bf16_small", kind="mlp", dtype="bf16", mode="fm", T=1024, d=768, F=2048, p=1024, K=2),
        # The benchmark's 500M-like width, forward masking at C = 0.5.
        dict(name="mlp_bf16_fm_500M", kind="mlp", dtype="bf16", mode="fm", T=8192, d=1536, F=4096, p=2048, K=4),
        # The paper's 1B width (hidden 1600) with a coverage and a micro-batch that fit no tile: p and T are odd
        # multiples of 8, as p = round(C F) and packed batches give them.
        dict(name="mlp_bf16_ragged", kind="mlp", dtype="bf16", mode="fm", T=5000, d=1600, F=4264, p=2664, K=2),
        # The benchmark's headline: 1B-like width, backward masking, eight workers.
        dict(name="mlp_bf16_bm_1B", kind="mlp", dtype="bf16", mode="bm", T=16384, d=2048, F=5504, p=4128, K=8),
        # The benchmark's head-masked attention block: heads of 64, half of them held.
        dict(name="attn_bf16_500M", kind="attn", dtype="bf16", mode="fm", Bt=4, S=2048, d=1536, H=24, hd=64, ph=12),
        # The same under backward masking at the paper's own 500M width: heads of 50.
        dict(name="attn_bf16_paper_width", kind="attn", dtype="bf16", mode="bm", Bt=4, S=2048, d=1200, H=24, hd=50, ph=12),
        # Heads of 128, the widest the block takes and a common choice, on one sequence of a length that fits no tile.
        dict(name="attn_bf16_hd128", kind="attn", dtype="bf16", mode="fm", Bt=1, S=1500, d=1024, H=8, hd=128, ph=4),
        # Block-level masking: a running block and one that is left out of the backward pass except for the gradient
        # that flows through it, at the paper's 500M width and sequence length.
        dict(name="block_bf16", kind="block", dtype="bf16", mode="bm", bits="10", Bt=4, S=1024, d=1200, H=24, hd=50, F=3200),
        # The average alone over one billion parameters: eight bf16 buffers, coverage 0.69.
        dict(name="avg_1B", kind="avg", dtype="bf16", K=8, R=488282, D=2048, p=336915),
        # The optimizer step of twelve MLP layers of the 500M-like width, clipped at 1.0, with bf16 weights for the next
        # forward pass.
        dict(name="update_500M", kind="update", dtype="bf16", K=8, R=147456, D=1536, p=101745),
    ]


def _log_int(rng, lo, hi, step=1):
    """An integer in [lo, hi], a multiple of `step`, spread evenly over the logarithm of the range."""
    v = lo * (hi / lo) ** rng.random()
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["mlp", "mlp", "mlp", "attn", "attn", "attn", "block", "avg", "update"])
    if kind == "mlp":
        f32 = rng.random() < 0.25
        step = 1 if f32 else 8
        T = _log_int(rng, 64, 1024, step) if f32 else _log_int(rng, 128, 16384, step)
        d = _log_int(rng, 64, 512, step) if f32 else _log_int(rng, 256, 2048, step)
        F = _log_int(rng, 128, 2048, step) if f32 else _log_int(rng, 512, 5504, step)
        K = rng.choice([2, 4, 8])
        cover = rng.uniform(max(0.375, 1.0 / K), 0.875)
        p = min(F, -(-int(round(cover * F)) // step) * step)
        return dict(kind="mlp", dtype="f32" if f32 else "bf16", mode=rng.choice(["fm", "bm"]), T=T, d=d, F=F, p=p, K=K)
    if kind == "attn":
        f32 = rng.random() < 0.15
        hd = rng.choice([32, 50, 64, 64, 80, 96, 128])
        H = rng.randint(2, max(2, (512 if f32 else 2048) // hd))
        Bt = rng.randint(1, 2 if f32 else 4)
        S = _log_int(rng, 32, 256 if f32 else 2048)
        ph = rng.randint((H + 1) // 2, H)
        d = max(64, -(-H * hd // 8) * 8)
        return dict(kind="attn", dtype="f32" if f32 else "bf16", mode=rng.choice(["fm", "bm"]), Bt=Bt, S=S, d=d, H=H, hd=hd, ph=ph)
    if kind == "block":
        f32 = rng.random() < 0.25
        hd = rng.choice([50, 64, 64, 128])
        H = rng.randint(2, max(2, (512 if f32 else 1600) // hd))
        d = -(-H * hd // 8) * 8
        F = max(128, int(d * rng.uniform(2.0, 4.0)) // 8 * 8)
        Bt = rng.randint(1, 2 if f32 else 4)
        S = _log_int(rng, 64, 256 if f32 else 1024, 1 if f32 else 8)
        mode = rng.choice(["fm", "bm"])
        return dict(kind="block", dtype="f32" if f32 else "bf16", mode=mode, bits=rng.choice(["1", "10", "01", "11"]), Bt=Bt, S=S,
                    d=d, H=H, hd=hd, F=F)
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    K = rng.choice([2, 4, 8, 12])
    D = _log_int(rng, 64, 4096, rng.choice([1, 8, 8, 8]))
    most = (4 << 30 if kind == "avg" else 2 << 30) // ((2 if dtype == "bf16" else 4) * K * D)  # bytes of all K buffers
    R = _log_int(rng, 500, max(501, min(488282, most)))
    p = max(1, int(round(rng.uniform(0.4, 0.9) * R)))
    return dict(kind=kind, dtype=dtype, K=K, R=R, D=D, p=p)


class _Draw:
    """Normal tensors on the GPU from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(1_000_003 * seed + 17)

    def __call__(self, shape, std, dtype):
        return (torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32) * std).to(dtype)


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _prepare_mlp(c, seed):
    dt, rnd = _DT[c["dtype"]], _Draw(seed)
    T, d, F, p, K, mode = c["T"], c["d"], c["F"], c["p"], c["K"], c["mode"]
    n = p if mode == "fm" else F
    mask, idx, pos, cov = sdp.make_masks(K, F, p, seed, True)
    s = dict(kind="mlp", mode=mode, K=K, F=F, mask=mask, W=[rnd((F, d), 0.02, dt) for _ in range(3)],
             X=[rnd((T, d), 1.0, dt) for _ in range(K)], dY=[rnd((T, d), 1.0, dt) for _ in range(K)],
             index=(idx, pos, _empty((K,), torch.int32), cov), p=p,
             G=_empty((T, n), dt), U=_empty((T, n), dt), Y=[_empty((T, d), dt) for _ in range(K)],
             dX=[_empty((T, d), dt) for _ in range(K)],
             # rows off a worker's mask are never written nor read
             grads=[torch.zeros((3 * F, d), dtype=dt, device="cuda") for _ in range(K)],
             mask3=mask.repeat(1, 3).contiguous(), avg=_empty((3 * F, d), torch.float32), cov3=_empty((3 * F,), torch.uint8),
             wsf=_bytes(sdp.masked_mlp_fwd_workspace_bytes(mode, dt, T, d, F, p)),
             wsb=_bytes(sdp.masked_mlp_bwd_workspace_bytes(mode, dt, T, d, F, p)))
    return s


def _run_mlp(s):
    F = s["F"]
    idx, pos, count, cov = sdp.index_masks_static(s["mask"], idx_ld=s["p"], out=s["index"])
    for k in range(s["K"]):
        Y, G, U = sdp.masked_mlp_fwd(s["mode"], s["X"][k], *s["W"], idx[k], out=(s["Y"][k], s["G"], s["U"]), ws=s["wsf"])
        g = s["grads"][k]
        sdp.masked_mlp_bwd(s["mode"], s["X"][k], s["dY"][k], *s["W"], idx[k], G, U, dw_layout="scatter",
                           out=(s["dX"][k], g[:F], g[F:2 * F], g[2 * F:]), ws=s["wsb"])
    sdp.coverage_grad_avg(s["grads"], s["mask3"], out=s["avg"], cov=s["cov3"])
    return dict(idx=idx, pos=pos, count=count, cov=cov, Y=s["Y"], dX=s["dX"], grads=s["grads"], avg=s["avg"], cov3=s["cov3"])


def _prepare_attn(c, seed):
    dt, rnd = _DT[c["dtype"]], _Draw(seed)
    Bt, S, d, H, hd, ph, mode = (c[k] for k in ("Bt", "S", "d", "H", "hd", "ph", "mode"))
    T, n, hw = Bt * S, ph if mode == "fm" else H, sdp.attn_saved_head_width(dt, hd)
    idx = sdp.make_masks(2, H, ph, seed, True)[1][0].contiguous()
    return dict(kind="attn", mode=mode, Bt=Bt, S=S, hd=hd, idx=idx, X=rnd((T, d), 1.0, dt), dY=rnd((T, d), 1.0, dt),
                Wqkv=rnd((3, H * hd, d), 0.02, dt), WoT=rnd((H * hd, d), 0.02, dt),
                fwd=(_empty((T, d), dt), _empty((T, 3 * n * hw), dt), _empty((T, n * hw), dt), _empty((Bt, n, S), torch.float32)),
                bwd=(_empty((T, d), dt), _empty((3, ph * hd, d), dt), _empty((ph * hd, d), dt)),
                wsf=_bytes(sdp.masked_attn_fwd_workspace_bytes(mode, dt, Bt, S, d, H, hd, ph)),
                wsb=_bytes(sdp.masked_attn_bwd_workspace_bytes(mode, dt, Bt, S, d, H, hd, ph)))


def _run_attn(s):
    a = (s["mode"], s["Bt"], s["S"], s["hd"])
    Y, QKV, O, LSE = sdp.masked_attn_fwd(*a, s["X"], s["Wqkv"], s["WoT"], s["idx"], out=s["fwd"], ws=s["wsf"])
    dX, dWqkv, dWoT = sdp.masked_attn_bwd(*a, s["X"], s["dY"], s["Wqkv"], s["WoT"], s["idx"], QKV, O, LSE, out=s["bwd"], ws=s["wsb"])
    return dict(Y=Y, LSE=LSE, dX=dX, dWqkv=dWqkv, dWoT=dWoT)


def _prepare_block(c, seed):
    dt, rnd = _DT[c["dtype"]], _Draw(seed)
    Bt, S, d, H, hd, F, mode = (c[k] for k in ("Bt", "S", "d", "H", "hd", "F", "mode"))
    T, E = Bt * S, H * hd
    Es = H * sdp.attn_saved_head_width(dt, hd)
    blocks = []
    for b in c["bits"]:
        m = int(b)
        runs = m or mode == "bm"
        shapes = ((3, E, d), (E, d), (F, d), (F, d), (F, d))  # Wqkv, WoT, W1, W3, W2T
        blocks.append(dict(
            m=m, W=[rnd(x, 0.02, dt) for x in shapes],
            fwd=(_empty((T, d), dt), _empty((T, d), dt), _empty((T, 3 * Es), dt), _empty((T, Es), dt),
                 _empty((Bt, H, S), torch.float32), _empty((T, F), dt), _empty((T, F), dt)) if runs else _empty((T, d), dt),
            bwd=(_empty((T, d), dt),) + (tuple(_empty(x, dt) for x in shapes) if m else ())))
    return dict(kind="block", mode=mode, Bt=Bt, S=S, hd=hd, X=rnd((T, d), 1.0, dt), dY=rnd((T, d), 1.0, dt), blocks=blocks,
                wsf=_bytes(sdp.block_fwd_workspace_bytes(dt, Bt, S, d, H, hd, F)),
                wsb=_bytes(sdp.block_bwd_workspace_bytes(dt, Bt, S, d, H, hd, F)))


def _run_block(s):
    a = (s["Bt"], s["S"], s["hd"])
    x, inputs, saved = s["X"], [], []
    for b in s["blocks"]:
        inputs.append(x)
        x, keep = sdp.block_fwd(s["mode"], b["m"], *a, x, *b["W"], out=b["fwd"], ws=s["wsf"])
        saved.append(keep)
    dy, grads = s["dY"], []
    for b, xin, keep in zip(reversed(s["blocks"]), reversed(inputs), reversed(saved)):
        dy, g = sdp.block_bwd(s["mode"], b["m"], *a, xin, dy, *b["W"], keep, dx_rule="through", out=b["bwd"], ws=s["wsb"])
        if g is not None:
            grads.append(g)
    return dict(Y=x, dX=dy, grads=grads)


def _gradients(c, rnd):
    dt = _DT[c["dtype"]]
    return [rnd((c["R"], c["D"]), 1e-3, dt) for _ in range(c["K"])]


def _prepare_avg(c, seed):
    mask = sdp.sample_masks_host(c["K"], c["R"], c["p"], seed, False).cuda()
    return dict(kind="avg", grads=_gradients(c, _Draw(seed)), mask=mask, out=_empty((c["R"], c["D"]), torch.float32),
                cov=_empty((c["R"],), torch.uint8))


def _run_avg(s):
    out, cov = sdp.coverage_grad_avg(s["grads"], s["mask"], out=s["out"], cov=s["cov"])
    return dict(avg=out, cov=cov)


def _prepare_update(c, seed):
    rnd = _Draw(seed)
    shape = (c["R"], c["D"])
    theta = rnd(shape, 0.02, torch.float32)
    return dict(kind="update", grads=_gradients(c, rnd), mask=sdp.sample_masks_host(c["K"], c["R"], c["p"], seed, False).cuda(),
                theta=theta, m=rnd(shape, 3e-4, torch.float32), v=rnd(shape, 6e-4, torch.float32).square_(),
                low=theta.to(torch.bfloat16), cov=_empty((c["R"],), torch.uint8), sq=_empty((1,), torch.float64),
                scale=_empty((1,), torch.float32), ws=_bytes(int(sdp.lib().sdp_coverage_grad_sqnorm_workspace_bytes(*shape))))


def _run_update(s):
    sdp.coverage_grad_sqnorm(s["grads"], s["mask"], out=s["sq"], ws=s["ws"])
    sdp.clip_scale(s["sq"], 1.0, out=s["scale"])
    sdp.coverage_avg_adamw(s["grads"], s["mask"], s["theta"], s["m"], s["v"], lr=1e-3, beta1=0.9, beta2=0.95, eps=1e-8,
                           weight_decay=0.1, step=100, theta_bf16=s["low"], cov=s["cov"], grad_scale_dev=s["scale"])
    return dict(sq=s["sq"], scale=s["scale"], theta=s["theta"], m=s["m"], v=s["v"], low=s["low"], cov=s["cov"])


def prepare(case, seed):
    return {"mlp": _prepare_mlp, "attn": _prepare_attn, "block": _prepare_block, "avg": _prepare_avg,
            "update": _prepare_update}[case["kind"]](case, seed)


def run(state):
    return {"mlp": _run_mlp, "attn": _run_attn, "block": _run_block, "avg": _run_avg, "update": _run_update}[state["kind"]](state)


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "mlp":
        T, d, F, p, K = c["T"], c["d"], c["F"], c["p"], c["K"]
        flops = K * (18 * T * d * p if c["mode"] == "fm" else 12 * T * d * F + 6 * T * d * p)
        # X, dY, Y, dX per worker, the weights, the covered gradient rows, the average and the integer tables
        nbytes = K * 4 * T * d * e + 3 * F * d * e + K * 3 * p * d * e + 3 * F * d * 4 + K * (F + 4 * p + 4 * F) + F
        return {"bytes": nbytes, "flops": flops}
    if c["kind"] == "attn":
        T, d, E_all, Eh = c["Bt"] * c["S"], c["d"], c["H"] * c["hd"], c["ph"] * c["hd"]
        E = Eh if c["mode"] == "fm" else E_all
        flops = 16 * T * d * E + 8 * T * d * Eh + 7 * c["Bt"] * E * c["S"] ** 2
        return {"bytes": (4 * T * d + 4 * E * d + 4 * Eh * d) * e + T * E // c["hd"] * 4, "flops": flops}
    if c["kind"] == "block":
        T, d, E, F = c["Bt"] * c["S"], c["d"], c["H"] * c["hd"], c["F"]
        flops = nbytes = 0
        for b in c["bits"]:
            runs, dw = b == "1" or c["mode"] == "bm", b == "1"
            params = (4 * E + 3 * F) * d
            nbytes += (4 * T * d + (params if runs else 0) + (params if dw else 0)) * e
            if runs:
                flops += (4 + (2 if dw else 0)) * T * params + 7 * c["Bt"] * E * c["S"] ** 2
        return {"bytes": nbytes, "flops": flops}
    K, R, D, p = c["K"], c["R"], c["D"], c["p"]
    grads = K * p * D * e + K * R
    if c["kind"] == "avg":
        return {"bytes": grads + R * D * 4 + R, "flops": K * p * D + R * D}
    # the norm has to be known before the first parameter moves: the gradients are read twice
    return {"bytes": 2 * grads + R * D * (24 + 2) + R, "flops": 2 * K * p * D + 16 * R * D}


def tolerance(case):
    # About four times what the path shows against itself at fp32 on the same inputs (bf16 cases: 2.3e-3 .. 3.4e-3 over
    # the MLP's and the attention block's outputs, up to 4.8e-3 over a block's, which chain two halves) and against fp64
    # torch (fp32 MLP: 7e-7; the average's order of summation is part of its interface).
    if case["dtype"] == "bf16" and case["kind"] in ("mlp", "attn", "block"):
        return {"rel": 1.8e-2 if case["kind"] == "block" else 1.2e-2}
    if case["kind"] == "update":
        # theta and its moments agree to 32-bit rounding; a bf16 copy that sits on a rounding boundary may go either way
        return {"rel": 1e-4, "max": 1e-2}
    if case["kind"] == "avg":
        return {"rel": 1e-6}
    return {"rel": 1e-5}
