"""Timed cases of the contrastive loss: what a training or evaluation program asks of it.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges,
``prepare`` makes one case's inputs on the GPU, ``run`` is one pass through the
public entry points, ``exact`` the same outputs in plain fp64 torch.

Kinds of call (a case's "kind"):
  autograd  clip_loss(img, txt, scale) and its gradients, in the inputs' type:
            the training step of a program that leaves the buffers to torch
  step      clip_loss_fwd + clip_loss_bwd with fp32 gradients and one workspace
            kept by the caller: the step of a program that manages its buffers
            (and the form that the benchmark times)
  fwd       clip_loss_fwd with a kept workspace: the loss of a held-out set
  noalloc   infcl_fwd_noalloc into kept outputs: the same for callers that
            cannot allocate
  shards    sharded_forward_backward: every GPU's share of a sharded batch,
            one after another on one device

Embeddings are unit rows, the text a noisy copy of its image: sigma sets the
positive cosine 1 / sqrt(1 + sigma^2).  scale 14.29 with sigma 1 is the start
of training, 50 with sigma 3 and 100 with sigma 4 its later stages (positives
at cosine 0.32 and 0.24, loss well above zero).
"""

import math

import torch

import paper_2410_17243_amd as infcl
from paper_2410_17243_amd.shards import sharded_forward_backward

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
STAGES = [(14.29, 1.0), (50.0, 3.0), (100.0, 4.0)]  # (scale, sigma)


def _case(kind, b, d, dtype, scale=14.29, sigma=1.0, shards=0):
    return {"kind": kind, "b": b, "d": d, "dtype": dtype, "scale": scale, "sigma": sigma, "shards": shards}


def listed():
    return [
        # one micro-batch of a small fine-tuning run: launches and host time
        dict(_case("autograd", 256, 512, "bf16"), name="autograd_b256_d512_bf16"),
        # the small fp32 workload of the benchmark (number 1)
        dict(_case("step", 1024, 512, "f32", scale=1.0 / 0.07), name="step_b1024_d512_f32"),
        # mixed-precision (fp16) training on one GPU at an ordinary batch
        dict(_case("autograd", 4096, 768, "f16", scale=100.0, sigma=4.0), name="autograd_b4096_d768_f16"),
        # held-out loss of a 5000-pair retrieval set, without allocation
        dict(_case("noalloc", 5000, 512, "bf16", scale=50.0, sigma=3.0), name="noalloc_b5000_d512_bf16"),
        # a projection width between the kernels' widths, ragged batch
        dict(_case("step", 6001, 200, "bf16"), name="step_b6001_d200_bf16"),
        # ragged batch at a width of several passes
        dict(_case("autograd", 10007, 640, "bf16"), name="autograd_b10007_d640_bf16"),
        # full-precision training of a small model
        dict(_case("step", 8192, 256, "f32"), name="step_b8192_d256_f32"),
        # the widest embedding at the batch of one large GPU
        dict(_case("autograd", 16384, 1024, "bf16", scale=50.0, sigma=3.0), name="autograd_b16384_d1024_bf16"),
        # benchmark workload 2
        dict(_case("step", 32768, 512, "bf16"), name="step_b32768_d512_bf16"),
        # the same batch as the shares of 8 GPUs
        dict(_case("shards", 32768, 512, "bf16", shards=8), name="shards8_b32768_d512_bf16"),
        # held-out loss of a large set
        dict(_case("fwd", 50000, 768, "f16", scale=100.0, sigma=4.0), name="fwd_b50000_d768_f16"),
        # the shape of benchmark workload 3, at a trained model's similarities
        dict(_case("step", 131072, 768, "bf16", scale=100.0, sigma=4.0), name="step_b131072_d768_bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["autograd", "autograd", "step", "step", "fwd", "noalloc", "shards"])
    dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
    f32 = dtype == "f32"
    if kind == "shards" or rng.random() < 0.7:  # a width the kernels are built for
        d = rng.randrange(1, 9) * (64 if f32 else 128)
        padded = False
    else:
        d = rng.randrange(16, 129) * (4 if f32 else 8)
        padded = True
    if kind == "shards":
        b = _log_int(rng, 2048, 8192 if f32 else 32768)
    elif kind == "noalloc":  # within the fixed scratch
        b = _log_int(rng, 200, 2000 if padded else 16384)
    else:
        b = _log_int(rng, 200, 16384 if f32 else 65536)
    scale, sigma = rng.choice(STAGES) if d >= 512 else STAGES[0]
    return _case(kind, b, d, dtype, scale, sigma, rng.choice([2, 4, 8]) if kind == "shards" else 0)


def _inputs(case, seed):
    b, d, sigma = case["b"], case["d"], case["sigma"]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    g = torch.randn(b, d, device="cuda", generator=gen)
    n = torch.randn(b, d, device="cuda", generator=gen)
    dt = DTYPES[case["dtype"]]
    img = torch.nn.functional.normalize(g, dim=1).to(dt)
    txt = torch.nn.functional.normalize(g + sigma * n, dim=1).to(dt)
    return img, txt, torch.tensor([case["scale"]], dtype=torch.float32, device="cuda")


def prepare(case, seed):
    img, txt, scale = _inputs(case, seed)
    st = {"kind": case["kind"], "shards": case["shards"], "img": img, "txt": txt, "scale": scale}
    if case["kind"] == "autograd":
        for k in ("img", "txt", "scale"):
            st[k].requires_grad_()
    elif case["kind"] in ("step", "fwd"):
        st["ws"] = infcl.workspace_for(img)
    elif case["kind"] == "noalloc":
        b = case["b"]
        st["out"] = {"loss": torch.empty((), dtype=torch.float32, device="cuda"),
                     "loss64": torch.empty((), dtype=torch.float64, device="cuda"),
                     "lse_r": torch.empty(b, dtype=torch.float32, device="cuda"),
                     "lse_c": torch.empty(b, dtype=torch.float32, device="cuda"),
                     "aux": torch.empty(3 * b, dtype=torch.float32, device="cuda")}
    else:
        st["ws"] = [infcl.workspace_for(img) for _ in range(case["shards"])]
    return st


def run(state):
    img, txt, scale = state["img"], state["txt"], state["scale"]
    kind = state["kind"]
    if kind == "autograd":
        loss = infcl.clip_loss(img, txt, scale)
        dimg, dtxt, dscale = torch.autograd.grad(loss, (img, txt, scale))
        return {"loss": loss.detach(), "dimg": dimg, "dtxt": dtxt, "dscale": dscale}
    if kind == "noalloc":
        o = state["out"]
        infcl.infcl_fwd_noalloc(img, txt, scale, o["loss"], o["loss64"], o["lse_r"], o["lse_c"], o["aux"])
        return dict(o)
    if kind == "shards":
        o = sharded_forward_backward(img, txt, scale, state["shards"], workspaces=state["ws"])
        return {"loss": o["loss64"], "lse_r": o["lse_r"], "lse_c": o["lse_c"], "aux": o["aux"], "dimg": o["dimg"],
                "dtxt": o["dtxt"], "dscale": o["dscale64"]}
    f = infcl.clip_loss_fwd(img, txt, scale, workspace=state["ws"])
    out = {k: f[k] for k in ("loss", "loss64", "lse_r", "lse_c", "aux")}
    if kind == "step":
        out["dimg"], out["dtxt"], out["dscale"] = infcl.clip_loss_bwd(img, txt, scale, f, workspace=state["ws"])
    return out


def work(case):
    """Inputs read once, outputs written once; 2 b^2 d flops for the forward's
    similarities, and 6 b^2 d for the backward (the similarities again and the
    two gradients; a shard also needs its columns' similarities: 8 b^2 d)."""
    b, d, kind = case["b"], case["d"], case["kind"]
    es = 4 if case["dtype"] == "f32" else 2
    nbytes = 2 * b * d * es + 4
    flops = 2 * b * b * d
    if kind == "autograd":
        return {"bytes": nbytes + 2 * b * d * es + 8, "flops": flops + 6 * b * b * d}
    nbytes += 5 * b * 4 + 12
    if kind in ("step", "shards"):
        nbytes += 2 * b * d * 4 + 4
        flops += (8 if kind == "shards" else 6) * b * b * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # fp32: sums in another order; 16-bit: the gradient weights (and autograd's
    # gradients) round to the input type; the per-sample terms carry the
    # similarities' fp32 rounding times the scale
    return {"rel": {"f32": 2e-5, "bf16": 1e-2, "f16": 1.5e-3}[case["dtype"]]}


def exact(case, seed):
    b, kind = case["b"], case["kind"]
    img, txt, scale = _inputs(case, seed)
    img, txt = img.double(), txt.double()
    s = float(scale.double().item())
    rows = max(1, min(b, (1 << 28) // b))
    u = (img * txt).sum(1)
    r = torch.empty(b, dtype=torch.float64, device="cuda")
    m = torch.full((b,), -math.inf, dtype=torch.float64, device="cuda")  # column maxima and sums
    l = torch.zeros(b, dtype=torch.float64, device="cuda")
    txt_t = txt.t().contiguous()
    for i in range(0, b, rows):
        x = torch.mm(img[i:i + rows], txt_t).mul_(s)
        r[i:i + rows] = torch.logsumexp(x, 1)
        m2 = torch.maximum(m, x.amax(0))
        l = l * torch.exp(m - m2) + x.sub_(m2).exp_().sum(0)
        m = m2
    c = m + torch.log(l)
    aux = torch.cat([r - s * u, c - s * u, u])
    loss = ((r - s * u).sum() + (c - s * u).sum()) / (2 * b)
    out = {"loss": loss, "lse_r": r, "lse_c": c, "aux": aux}
    if kind in ("fwd", "noalloc"):
        return dict(out, loss64=loss)
    dimg = torch.empty_like(img)
    dtxt = torch.zeros_like(txt)
    ds = torch.zeros((), dtype=torch.float64, device="cuda")
    for i in range(0, b, rows):
        x = torch.mm(img[i:i + rows], txt_t)
        g = x.mul(s).sub_(r[i:i + rows, None]).exp_()
        g += x.mul(s).sub_(c).exp_()
        k = torch.arange(g.shape[0], device="cuda")
        g[k, i + k] -= 2.0
        g /= 2 * b
        ds += (g * x).sum()
        dimg[i:i + rows] = torch.mm(g, txt).mul_(s)
        dtxt += torch.mm(g.t().contiguous(), img[i:i + rows])
    dtxt *= s
    ds = ds.reshape(1) if kind == "autograd" else ds
    if kind == "autograd":
        return {"loss": loss, "dimg": dimg, "dtxt": dtxt, "dscale": ds}
    out.update(dimg=dimg, dtxt=dtxt, dscale=ds)
    return dict(out, loss64=loss) if kind == "step" else out
