"""What a workspace serves.

A program keeps one workspace, sized for its largest batch, and runs smaller
ones with it: every call accepts what infcl_workspace_size gives for a larger
batch of the same width and type, also where the smaller batch would split
its row blocks into more partial sums than that workspace holds (it then
splits into fewer).  The forward results do not depend on the workspace's
size; the gradients are sums of the same terms in another order."""

import pytest

import paper_2410_17243_amd as infcl

SHAPES = [(512, 0), (768, 0), (1024, 2), (128, 2), (200, 0), (512, 1), (256, 1), (64, 1), (100, 1)]


def _size(b, d, dt):
    return infcl.infcl_workspace_size(b, d, dt)


@pytest.mark.parametrize("d,dt", SHAPES)
def test_workspace_of_a_larger_batch_is_accepted(d, dt):
    import torch

    if torch.cuda.is_available():
        pytest.skip("made-up addresses: only where nothing can be launched")
    lib, A = infcl.load_library(), 1 << 20
    batches = [1, 31, 33, 256, 1000, 2000, 4097, 8192, 16420, 32768, 32769, 40000, 50000, 65536, 98304, 131072, 140001,
               209716, 262145, 1 << 20]
    for i, b in enumerate(batches):
        for big in batches[i:]:
            n = _size(big, d, dt)
            f = lib.infcl_fwd(A, A, b, d, dt, A, A, A, A, A, A, A, n, None)
            g = lib.infcl_bwd(A, A, b, d, dt, A, A, A, A, None, A, A, 1, A, A, n, None)
            s = lib.infcl_bwd_shard(A, A, b, d, dt, 0, (b + 7) // 8, A, A, A, A, None, A, A, 1, A, A, n, None)
            # accepted: the launch is what fails here
            assert f == g == s == infcl.INFCL_ERR_HIP, (b, big, f, g, s)


@pytest.mark.parametrize("d,dt", SHAPES)
def test_refused_workspace(d, dt):
    """The vectors, padded copies and padded gradients are needed in any case."""
    lib, A = infcl.load_library(), 1 << 20
    for b in (32, 1000, 32768, 131072):
        for n in (0, 256, 8 * b - 8):
            assert lib.infcl_fwd(A, A, b, d, dt, A, A, A, A, A, A, A, n, None) == infcl.INFCL_ERR_WORKSPACE
            assert lib.infcl_bwd(A, A, b, d, dt, A, A, A, A, None, A, A, 1, A, A, n, None) == infcl.INFCL_ERR_WORKSPACE


@pytest.mark.parametrize("d,dt,limit", [(128, 0, 99776), (512, 0, 99776), (1024, 2, 99768), (200, 0, 9844),
                                        (1000, 0, 2676), (64, 1, 43002), (512, 1, 43002), (100, 1, 11863)])
def test_noalloc_limit(d, dt, limit):
    """Which batches the fixed scratch takes is part of the interface, whatever
    infcl_workspace_size includes for the backward."""
    import torch

    if torch.cuda.is_available():
        pytest.skip("made-up addresses: only where nothing can be launched")
    lib, A = infcl.load_library(), 1 << 20
    for b in (1, 1000, limit // 2, limit, limit + 1, limit + 300, 2 * limit):
        st = lib.infcl_fwd_noalloc(A, A, b, d, dt, A, A, A, A, A, A, None)
        assert st == (infcl.INFCL_ERR_HIP if b <= limit else infcl.INFCL_ERR_WORKSPACE), b
    dk = -(-d // (64 if dt == 1 else 128)) * (64 if dt == 1 else 128)
    per = (780 if dt == 1 else 336) + (0 if dk == d else (16 if dt == 1 else 12) * dk)
    # (a batch of fewer than 32 row blocks leaves fewer pairs: up to 88 of the 336 bytes)
    assert limit == pytest.approx((32 << 20) / per, rel=1e-2)


@pytest.mark.gpu
@pytest.mark.parametrize("b,big,d,dtype", [(2000, 65536, 768, "bf16"), (1000, 1100, 512, "f16"),
                                            (3001, 40000, 200, "bf16"), (1500, 33000, 256, "f32"),
                                            (4100, 131072, 1024, "bf16")])
def test_smaller_batch_in_a_kept_workspace(b, big, d, dtype):
    import torch

    from gpu_util import device_inputs, f32_scale, max_rel, synth

    img, txt = device_inputs(*synth.clip_pairs(b, d, 1.0, seed=b + d, dtype=dtype), dtype)
    sc = torch.tensor([f32_scale(14.29)], dtype=torch.float32, device="cuda")
    n = _size(big, d, infcl._dtype_code(img))
    guard = 1 << 20
    buf = torch.full((n + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    ref = infcl.clip_loss_fwd(img, txt, sc)
    ref_g = infcl.clip_loss_bwd(img, txt, sc, ref)
    got = infcl.clip_loss_fwd(img, txt, sc, workspace=buf[:n])
    got_g = infcl.clip_loss_bwd(img, txt, sc, got)
    torch.cuda.synchronize()
    for k in ("loss64", "lse_r", "lse_c", "aux"):
        assert torch.equal(ref[k], got[k]), k
    errs = [max_rel(o.double().cpu().numpy(), r.double().cpu().numpy()) for o, r in zip(got_g, ref_g)]
    print(f"b={b} workspace of {big} ({n} bytes against {_size(b, d, infcl._dtype_code(img))}) d={d} {dtype}: {errs}",
          flush=True)
    # G' is formed alike; its fp32 sums of up to b terms are taken in another order
    assert max(errs) <= 1e-5
    assert bool((buf[n:] == 0xA5).all())


@pytest.mark.gpu
@pytest.mark.parametrize("b,n,d,dtype", [(33000, 8, 256, "bf16"), (34001, 16, 640, "f16")])
def test_shards_above_the_split_batch(b, n, d, dtype):
    """With workspace_for(shard=True) the shards' row blocks split; the results
    are those of the whole batch."""
    import torch

    from gpu_util import device_inputs, f32_scale, max_rel, synth
    from paper_2410_17243_amd.shards import sharded_forward_backward

    img, txt = device_inputs(*synth.clip_pairs(b, d, 1.0, seed=b + d, dtype=dtype), dtype)
    sc = torch.tensor([f32_scale(14.29)], dtype=torch.float32, device="cuda")
    f = infcl.clip_loss_fwd(img, txt, sc)
    dI, dT, ds = infcl.clip_loss_bwd(img, txt, sc, f)
    size = infcl.workspace_for(img, shard=True).numel()
    bufs = [torch.full((size + 4096,), 0xA5, dtype=torch.uint8, device="cuda") for _ in range(n)]
    r = sharded_forward_backward(img, txt, sc.reshape(()), n, workspaces=[w[:size] for w in bufs])
    torch.cuda.synchronize()
    errs = [max_rel(x.double().cpu().numpy(), y.double().cpu().numpy())
            for x, y in ((r["dimg"], dI), (r["dtxt"], dT), (r["dscale64"], ds), (r["loss64"], f["loss64"]))]
    print(f"b={b} n={n} d={d} {dtype}: {errs}", flush=True)
    # G' of a shard differs by the rounding of its log-sum-exp values, which another
    # grid merges in another order: 2^-23 |lse| at |lse| up to 15
    assert max(errs) <= 2e-5
    assert all(bool((w[size:] == 0xA5).all()) for w in bufs)


@pytest.mark.gpu
def test_pending_losses_hold_no_workspace():
    """Losses whose backward is still to come (several batches in flight) keep
    their per-sample statistics, 20 bytes per sample, not their workspace."""
    import torch

    from gpu_util import f32_scale

    b, d, pending = 1000, 512, 6
    x = [torch.nn.functional.normalize(torch.randn(b, d, device="cuda"), dim=1).to(torch.bfloat16) for _ in range(2)]
    sc = torch.tensor([f32_scale(14.29)], dtype=torch.float32, device="cuda")
    leaves = [x[0].requires_grad_(), x[1].requires_grad_(), sc.requires_grad_()]
    ref = torch.autograd.grad(infcl.clip_loss(*leaves), leaves)
    base = torch.cuda.memory_allocated()
    losses = [infcl.clip_loss(*leaves) for _ in range(pending)]
    held = torch.cuda.memory_allocated() - base
    print(f"{held} bytes held by {pending} pending losses", flush=True)
    assert held <= pending * (20 * b + 4096)
    for loss in reversed(losses):
        for g, r in zip(torch.autograd.grad(loss, leaves), ref):
            assert torch.equal(g, r)
