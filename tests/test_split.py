"""Row blocks of the backward swept in several parts (batches, and remainders
of batches, with fewer row blocks than compute units): the partial sums are
added in a fixed order by a reduction kernel.

On the GPU the split is compared with the oracle at the parity bars of
test_parity (same inputs, same precision: only the order of the fp32 sums
differs), for whole blocks followed by a split remainder, for ragged last
blocks, for shards whose place for partial sums is limited, and bit for bit
against a second run.  Without a GPU: the workspace stays linear in b apart
from a bounded constant."""

import ctypes

import numpy as np
import pytest

import paper_2410_17243_amd as infcl
from test_plan import plans  # noqa: F401  (fixture)


def _ws(b, d, dt):
    out = ctypes.c_size_t(0)
    assert infcl.load_library().infcl_workspace_size(b, d, dt, ctypes.byref(out)) == infcl.INFCL_OK
    return out.value


@pytest.mark.parametrize("d,dt,per", [(128, 0, 336), (512, 0, 336), (768, 0, 336), (1024, 2, 336), (64, 1, 780),
                                       (512, 1, 780)])
def test_workspace_grows_by_a_bounded_constant(d, dt, per):
    for b in (1, 31, 257, 1000, 4096, 8191, 10007, 16500, 32768, 50000, 131071, 1 << 20, (1 << 22) + 5):
        w = _ws(b, d, dt)
        assert w <= per * b + b + (64 << 20) + (1 << 14), (b, w)


SPLIT = [
    (16420, 128, "bf16"),   # 128-row blocks: 256 whole, 2 split, the last of each side ragged
    (8320, 768, "bf16"),    # 64-row blocks: 256 whole, 4 split
    (193, 512, "f16"), (2049, 256, "bf16"), (1057, 512, "f32"), (65, 1024, "bf16"), (353, 64, "f32"),
]
WHOLE = [(129, 512, "f16"), (33, 64, "f32")]  # too few tiles to split
SPLIT_SHARDS = [(4000, 512, "bf16", 1024, 999), (3000, 768, "f16", 2976, 24), (2500, 128, "f32", 0, 1300)]


def test_the_shapes_below_are_split(plans):
    code = {"bf16": 0, "f32": 1, "f16": 2}
    q = [(b, b, d, code[dt], infcl.INFCL_SPLIT_BYTES) for b, d, dt in SPLIT]
    q += [(b, bs, d, code[dt], infcl.INFCL_SPLIT_BYTES) for b, d, dt, _, bs in SPLIT_SHARDS]
    q += [(b, b, d, code[dt], infcl.INFCL_SPLIT_BYTES) for b, d, dt in WHOLE]
    ns = [p["ns"] for p in plans(q)]
    assert min(ns[:-len(WHOLE)]) > 1 and set(ns[-len(WHOLE):]) == {1}, list(zip(q, ns))


@pytest.mark.gpu
def test_batch_of_one():
    """The only entry of S is the positive: no gradient at all."""
    from gpu_util import f32_scale, run, synth

    for d, dtype in ((256, "bf16"), (768, "f16"), (64, "f32")):
        img, txt = synth.clip_pairs(1, d, 1.0, seed=d, dtype=dtype)
        g = run(img, txt, dtype, f32_scale(14.29))
        assert g["loss64"] == 0.0 and g["dscale"] == 0.0
        assert not g["dI"].any() and not g["dT"].any()


@pytest.mark.gpu
@pytest.mark.parametrize("b,d,dtype", SPLIT + WHOLE)
def test_split_blocks_match_oracle(b, d, dtype):
    import oracle
    from gpu_util import f32_scale, max_rel, run, synth

    img, txt = synth.clip_pairs(b, d, 1.0, seed=b + d, dtype=dtype)
    s = f32_scale(14.29)
    ref, dI, dT, ds = oracle.forward_backward(synth.as_f64(img, dtype), synth.as_f64(txt, dtype), s)
    g = run(img, txt, dtype, s)
    tol = {"bf16": 2e-2, "f16": 2.5e-3, "f32": 1e-4}[dtype]
    eI, eT = max_rel(g["dI"], dI), max_rel(g["dT"], dT)
    print(f"b={b} d={d} {dtype}: dI {eI:.2e} dT {eT:.2e} ds {g['dscale']:.6e} ref {ds:.6e}", flush=True)
    assert eI <= tol and eT <= tol
    assert g["dscale"] == pytest.approx(ds, rel=tol, abs=1e-30)
    again = run(img, txt, dtype, s)
    assert np.array_equal(again["dI"], g["dI"]) and np.array_equal(again["dT"], g["dT"])
    assert again["dscale"] == g["dscale"]


@pytest.mark.gpu
@pytest.mark.parametrize("b,d,dtype,r0,bs", SPLIT_SHARDS)
def test_split_shard_matches_whole(b, d, dtype, r0, bs):
    import torch

    from gpu_util import device_inputs, f32_scale, max_rel, synth

    img, txt = synth.clip_pairs(b, d, 1.0, seed=b, dtype=dtype)
    I, T = device_inputs(img, txt, dtype)
    sc = torch.tensor([f32_scale(14.29)], dtype=torch.float32, device=I.device)
    f = infcl.clip_loss_fwd(I, T, sc)
    dI, dT, _ = infcl.clip_loss_bwd(I, T, sc, f)
    oI, oT = (torch.full((bs, d), float("nan"), dtype=torch.float32, device=I.device) for _ in range(2))
    ds = torch.empty((), dtype=torch.float64, device=I.device)
    infcl.infcl_bwd_shard(I, T, sc.reshape(()), r0, bs, f["lse_r"], f["lse_c"], f["aux"], None, oI, oT, ds,
                          f["workspace"])
    torch.cuda.synchronize()
    for o, w in ((oI, dI), (oT, dT)):
        # the same entries summed in another order; G' is formed alike
        assert max_rel(o.cpu().numpy().astype(np.float64), w[r0:r0 + bs].cpu().numpy().astype(np.float64)) <= 1e-5
    # the shard's share of dscale, in fp64: its rows' and its columns' terms
    x = f32_scale(14.29) * (synth.as_f64(img, dtype) @ synth.as_f64(txt, dtype).T)
    own = slice(r0, r0 + bs)
    u = np.diag(x) / f32_scale(14.29)

    def terms(x):  # rows own of x: softmax weights times u_ij - u_ii (the diagonal's is zero)
        m = x[own] - x[own].max(axis=1, keepdims=True)
        return np.sum(np.exp(m) / np.exp(m).sum(axis=1, keepdims=True) * (x[own] / f32_scale(14.29) - u[own, None]))

    want = (terms(x) + terms(x.T)) / (2 * b)
    print(f"b={b} d={d} {dtype} shard ({r0}, {bs}): dscale {float(ds):.9e} ref {want:.9e}", flush=True)
    assert float(ds) == pytest.approx(want, rel={"bf16": 2e-2, "f16": 2.5e-3, "f32": 1e-4}[dtype])
