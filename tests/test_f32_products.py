"""fp32 inputs: products of three-part bf16 operands against the fp64 oracle.

The parts of an fp32 number add up to it exactly (of magnitudes from 2^-110 on;
below, to within 2^-134) and the part products left out are at most 2^-24 of
the full product, as much as fp32's own rounding of it, so the results carry
fp32 rounding only: the log-sum-exp bound of gpu_util.lse_tol, and for the gradients 1e-5 of
their maximum (fp32 accumulation over up to 3300 terms, 2^-24 sqrt(3300) =
3.4e-6, and the exponents' own rounding, 2^-24 |y| ln 2 with |y| up to 144 at
s = 100, which 1e-4 covers there).  Shapes: both tile shapes of the forward (32 x 128
below 192 tiles of 64 x 256), every width class of the backward (whole and half
last segments), ragged ends; a well-separated batch, whose weights are as
small as 1e-31 (their low parts are kept normal by a power of two); rows of
very different magnitude; the error against fp64 of products of awkward
mantissas (all 24 bits set)."""

import numpy as np
import pytest

import oracle
from gpu_util import f32_scale, lse_tol, max_rel, run, synth

pytestmark = pytest.mark.gpu


def _check(img, txt, s, d, tol, lse_s=None):
    ref, dI, dT, ds = oracle.forward_backward(img.astype(np.float64), txt.astype(np.float64), s)
    g = run(img, txt, "f32", s)
    print(f"dI {max_rel(g['dI'], dI):.2e} dT {max_rel(g['dT'], dT):.2e} "
          f"lse {np.max(np.abs(g['lse_r'] - ref['lse_r'])):.2e} ds {g['dscale']:.8e} ref {ds:.8e}", flush=True)
    assert np.all(np.abs(g["lse_r"] - ref["lse_r"]) <= lse_tol(lse_s or s, d, ref["lse_r"]))
    assert np.all(np.abs(g["lse_c"] - ref["lse_c"]) <= lse_tol(lse_s or s, d, ref["lse_c"]))
    assert max_rel(g["dI"], dI) <= tol and max_rel(g["dT"], dT) <= tol
    assert g["dscale"] == pytest.approx(ds, rel=tol, abs=1e-30)
    assert g["loss64"] == pytest.approx(ref["loss"], rel=tol, abs=1e-30)


@pytest.mark.parametrize("b,d", [(3300, 64), (3201, 192), (700, 320), (513, 448), (1100, 512), (257, 128), (33, 256)])
def test_shapes(b, d):
    img, txt = synth.clip_pairs(b, d, 1.0, seed=b + d, dtype="f32")
    _check(img, txt, f32_scale(14.29), d, 1e-5)


@pytest.mark.parametrize("s,sigma", [(50.0, 1.0), (100.0, 0.5)])
def test_separated_batch(s, sigma):
    img, txt = synth.clip_pairs(1200, 512, sigma, seed=3, dtype="f32")
    _check(img, txt, f32_scale(s), 512, 1e-4)


def test_mixed_row_norms():
    b, d = 900, 256
    img, txt = synth.clip_pairs(b, d, 1.0, seed=5, dtype="f32")
    img = (img * (2.0 ** ((np.arange(b) % 7) - 3))[:, None]).astype(np.float32)
    txt = (txt * (2.0 ** ((np.arange(b) * 3 % 7) - 3))[:, None]).astype(np.float32)
    _check(img, txt, f32_scale(1.0), d, 1e-4, lse_s=64.0)


def test_full_mantissas():
    """Entries with all 24 mantissa bits set: a part dropped or misplaced shows
    as 2^-16 or 2^-8 of the entries' scale."""
    b, d = 384, 128
    rng = np.random.default_rng(7)
    full = np.float32(2.0) - np.float32(2.0 ** -23)
    sgn = rng.choice([-1.0, 1.0], size=(2, b, d)).astype(np.float32)
    e = rng.integers(-6, -3, size=(2, b, d))
    img, txt = (full * sgn * np.exp2(e.astype(np.float32))).astype(np.float32)
    _check(img, txt, f32_scale(4.0), d, 1e-5)


@pytest.mark.parametrize("b,d", [(300, 128), (8192, 64)])  # split row blocks and the reduction; whole row blocks
def test_tiny_upstream_gradient(b, d):
    """A power of two in dloss scales the gradients exactly (where they are
    normal numbers): the power of two that G' carries is divided out of the
    sums, not of the factor dloss s / 2b, which it would make subnormal."""
    e = -112
    img, txt = synth.clip_pairs(b, d, 1.0, seed=b, dtype="f32")
    one, tiny = (run(img, txt, "f32", f32_scale(14.29), dloss=v) for v in (1.0, 2.0 ** e))
    for k in ("dI", "dT"):
        want = one[k] * 2.0 ** e
        normal = np.abs(want) >= 2.0 ** -126
        print(f"b={b} {k}: {normal.mean():.3f} normal, "
              f"max rel {np.max(np.abs(tiny[k] - want)[normal] / np.abs(want)[normal]):.2e}", flush=True)
        assert normal.mean() > 0.5
        assert np.array_equal(tiny[k][normal], want[normal])


@pytest.mark.parametrize("b,d", [(700, 128), (8192, 64)])
@pytest.mark.parametrize("big", [2.0 ** 127, 3.4028235e38])
def test_large_entries(b, d, big):
    """The power of two that G' carries must not take finite sums past the
    largest float, and entries from 2^128 - 2^119 on, which round to
    an infinite bf16, have the largest bf16 as their first part.  One entry of each
    column is large (in a row that finds its text, |G'_ii| < 1) and the others
    are below 2^122, so that no sum overflows by itself; the fp32 result then
    carries fp32 rounding only."""
    rng = np.random.default_rng(b)
    img, txt = synth.clip_pairs(b, d, 1.0, seed=b, dtype="f32")
    img = (img * np.float32(2.0 ** 121)).astype(np.float32)
    rows = rng.choice(b, size=d, replace=False)
    sgn = rng.choice([-1.0, 1.0], size=d).astype(np.float32)
    img[rows, np.arange(d)] = np.float32(big) * sgn
    txt[rows, np.arange(d)] = 0.9 * sgn
    txt = (txt * np.float32(2.0 ** -100)).astype(np.float32)
    s, dl = f32_scale(2.0 ** -24), 2.0 ** 24
    ref, dI, dT, ds = oracle.forward_backward(img.astype(np.float64), txt.astype(np.float64), s)
    g = run(img, txt, "f32", s, dloss=dl)
    print(f"b={b} loss {g['loss64']:.9e} ref {ref['loss']:.9e} dI {max_rel(g['dI'], dl * dI):.2e} "
          f"dT {max_rel(g['dT'], dl * dT):.2e} ds {g['dscale']:.6e} ref {dl * ds:.6e}", flush=True)
    assert np.max(np.abs(dT)) * 2 * b / s < 3e38  # the sum before the factor s / 2b
    assert g["loss64"] == pytest.approx(ref["loss"], rel=1e-5)
    assert max_rel(g["dI"], dl * dI) <= 1e-4 and max_rel(g["dT"], dl * dT) <= 1e-4
    assert g["dscale"] == pytest.approx(dl * ds, rel=1e-4)


@pytest.mark.parametrize("e", [-104, -116])
def test_tiny_entries(e):
    """Parts of entries below 2^-110 are subnormal, which the conversion and the
    MFMA keep: each entry is right to within 2^-134, so an exponent is right to
    within s 2^-134 times its text row's 1-norm (at most sqrt(d) for unit rows)."""
    b, d = 500, 128
    img, txt = synth.clip_pairs(b, d, 1.0, seed=11, dtype="f32")
    img = (img * np.float32(2.0 ** e)).astype(np.float32)
    s = f32_scale(14.29 * 2.0 ** -e)
    ref, dI, dT, ds = oracle.forward_backward(img.astype(np.float64), txt.astype(np.float64), s)
    g = run(img, txt, "f32", s)
    dx = s * np.sqrt(d) * 2.0 ** -134
    print(f"e={e} dx {dx:.2e} lse {np.max(np.abs(g['lse_r'] - ref['lse_r'])):.2e} dI {max_rel(g['dI'], dI):.2e} "
          f"dT {max_rel(g['dT'], dT):.2e}", flush=True)
    for k in ("lse_r", "lse_c"):
        assert np.all(np.abs(g[k] - ref[k]) <= lse_tol(14.29, d, ref[k]) + dx)
    # a weight's relative error is at most that of its two exponents, 2 dx each
    assert max_rel(g["dI"], dI) <= 1e-5 + 4 * dx and max_rel(g["dT"], dT) <= 1e-5 + 4 * dx
