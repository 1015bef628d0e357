"""Nothing behind the inputs takes part in a result.

The sweeps load whole 32-row tiles, and one or two tiles past the last, and
rely on the range check of their buffer resources to fill rows past the end
with zeros (sweep_tile_rsrc in csrc/sweep.hpp).  Here img and txt are the
first b rows of larger allocations whose other rows are NaN (every read, right
or wrong, stays inside the allocation), and the workspace starts as NaN bit
patterns.  A row past the end that got into a product would turn gradients or
statistics into NaN: every output must equal, bit for bit, that of the same
rows alone."""

import pytest
import torch

import paper_2410_17243_amd as infcl
from gpu_util import device_inputs, f32_scale, synth

pytestmark = pytest.mark.gpu

TAIL = 160  # rows behind the inputs: a ragged tile and four whole ones


def _outputs(img, txt, sc, fill):
    ws = infcl.workspace_for(img)
    ws.fill_(fill)
    f = infcl.clip_loss_fwd(img, txt, sc, workspace=ws)
    g = infcl.clip_loss_bwd(img, txt, sc, f)
    return [f[k] for k in ("loss64", "lse_r", "lse_c", "aux")] + list(g)


@pytest.mark.parametrize("d,dtype", [(128, "bf16"), (384, "bf16"), (512, "bf16"), (640, "bf16"), (768, "bf16"),
                                     (896, "bf16"), (1024, "bf16"), (128, "f16"), (512, "f16"), (640, "f16"),
                                     (768, "f16"), (1024, "f16"), (64, "f32"), (256, "f32"), (512, "f32")])
def test_rows_behind_the_inputs_take_no_part(d, dtype):
    sc = torch.tensor([f32_scale(14.29)], dtype=torch.float32, device="cuda")
    for b in (1, 15, 353, 367, 369, 372, 383):  # b % 32: 1, 15, 1, 15, 17, 20, 31
        img, txt = device_inputs(*synth.clip_pairs(b, d, 1.0, seed=b + d, dtype=dtype), dtype)
        ref = _outputs(img, txt, sc, 0)
        big = [torch.full((b + TAIL, d), float("nan"), dtype=img.dtype, device="cuda") for _ in range(2)]
        big[0][:b], big[1][:b] = img, txt
        got = _outputs(big[0][:b], big[1][:b], sc, 0xFF)
        print(f"b={b} d={d} {dtype}", flush=True)
        for r, o in zip(ref, got):
            assert not torch.isnan(r).any()
            assert torch.equal(r, o)
