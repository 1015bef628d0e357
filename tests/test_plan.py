"""How the backward is split over workgroups (plan_bwd), on the host: a small
program linked to the library asks it for plans; nothing launches on a GPU."""

import os
import subprocess

import pytest

import paper_2410_17243_amd as infcl
from test_layout import ROOT, _hipcc

SRC = r"""
#include "bwd.hpp"
#include "infcl.h"
#include <cstdio>
namespace infcl { BwdPlan plan_bwd(int64_t b, int64_t nrows, int64_t d, int dtype, size_t cap); }
int main() {
  printf("%zu %lld\n", (size_t)INFCL_SPLIT_BYTES, (long long)INFCL_SPLIT_BATCH);
  long long b, nrows, d, cap;
  int dtype;
  while (scanf("%lld %lld %lld %d %lld", &b, &nrows, &d, &dtype, &cap) == 5) {
    const infcl::BwdPlan p = infcl::plan_bwd(b, nrows, d, dtype, (size_t)cap);
    printf("%d %d %d %d %d %d %zu\n", p.bm, p.nblk, p.nfull, p.ns, p.gran, p.nwg, p.part_bytes);
  }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    cc = _hipcc()
    if cc is None:
        pytest.skip("hipcc not available")
    pkg = os.path.join(ROOT, "paper_2410_17243_amd")
    tmp = tmp_path_factory.mktemp("plan")
    src, exe = tmp / "plan.hip", str(tmp / "plan")
    src.write_text(SRC)
    r = subprocess.run([cc, "--offload-arch=gfx950", "-O1", "-std=c++17",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-I", f"{pkg}/csrc", "-I", f"{ROOT}/include", str(src), "-o", exe,
                        "-L", pkg, "-linfcl", f"-Wl,-rpath,{pkg}"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def ask(queries):
        """(b, nrows, d, dtype code, bytes of room) -> dicts"""
        text = "\n".join(" ".join(str(x) for x in q) for q in queries)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60)
        assert r.returncode == 0
        lines = r.stdout.splitlines()
        assert [int(x) for x in lines[0].split()] == [infcl.INFCL_SPLIT_BYTES, infcl.INFCL_SPLIT_BATCH]
        names = ("bm", "nblk", "nfull", "ns", "gran", "nwg", "part_bytes")
        return [dict(zip(names, (int(x) for x in ln.split()))) for ln in lines[1:]]

    return ask


ROOM = infcl.INFCL_SPLIT_BYTES


def test_plans_cover_the_row_blocks_within_their_room(plans):
    q = [(b, n, d, dt, cap) for d, dt in ((128, 0), (512, 0), (640, 2), (768, 0), (1024, 0), (64, 1), (512, 1))
         for b in (1, 33, 1000, 8320, 16420, 32768, 32769, 65536, 131072, 1 << 30)
         for n in sorted({1, min(b, 999), (b + 7) // 8, b}) for cap in (0, 1 << 20, 20 << 20, ROOM)]
    for (b, n, d, dt, cap), p in zip(q, plans(q)):
        assert p["nblk"] * p["bm"] >= n > (p["nblk"] - 1) * p["bm"]
        rem = 2 * p["nblk"] - p["nfull"]
        assert p["nwg"] == p["nfull"] + rem * p["ns"]
        if p["ns"] == 1:
            assert rem == 0 and p["part_bytes"] == 0
        else:
            assert p["nfull"] % 256 == 0 and rem < 256 and p["part_bytes"] <= cap
            assert p["part_bytes"] == rem * p["ns"] * p["bm"] * d * 4 + 8 * p["nwg"]
            units = -(-(-(-b // 32)) // p["gran"])
            assert p["ns"] <= units  # every part has tiles


@pytest.mark.parametrize("b,n,d,dt", [
    (32768, 8, 512, 0), (32800, 8, 512, 0), (49152, 8, 512, 0), (65536, 8, 512, 0), (65536, 8, 256, 2),
    (65536, 8, 384, 0), (131072, 16, 512, 0), (65536, 16, 768, 0), (65536, 16, 512, 1),
])
def test_shards_fill_the_compute_units(plans, b, n, d, dt):
    """A shard whose row blocks are fewer than the compute units is split, on
    both sides of INFCL_SPLIT_BATCH, with the room that workspace_for(shard=True)
    gives."""
    bs = -(-b // n // 32) * 32
    whole, split = plans([(b, bs, d, dt, 0), (b, bs, d, dt, ROOM)])
    assert whole["ns"] == 1 and whole["nwg"] <= 170
    assert split["ns"] > 1 and split["nwg"] >= 192


def test_workspace_for_a_shard_has_the_room():
    import torch

    for b in (32768, 32769, 65536):
        x = torch.empty((b, 64), dtype=torch.bfloat16, device="meta")
        extra = infcl.workspace_for(x, shard=True).numel() - infcl.workspace_for(x).numel()
        assert extra == (ROOM if b > infcl.INFCL_SPLIT_BATCH else 0)
