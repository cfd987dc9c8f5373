"""Featureless nodes around the in-degree from which a whole workgroup sums a node: one edge
below and above it, hubs, more heavy nodes than a workgroup keeps, one and several 16-byte
chunks per lane; against float64 means of the same rows."""
import numpy as np
import pytest
import torch

from paper_2406_06022_amd import rgcn, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,nodes,nrel,degs", [
    ("bf16", 128, 700, 3, (0, 42, 43, 44, 300)),      # around 128 over three relations
    ("f32", 64, 333, 1, (127, 128, 129, 1, 5000)),
    ("f32", 8, 40_000, 1, (130, 129, 128, 131)),      # nearly every node heavy: lists fill up
    ("bf16", 520, 60, 2, (65, 64, 700)),              # 65 chunks: two per lane
    ("bf16", 2048, 30, 1, (128, 129, 900)),
    ("f32", 1024, 25, 4, (32, 33, 400)),
    ("bf16", 16, 90, 40, (3, 4, 30)),                 # groups as wide as the relations
])
def test_heavy_nodes(dtype, d, nodes, nrel, degs):
    gen = torch.Generator(device="cuda").manual_seed(nodes + d)
    tdt = synth.torch_dtype(dtype)
    rows = 500
    rels, total = [], torch.zeros((nodes, d), dtype=torch.float64, device="cuda")
    scale = torch.zeros_like(total)
    cnt = torch.zeros(nodes, dtype=torch.float64, device="cuda")
    for r in range(nrel):
        deg = torch.tensor(degs, device="cuda")[(torch.arange(nodes, device="cuda") + r // 2) % len(degs)]
        ip = torch.zeros(nodes + 1, dtype=torch.int64, device="cuda")
        torch.cumsum(deg, 0, out=ip[1:])
        ix = torch.randint(0, rows, (int(ip[-1]),), generator=gen, device="cuda")
        f = torch.randn((rows, d), generator=gen, device="cuda").to(tdt)
        rels.append((ip, ix, f))
        seg = torch.repeat_interleave(torch.arange(nodes, device="cuda"), deg)
        total.index_add_(0, seg, f[ix].double())
        scale.index_add_(0, seg, f[ix].double().abs())
        cnt += deg
    out = torch.full((nodes, d), float("nan"), dtype=tdt, device="cuda")
    print(f"case heavy {dtype} d={d} nodes={nodes} nrel={nrel}", flush=True)
    rgcn.rgcn_featureless_mean(rels, nodes, out, flags=rgcn.RGCN_VALIDATE_DEVICE)
    n = cnt.clamp(min=1)[:, None]
    want, mag = total / n, scale / n
    # compensated sums: 2^-23 of the mean magnitude, the quotient an ulp, bf16 half an ulp
    bound = 2.0 ** -22 * mag + 2.0 ** -23 * want.abs()
    if dtype == "bf16":
        bound = bound + 2.0 ** -8 * want.abs()
    assert bool(((out.double() - want).abs() <= bound + 1e-30).all())
