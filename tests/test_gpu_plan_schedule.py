"""The plan's schedules item by item (a stable sort by degree key, as the header defines it)
and its transposes, where the number of sort tiles (4,096 items) changes the way a tile finds
its place: one tile, a few, more than 128; types with few, many and no rows or relations;
more slots than the first launch carries."""
import numpy as np
import pytest
import torch

import oracle
from paper_2406_06022_amd import rgcn, synth

pytestmark = pytest.mark.gpu


def _key(deg):
    deg = np.asarray(deg, dtype=np.int64)
    lg = np.floor(np.log2(np.maximum(deg, 1))).astype(np.int64)
    return np.where(deg <= 32, 31, np.maximum(0, 30 - (lg - 5)))


def _relation(rng, s, t, n_src, n_dst, heavy):
    deg = rng.integers(0, 4, size=n_dst)
    if heavy and n_dst:
        deg[rng.random(n_dst) < heavy] = rng.integers(33, 150)
    ip = np.zeros(n_dst + 1, np.int64)
    np.cumsum(deg, out=ip[1:])
    # squared draws: popular sources, so the transpose has heavy rows too
    ix = (rng.random(int(ip[-1])) ** 2 * n_src).astype(np.int32)
    return synth.Relation(s, t, ip.astype(np.int32), ix)


@pytest.mark.parametrize("n_src,n_dst,rels,heavy", [
    ([50, 20], [30, 20], [(0, 0), (1, 0), (0, 1)], 0.1),                  # one tile each
    ([9000, 4096, 0, 5000], [4097, 4096, 0, 0], [(0, 0), (0, 1), (1, 0)], 0.02),
    ([600_000, 3000], [530_000, 3000], [(0, 0), (1, 0), (0, 1)], 0.001),  # over 128 tiles
    ([700, 500], [400, 300], [(0, 0), (1, 1), (0, 1), (1, 0)] * 16, 0.05),  # 66 slots
    ([20_000, 100], [19_000, 100], [(0, 0), (1, 0)], 0.0),                # light: enumeration order
])
@pytest.mark.parametrize("keep", [False, True])
def test_schedules_and_transposes(n_src, n_dst, rels, heavy, keep):
    rng = np.random.default_rng(sum(n_src) + len(rels))
    blk = synth.Block(list(n_src), list(n_dst), [
        _relation(rng, s, t, n_src[s], n_dst[t], heavy) for s, t in rels])
    T = len(n_src)
    dblk = rgcn.DeviceBlock(blk, (1 << T) - 1)
    w = [torch.zeros((4, 4), device="cuda") for _ in range(T)]
    params = rgcn.Params("f32", 4, 4, [w[0]] * len(rels), w)
    ws = rgcn.new_workspace(dblk, params)
    ws.fill_(0xFF)
    print(f"case plan n_src={n_src} rels={len(rels)} nnz={blk.nnz} keep={keep}", flush=True)
    rgcn.rgcn_block_plan(dblk, params, ws, rgcn.RGCN_PLAN_ENUMERATION_ORDER if keep else 0)
    torch.cuda.synchronize()
    lay = rgcn.rgcn_block_plan_layout(dblk, params)

    def arr(off, n):
        return np.frombuffer(ws[off:off + 4 * n].cpu().numpy().tobytes(), dtype=np.int32)

    deg = []
    for t in range(T):
        if n_dst[t]:
            deg.append(np.ones(n_dst[t], np.int64))
            deg += [np.diff(r.indptr) for r in blk.rels if r.dst_type == t]
    deg = np.concatenate(deg)
    want = np.arange(deg.size) if keep else np.argsort(_key(deg), kind="stable")
    assert np.array_equal(arr(lay["fwd_order"], lay["n_fwd_segments"]), want)
    csc_deg = [np.zeros(n, np.int64) for n in n_src]
    for r, rel in enumerate(blk.rels):
        want_ip, want_dst, _ = oracle.csc(n_src[rel.src_type], rel.indptr, rel.indices)
        ip = arr(lay["csc_indptr"][r], n_src[rel.src_type] + 1)
        assert np.array_equal(ip - ip[0], want_ip), r
        assert np.array_equal(arr(lay["csc_dst"][r], rel.nnz), want_dst), r
        csc_deg[rel.src_type] += np.diff(want_ip)
    got, base = arr(lay["bwd_order"], lay["n_bwd_rows"]), 0
    for t in range(T):
        want = np.arange(n_src[t]) if keep else np.argsort(_key(csc_deg[t]), kind="stable")
        assert np.array_equal(got[base:base + n_src[t]], want), t
        base += n_src[t]
    assert base == got.size
