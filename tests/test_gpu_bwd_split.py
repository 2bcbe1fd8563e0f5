"""The backward where its plan cuts work units in two (few units per CU): the
halves' atomic adds into zeroed outputs, against the fp64 oracle with the
per-element bound of tests/test_gpu_bwd.py, and bit for bit between two calls.
The outputs start as NaN, so a row that is not zeroed first shows."""
import pytest
import torch

import oracle
from paper_2609_36757_amd import fastvr
from paper_2609_36757_amd.workloads import make_qkv

from parity import default_scale, fp32_scale, to_np
from test_gpu_bwd import _draw_do, _rounding_sigmas, compare_grad, dev  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

# name, B, H, d, Nq, chunk_len, q_chunk_offset, W: the plan splits dQ units only in the
# first two and both kinds in the others (256 CUs; tests/bwd_plan_check.cpp checks that)
CASES = [
    ("dq_ragged_tiles", 2, 4, 128, 1616, 230, 0, -1),
    ("dq_stream_d64", 1, 2, 64, 300, 300, 2, -1),
    ("both_ragged", 1, 2, 128, 1537, 500, 0, -1),
    ("both_grouped_chunks", 1, 1, 64, 2105, 100, 0, -1),
    ("both_unseen_keys", 1, 1, 128, 1300, 1300, 2, 0),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_bwd_split_units(dev, case):  # noqa: F811
    name, B, H, d, nq, L, off, W = case
    nkv = off * L + nq
    print(f"\n[gpu case] bwd split {name} B={B} H={H} d={d} Nq={nq} Nkv={nkv} L={L} off={off} W={W}", flush=True)
    scale = default_scale(d)
    q, k, v = make_qkv(B, nq, nkv, H, d, 900 + nq)
    do = _draw_do(B, nq, H, d, 901 + nq)
    qd, kd, vd, dod = (t.to(dev) for t in (q, k, v, do))
    kw = dict(chunk_len=L, q_chunk_offset=off, window_chunks=W, scale=scale)
    o, lse = fastvr.chunk_attn(qd, kd, vd, **kw)
    runs = []
    for _ in range(2):
        outs = [torch.full((B, n, H, d), float("nan"), device=dev) for n in (nq, nkv, nkv)]
        runs.append(fastvr.chunk_attn_bwd(qd, kd, vd, o, lse, dod, dq=outs[0], dk=outs[1], dv=outs[2], **kw))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*runs))
    s32 = fp32_scale(scale)
    ref = oracle.attention_bwd(q, k, v, do, chunk_len=L, q_chunk_offset=off, window_chunks=W, scale=s32)
    sig = _rounding_sigmas(q, k, v, do, L, off, W, s32)
    for n, g, r, s in zip(("dq", "dk", "dv"), runs[0], ref, sig):
        compare_grad(n, to_np(g), r, s, name)
    seen = oracle.visibility_mask(nq, nkv, L, off, W).any(axis=0)
    assert (to_np(runs[0][1])[:, ~seen] == 0).all() and (to_np(runs[0][2])[:, ~seen] == 0).all()


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_bwd_outputs_in_pinned_host_memory(dev, case):  # noqa: F811
    """Outputs that are not the GPU's own memory take no atomic adds: the plan
    must not cut units in two, so pinned host outputs hold the bits of the
    unsplit units, which the same heads repeated as a large call run."""
    name, B, H, d, nq, L, off, W = case
    nkv = off * L + nq
    reps = 1 + 4 * 256 // (B * H)  # one 256-row query tile per head alone is then over 4 units per CU
    print(f"\n[gpu case] bwd pinned outputs {name} B={B} H={H} d={d} Nq={nq} L={L} reps={reps}", flush=True)
    kw = dict(chunk_len=L, q_chunk_offset=off, window_chunks=W, scale=default_scale(d))
    q, k, v = (t.to(dev) for t in make_qkv(B, nq, nkv, H, d, 900 + nq))
    do = _draw_do(B, nq, H, d, 901 + nq).to(dev)
    o, lse = fastvr.chunk_attn(q, k, v, **kw)
    host = [torch.full((B, n, H, d), float("nan"), pin_memory=True) for n in (nq, nkv, nkv)]
    fastvr.chunk_attn_bwd(q, k, v, o, lse, do, dq=host[0], dk=host[1], dv=host[2], **kw)
    wide = [t.repeat(1, 1, reps, 1) for t in (q, k, v, o)]
    ref = fastvr.chunk_attn_bwd(*wide, lse.repeat(1, reps, 1), do.repeat(1, 1, reps, 1), **kw)
    torch.cuda.synchronize()
    for n, a, b in zip(("dq", "dk", "dv"), host, ref):
        assert torch.equal(a, b[:, :, :H].cpu()), (name, n)
