"""The edge cases of the other GPU tests on the kernels that large calls run.

Small calls run the forward's 128-row items, and the backward's units cut in two,
so the shapes of tests/test_gpu_parity.py, test_gpu_ring.py, test_gpu_zero_fill.py
and test_gpu_bwd.py, taken alone, do not reach the 256-row kernels (plain and ring
step) and reach the uncut units only in part.  Here their heads are repeated until
there are more than 1024 of them (batch * heads): then every call has more than
four items per CU, the plan keeps 256 rows, no item lists (at most 1024 items) and
whole units (tests/fwd_plan_check.cpp and bwd_plan_check.cpp check those plans).
The first copy of the heads is held against the fp64 oracle, the others against
the first, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_36757_amd import fastvr
from paper_2609_36757_amd.workloads import make_qkv, randn_bf16

from parity import compare, default_scale, fp32_scale, run_oracle, sample_rows, to_np
from test_gpu_bwd import BWD_CASES, _rounding_sigmas, compare_grad
from test_gpu_parity import CASES
from test_gpu_ring import RING_CASES
from test_gpu_zero_fill import BWD_CASES as BWD_TAIL_CASES
from test_gpu_zero_fill import FWD_CASES, PAD, _bits, _tail

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fastvr.load()
    return torch.device("cuda:0")


def _announce(label):
    print(f"\n[gpu case] full items: {label}", flush=True)


def _reps(bh):
    """Copies of bh heads that make more than 1024."""
    return 1024 // bh + 1


def _wide(t, reps):
    """[B, N, H, ...] -> [B, N, reps * H, ...], head r * H + h a copy of head h."""
    return t.repeat(1, 1, reps, *([1] * (t.dim() - 3)))


def _first_heads(o, lse, H):
    """The first H heads of O and LSE, after checking that all copies equal them."""
    ov, lv = o.unflatten(2, (-1, H)), lse.unflatten(1, (-1, H))
    assert torch.equal(_bits(ov[:, :, :1].expand_as(ov).contiguous()), _bits(ov.contiguous()))
    assert torch.equal(_bits(lv[:, :1].expand_as(lv).contiguous()), _bits(lv.contiguous()))
    return o[:, :, :H], lse[:, :H]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_forward(dev, case):
    name, B, H, d, nq, nkv, L, off, W, scale, seed = case
    scale = default_scale(d) if scale is None else scale
    reps = _reps(B * H)
    _announce(f"{name} B={B} H={H}x{reps} d={d} Nq={nq} Nkv={nkv} L={L} off={off} W={W} scale={scale}")
    q, k, v = make_qkv(B, nq, nkv, H, d, seed)
    out = torch.full((B, nq, reps * H, d), float("nan"), device=dev)
    o, lse = fastvr.chunk_attn(*(_wide(t.to(dev), reps) for t in (q, k, v)), chunk_len=L, q_chunk_offset=off,
                               window_chunks=W, scale=scale, out=out)
    torch.cuda.synchronize()
    o, lse = _first_heads(o, lse, H)
    o_ref, l_ref = run_oracle(q, k, v, L, off, W, scale)
    compare(to_np(o), to_np(lse), o_ref, l_ref, label=f"full items {name}")


@pytest.mark.parametrize("case", FWD_CASES, ids=[c[0] for c in FWD_CASES])
def test_forward_poisoned_tails(dev, case):
    """Rows past Nq and past the filled keys hold NaN (see test_gpu_zero_fill.py)."""
    name, H, d, nq, nkv, extra, L, off, W = case
    reps = _reps(H)
    _announce(f"poisoned {name} H={H}x{reps} d={d} Nq={nq} Nkv={nkv}+{extra} L={L} off={off} W={W}")
    scale = default_scale(d)
    q, k, v = make_qkv(1, nq, nkv, H, d, seed=900 + nq)
    qd = _tail(_wide(q.to(dev), reps), PAD, True, dev, 1)
    kd, vd = (_tail(_wide(t.to(dev), reps), extra + PAD, True, dev, 2) for t in (k, v))
    if extra:
        kd, vd = (t.as_strided((1, nkv + extra, reps * H, d), t.stride()) for t in (kd, vd))
    o, lse = fastvr.chunk_attn(qd, kd, vd, chunk_len=L, q_chunk_offset=off, window_chunks=W, scale=scale)
    torch.cuda.synchronize()
    o, lse = _first_heads(o, lse, H)
    kf, vf = (torch.cat([t, torch.zeros((1, extra, H, d), dtype=t.dtype)], dim=1) for t in (k, v))
    o_ref, l_ref = run_oracle(q, kf, vf, L, off, W, scale)
    compare(to_np(o), to_np(lse), o_ref, l_ref, label=f"full items poisoned {name}")


@pytest.mark.parametrize("d,W", [(128, -1), (128, 1), (64, 1)])
def test_strided_cache_bf16_output(dev, d, W):
    """Two batch rows of a cache whose rows past the filled ones are NaN, q a strided
    view, O as bf16 into a strided view: the fp32 call's bits rounded, nothing
    written outside the view."""
    B, H, L, cap, n_new, off = 2, 2, 300, 1500, 200, 3
    reps, n = _reps(B * H), off * L + n_new
    _announce(f"strided cache B={B} H={H}x{reps} d={d} L={L} cap={cap} len={n} W={W}")
    q, k, v = make_qkv(B, n_new, n, H, d, seed=950 + d + W)
    cache = [torch.full((B, cap, reps * H, d), float("nan"), dtype=torch.bfloat16, device=dev) for _ in range(2)]
    for c, t in zip(cache, (k, v)):
        c[:, :n] = _wide(t.to(dev), reps)
    qbuf = torch.full((B, n_new + PAD, reps * H, d), float("nan"), dtype=torch.bfloat16, device=dev)
    qbuf[:, :n_new] = _wide(q.to(dev), reps)
    kw = dict(chunk_len=L, q_chunk_offset=off, window_chunks=W)
    args = (qbuf[:, :n_new], cache[0][:, :n], cache[1][:, :n])
    o, lse = fastvr.chunk_attn(*args, **kw)
    big = torch.full((B, n_new + 9, reps * H, d), float("nan"), dtype=torch.bfloat16, device=dev)
    ob = big[:, 4:4 + n_new]
    _, lse_b = fastvr.chunk_attn(*args, out=ob, **kw)
    torch.cuda.synchronize()
    assert torch.equal(ob, o.to(torch.bfloat16)) and torch.equal(lse_b, lse)
    assert torch.isnan(big[:, :4].float()).all() and torch.isnan(big[:, 4 + n_new:].float()).all()
    o, lse = _first_heads(o, lse, H)
    o_ref, l_ref = run_oracle(q, k, v, L, off, W, default_scale(d))
    compare(to_np(o), to_np(lse), o_ref, l_ref, label=f"full items strided cache d={d} W={W}")


@pytest.mark.parametrize("case", RING_CASES, ids=[c[0] for c in RING_CASES])
def test_ring_stream(dev, case):
    """Streaming through the ring: every step's bits are the parallel call's, the
    ring holds the last W + 1 chunks.  The slot a step replaces is NaN before it,
    and with one batch row so is the memory after the new chunk."""
    name, B, H, d, N, L, W, seed, *opt = case
    scale = opt[0] if opt else default_scale(d)
    reps = _reps(B * H)
    _announce(f"ring {name} B={B} H={H}x{reps} d={d} N={N} L={L} W={W} scale={scale}")
    q, k, v = make_qkv(B, N, N, H, d, seed)
    qd, kd, vd = (_wide(t.to(dev), reps) for t in (q, k, v))
    full_o, full_l = fastvr.chunk_attn(qd, kd, vd, chunk_len=L, window_chunks=W, scale=scale)
    ring_k = torch.full((B, (W + 1) * L, reps * H, d), float("nan"), dtype=torch.bfloat16, device=dev)
    ring_v = torch.full_like(ring_k, float("nan"))
    for c in range(-(-N // L)):
        s = slice(c * L, min((c + 1) * L, N))
        slot = c % (W + 1) * L
        for r in (ring_k, ring_v):
            r[:, slot:slot + L] = float("nan")
        new = [t[:, s].contiguous() for t in (qd, kd, vd)]
        if B == 1:
            new = [_tail(t, PAD, True, dev, 0) for t in new]
        o, lse = fastvr.chunk_attn_ring_step(*new, ring_k, ring_v, chunk_len=L, chunk_index=c, window_chunks=W,
                                             scale=scale)
        torch.cuda.synchronize()
        assert torch.equal(_bits(o), _bits(full_o[:, s].contiguous())), f"chunk {c}"
        assert torch.equal(_bits(lse), _bits(full_l[:, :, s].contiguous())), f"chunk {c}"
        n = s.stop - s.start
        assert torch.equal(ring_k[:, slot:slot + n], kd[:, s]) and torch.equal(ring_v[:, slot:slot + n], vd[:, s]), c
    o, lse = _first_heads(full_o, full_l, H)
    o_ref, l_ref = run_oracle(q, k, v, L, 0, W, scale)
    compare(to_np(o), to_np(lse), o_ref, l_ref, label=f"full items ring {name}")


def _bwd(dev, q, k, v, do, reps, pad, **kw):
    """Gradients of the repeated heads; with pad, rows past Nq and Nkv hold NaN."""
    H = q.shape[2]
    w = [_wide(t.to(dev), reps) for t in (q, k, v, do)]
    o, lse = fastvr.chunk_attn(*w[:3], **kw)
    if pad:
        w, o = [_tail(t, PAD, True, dev, 0) for t in w], _tail(o, PAD, True, dev, 0)
    outs = [torch.full(t.shape, float("nan"), device=dev) for t in w[:3]]
    fastvr.chunk_attn_bwd(*w[:3], o, lse, w[3], dq=outs[0], dk=outs[1], dv=outs[2], **kw)
    torch.cuda.synchronize()
    for name, g in zip(("dq", "dk", "dv"), outs):
        gv = g.unflatten(2, (-1, H))
        assert torch.equal(gv, gv[:, :, :1].expand_as(gv)), name
    return [g[:, :, :H] for g in outs]


@pytest.mark.parametrize("case", BWD_CASES, ids=[c[0] for c in BWD_CASES])
def test_backward(dev, case):
    name, B, H, d, nq, nkv, L, off, W, scale, seed = case
    scale = default_scale(d) if scale is None else scale
    reps = _reps(B * H)
    _announce(f"bwd {name} B={B} H={H}x{reps} d={d} Nq={nq} Nkv={nkv} L={L} off={off} W={W} scale={scale}")
    q, k, v = make_qkv(B, nq, nkv, H, d, seed)
    do = randn_bf16((B, nq, H, d), torch.Generator().manual_seed(seed + 1000))
    kw = dict(chunk_len=L, q_chunk_offset=off, window_chunks=W)
    grads = _bwd(dev, q, k, v, do, reps, False, scale=scale, **kw)
    s32 = fp32_scale(scale)
    refs = oracle.attention_bwd(q, k, v, do, scale=s32, **kw)
    sig = _rounding_sigmas(q, k, v, do, L, off, W, s32)
    for n, g, r, s in zip(("dq", "dk", "dv"), grads, refs, sig):
        compare_grad(n, to_np(g), r, s, f"full items {name}")


@pytest.mark.parametrize("case", BWD_TAIL_CASES, ids=[c[0] for c in BWD_TAIL_CASES])
def test_backward_poisoned_tails(dev, case):
    name, H, d, nq, nkv, L, off, W = case
    reps = _reps(H)
    _announce(f"bwd poisoned {name} H={H}x{reps} d={d} Nq={nq} Nkv={nkv} L={L} off={off} W={W}")
    q, k, v = make_qkv(1, nq, nkv, H, d, seed=980 + nq)
    do = randn_bf16((1, nq, H, d), torch.Generator().manual_seed(981))
    kw = dict(chunk_len=L, q_chunk_offset=off, window_chunks=W, scale=default_scale(d))
    for n, a, b in zip(("dq", "dk", "dv"), *(_bwd(dev, q, k, v, do, reps, pad, **kw) for pad in (True, False))):
        assert torch.isfinite(a).all(), f"{name}: NaN in {n}"
        assert np.array_equal(to_np(a), to_np(b)), f"{name}: {n} differs from the run without NaN tails"


def test_backward_more_units_than_one_launch(dev):
    """65536 heads of 65 one-token chunks: 8519680 units, more than a grid of 512-thread
    workgroups holds (8388607), so the last ones come from a second launch.  Gradients
    against the same two batch rows in a call of one launch, bit for bit."""
    B, H, d, N, reps = 2, 64, 64, 65, 512
    assert 2 * reps * B * H * N > (1 << 32) // 512 - 1
    _announce(f"bwd two launches B={B}x{reps} H={H} d={d} N={N} L=1 W=1")
    kw = dict(chunk_len=1, window_chunks=1)
    q, k, v = (t.to(dev) for t in make_qkv(B, N, N, H, d, seed=77))
    do = randn_bf16((B, N, H, d), torch.Generator().manual_seed(78)).to(dev)
    o, lse = fastvr.chunk_attn(q, k, v, **kw)
    ref = fastvr.chunk_attn_bwd(q, k, v, o, lse, do, **kw)
    big = [t.repeat(reps, 1, 1, 1) for t in (q, k, v, o)]
    outs = [torch.full((reps * B, N, H, d), float("nan"), device=dev) for _ in range(3)]
    fastvr.chunk_attn_bwd(*big, lse.repeat(reps, 1, 1), do.repeat(reps, 1, 1, 1), dq=outs[0], dk=outs[1], dv=outs[2], **kw)
    torch.cuda.synchronize()
    for n, g, r in zip(("dq", "dk", "dv"), outs, ref):
        assert r.abs().max() > 0 and torch.equal(g.view(reps, B, N, H, d), r.expand(reps, B, N, H, d)), n


def test_streaming_chunk_past_4gib(dev):
    """256-row items (256 in all, one per CU) far from the tensors' base: the
    query chunk is the last of 258 chunks of 32768 tokens, W = 1, so the key rows it
    sees start 2.15 GB (batch 0) and 4.31 GB (batch 1) from the base of k and v.
    Every other key row is NaN."""
    B, d, L, n_chunks, W = 2, 128, 32768, 258, 1
    N, lo = n_chunks * L, (n_chunks - 2) * L
    _announce(f"far streaming chunk B={B} H=1 d={d} Nkv={N} L={L} offset={n_chunks - 1} W={W}")
    q, kc, vc = make_qkv(B, L, 2 * L, 1, d, seed=905)
    kv = []
    for t in (kc, vc):
        far = torch.full((B, N, 1, d), float("nan"), dtype=torch.bfloat16, device=dev)
        far[:, lo:] = t.to(dev)
        kv.append(far)
    o, lse = fastvr.chunk_attn(q.to(dev), *kv, chunk_len=L, q_chunk_offset=n_chunks - 1, window_chunks=W)
    torch.cuda.synchronize()
    rows = sample_rows(L, L, n_random=16, seed=5, band=0)
    ridx = torch.as_tensor(rows, device=dev)
    # the same mask on the compact key range: the two visible chunks
    o_ref, l_ref = run_oracle(q, kc, vc, L, 1, W, default_scale(d), rows=rows)
    compare(to_np(o[:, ridx]), to_np(lse[:, :, ridx]), o_ref, l_ref, label=f"full items far chunk ({len(rows)} rows)")
