"""Lower against 256-row items of the forward, bit for bit: a small call runs
128-row items (160 to 224 rows where those would need a second wave), the same
tensors repeated as a large batch 256-row ones (tests/fwd_plan_check.cpp checks
the plans).  Odd chunk lengths leave ragged
tiles in both heights and a ragged last key tile; interval lengths are even and
odd numbers of key tiles.  One case of each is also held against the oracle."""
import numpy as np
import pytest
import torch

from paper_2609_36757_amd import fastvr
from paper_2609_36757_amd.workloads import make_qkv

from parity import compare, run_oracle, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fastvr.load()
    return torch.device("cuda:0")


@pytest.mark.parametrize("d,scale,L,N,off,W,reps", [
    (64, 0.125, 259, 900, 0, -1, 128), (128, 1 / np.sqrt(128), 259, 900, 0, -1, 128),
    (64, -0.2, 259, 900, 0, -1, 128), (128, -0.08, 259, 900, 0, -1, 128),
    (128, 1 / np.sqrt(128), 259, 259, 1, 1, 256), (64, 0.125, 259, 259, 1, 1, 256)])
def test_half_items_equal_full_items(dev, d, scale, L, N, off, W, reps):
    H, nkv = 2, off * L + N
    print(f"\n[gpu case] half items: H={H} d={d} N={N} Nkv={nkv} L={L} off={off} W={W} scale={scale:.3f}", flush=True)
    q, k, v = make_qkv(1, N, nkv, H, d, seed=600 + d + off)
    kw = dict(chunk_len=L, q_chunk_offset=off, window_chunks=W, scale=scale)
    small = [t.to(dev) for t in (q, k, v)]
    o, lse = fastvr.chunk_attn(*small, **kw)
    big_o, big_l = fastvr.chunk_attn(*(t.expand(reps, *t.shape[1:]).contiguous() for t in small), **kw)
    ob = torch.empty_like(o, dtype=torch.bfloat16)
    fastvr.chunk_attn(*small, out=ob, return_lse=False, **kw)
    torch.cuda.synchronize()
    assert torch.equal(o.expand_as(big_o), big_o) and torch.equal(lse.expand_as(big_l), big_l)
    assert torch.equal(ob, o.to(torch.bfloat16))
    o_ref, l_ref = run_oracle(q, k, v, L, off, W, scale)
    compare(to_np(o), to_np(lse), o_ref, l_ref, label=f"half items d={d} scale={scale:.3f} off={off}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bh", [80, 62, 50])
def test_low_items_equal_full_items(dev, d, bh):
    """224, 192 and 160 rows (bh = 80, 62, 50) over one ragged chunk of 650 rows."""
    L, off, H = 650, 1, 2
    print(f"\n[gpu case] low items: B={bh // H} H={H} d={d} L={L} off={off}", flush=True)
    q, k, v = make_qkv(1, L, (off + 1) * L, H, d, seed=700 + d)
    small = [t.to(dev) for t in (q, k, v)]
    outs = []
    for reps in (bh // H, 256):
        x = [t.expand(reps, *t.shape[1:]).contiguous() for t in small]
        outs.append(fastvr.chunk_attn(*x, chunk_len=L, q_chunk_offset=off))
    torch.cuda.synchronize()
    for a, b in zip(*outs):
        assert torch.equal(a[:1].expand_as(a), a) and torch.equal(a[:1].expand_as(b), b)
    o_ref, l_ref = run_oracle(q, k, v, L, off, -1, 1 / np.sqrt(d))
    compare(to_np(outs[0][0][:1]), to_np(outs[0][1][:1]), o_ref, l_ref, label=f"low items d={d} bh={bh}")


@pytest.mark.parametrize("d,scale", [(64, 0.125), (64, -0.2), (128, 1 / np.sqrt(128)), (128, -0.08)])
@pytest.mark.parametrize("bh", [80, 62, 50])
def test_low_items_strided_bf16(dev, bh, d, scale):
    """The same heights on views of a cache whose rows past the filled ones are NaN,
    a strided q, O as bf16 into a strided view, and both signs of the scale."""
    L, off, H, cap = 650, 1, 2, 1400
    n = (off + 1) * L
    print(f"\n[gpu case] low items strided: B={bh // H} H={H} d={d} L={L} off={off} scale={scale:.3f}", flush=True)
    q, k, v = make_qkv(1, L, n, H, d, seed=720 + d)
    kw = dict(chunk_len=L, q_chunk_offset=off, scale=scale)
    outs = []
    for reps in (bh // H, 256):
        views = []
        for t in (q, k, v):
            buf = torch.full((reps, cap, H, d), float("nan"), dtype=torch.bfloat16, device=dev)
            buf[:, :t.shape[1]] = t.to(dev)
            views.append(buf[:, :t.shape[1]])
        big = torch.full((reps, L + 9, H, d), float("nan"), dtype=torch.bfloat16, device=dev)
        o, lse = fastvr.chunk_attn(*views, **kw)
        _, lse_b = fastvr.chunk_attn(*views, out=big[:, 3:3 + L], **kw)
        torch.cuda.synchronize()
        assert torch.equal(big[:, 3:3 + L], o.to(torch.bfloat16)) and torch.equal(lse_b, lse)
        assert torch.isnan(big[:, :3].float()).all() and torch.isnan(big[:, 3 + L:].float()).all()
        outs.append((o, lse))
    for a, b in zip(*outs):
        assert torch.equal(a[:1].expand_as(a), a) and torch.equal(a[:1].expand_as(b), b)
    o_ref, l_ref = run_oracle(q, k, v, L, off, -1, scale)
    compare(to_np(outs[0][0][:1]), to_np(outs[0][1][:1]), o_ref, l_ref, label=f"low items strided d={d} bh={bh}")


@pytest.mark.parametrize("d,scale", [(64, -0.2), (128, 1 / np.sqrt(128))])
@pytest.mark.parametrize("bh", [80, 62, 50])
def test_low_items_ring_step(dev, bh, d, scale):
    """The ring step at these heights, whose workgroups share the append: outputs and
    ring against a large batch (256-row items), the replaced slot NaN before."""
    H, L, W, c, n_new = 2, 656, 1, 3, 650
    print(f"\n[gpu case] low items ring: B={bh // H} H={H} d={d} L={L} W={W} n_new={n_new}", flush=True)
    q, k, v = (t.to(dev) for t in make_qkv(1, n_new, n_new, H, d, seed=740 + d))
    _, rk, rv = (t.to(dev) for t in make_qkv(1, 1, (W + 1) * L, H, d, seed=741 + d))
    slot = c % (W + 1) * L
    rk[:, slot:slot + L] = float("nan")
    rv[:, slot:slot + L] = float("nan")
    outs = []
    for reps in (bh // H, 256):
        args = [t.expand(reps, *t.shape[1:]).contiguous() for t in (q, k, v, rk, rv)]
        o, lse = fastvr.chunk_attn_ring_step(*args, chunk_len=L, chunk_index=c, window_chunks=W, scale=scale)
        torch.cuda.synchronize()
        for ring, old, new in ((args[3], rk, k), (args[4], rv, v)):
            want = old.clone()
            want[:, slot:slot + n_new] = new
            assert torch.equal(ring.view(torch.int16), want.view(torch.int16).expand(reps, *ring.shape[1:]))
        outs.append((o, lse))
    for a, b in zip(*outs):
        assert torch.equal(a[:1].expand_as(a), a) and torch.equal(a[:1].expand_as(b), b)
    prev = slice(L - slot, 2 * L - slot)  # the other slot holds chunk c - 1
    kf, vf = (torch.cat([r[:, prev], t], dim=1).cpu() for r, t in ((rk, k), (rv, v)))
    o_ref, l_ref = run_oracle(q.cpu(), kf, vf, L, 1, W, scale)
    compare(to_np(outs[0][0][:1]), to_np(outs[0][1][:1]), o_ref, l_ref, label=f"low items ring d={d} bh={bh}")


@pytest.mark.parametrize("d,L", [(128, 260), (64, 264)])
def test_half_items_ring_step(dev, d, L):
    """The ring step with 128-row items, whose key tiles straddle two slots, against
    the same step over a large batch (256-row items): outputs and ring."""
    H, W, c, n_new, reps = 2, 1, 3, 200, 256
    print(f"\n[gpu case] half items ring: H={H} d={d} L={L} W={W} c={c} n_new={n_new}", flush=True)
    q, k, v = (t.to(dev) for t in make_qkv(1, n_new, n_new, H, d, seed=640 + d))
    _, rk, rv = (t.to(dev) for t in make_qkv(1, 1, (W + 1) * L, H, d, seed=641 + d))
    outs = []
    for r in (1, reps):
        args = [t.expand(r, *t.shape[1:]).contiguous() for t in (q, k, v, rk, rv)]
        o, lse = fastvr.chunk_attn_ring_step(*args, chunk_len=L, chunk_index=c, window_chunks=W)
        outs.append((o, lse, args[3], args[4]))
    torch.cuda.synchronize()
    for a, b in zip(*outs):
        assert torch.equal(a.expand_as(b), b)
