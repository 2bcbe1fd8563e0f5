"""Measured cases: the calls a user of this library makes, through its Python
entry points, from the smallest to the largest shapes of the repository's own
workloads (``paper_2609_36757_amd/workloads.py``, ``bench.py``).

A case is a dict of plain values.  ``kind`` says which call it is:

* ``attn``      chunk-causal attention of a whole sequence (training, or offline restoration);
* ``stream``    KV-cache append of a new chunk, then its attention over the cached prefix;
* ``ring``      one streaming step with the bounded ring cache (append fused);
* ``bwd``       the gradients of an ``attn`` call;
* ``gather``    spatial tiles of a token field;
* ``blend``     weight-normalised blend of per-tile results, plain or fused with the one-step update;
* ``one_step``  the one-step latent update of a whole latent.
"""
from __future__ import annotations

import math

import torch

from paper_2609_36757_amd import fastvr

MAX_FLOPS = 1.64e13   # the 1080p sequence's forward, the largest listed case
MAX_BYTES = 2.0e9     # the largest field of the memory-bound calls


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def _attn(name, B, H, d, L, n, W, packed=False, bf16_out=False):
    return dict(name=name, kind="attn", B=B, H=H, d=d, L=L, n=n, W=W, packed=packed, bf16_out=bf16_out)


def listed():
    return [
        # smallest call: 4 chunks of 256 tokens, head_dim 64; latency and launch count
        _attn("attn_tiny", 1, 2, 64, 256, 1024, -1),
        # a 480p clip at once: 30 x 52 tokens a frame, 2 frames a chunk, 6 chunks, full causal prefix
        _attn("attn_480p", 1, 12, 128, 3120, 18720, -1),
        # the 1080p sequence at once: 68 x 120 tokens a frame, 4 chunks (the largest call)
        _attn("attn_1080p", 1, 12, 128, 16320, 65280, -1),
        # a batch of small odd crops as views of one packed QKV projection, bf16 output, head_dim 64, ragged tail
        _attn("attn_crops_d64", 2, 8, 64, 1365, 5003, 2, packed=True, bf16_out=True),
        # streaming 480p: chunk 3 is appended to the cache and attends to chunks 0..3
        dict(name="stream_480p", kind="stream", B=1, H=12, d=128, L=3120, c=3, n_new=3120, cap=18720),
        # streaming 1080p in the paper's setting (a chunk and its predecessor, bounded cache)
        dict(name="ring_1080p_w1", kind="ring", B=1, H=12, d=128, L=16320, c=3, n_new=16320, W=1),
        # gradients of the smallest call, with the library's own workspace
        dict(name="bwd_tiny", kind="bwd", B=1, H=2, d=64, L=256, n=1024, W=-1, noalloc=True),
        # training on 480p clips
        dict(name="bwd_480p", kind="bwd", B=1, H=12, d=128, L=3120, n=18720, W=-1, noalloc=False),
        # training on 1024 x 1024 clips of 45 frames: 64 x 64 tokens a frame, 3 frames a chunk, W = 1
        dict(name="bwd_clip1024", kind="bwd", B=1, H=12, d=128, L=12288, n=49152, W=1, noalloc=False),
        # tiled 1080p inference: one projection's tokens cut into overlapping 64 x 64 tiles
        dict(name="gather_1080p", kind="gather", B=1, T=8, Hg=68, Wg=120, C=1536, tile=64, overlap=16),
        # tiled 1080p inference: the velocity tiles blended and applied to the 48-channel latent
        dict(name="blend_latent_1080p", kind="blend", B=1, T=8, Hg=68, Wg=120, C=48, tile=64, overlap=16, update=True),
        # untiled inference: the update of the whole 1080p latent
        dict(name="one_step_1080p", kind="one_step", n=48 * 8 * 68 * 120, bf16_out=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: crops of 64 tokens a chunk up to 1080p chunks,
    1 to 8 chunks with a ragged tail, 2 to 24 heads, both head dims, all windows."""
    while True:
        kind = rng.choice(["attn", "attn", "attn", "stream", "ring", "bwd", "bwd", "bwd", "gather", "blend", "one_step"])
        if kind in ("attn", "stream", "ring", "bwd"):
            B, H, d = rng.choice([1, 1, 2]), rng.choice([2, 4, 8, 12, 16, 24]), rng.choice([64, 128, 128])
            L = _log_int(rng, 64, 16320)
            W = rng.choice([-1, -1, 1, 2])
            chunks = rng.randint(1, 8)
            tail = L if rng.random() < 0.5 else rng.randint(1, L)
            if kind == "attn":
                case = dict(kind=kind, B=B, H=H, d=d, L=L, n=(chunks - 1) * L + tail, W=W,
                            packed=rng.random() < 0.3, bf16_out=rng.random() < 0.3)
            elif kind == "bwd":
                case = dict(kind=kind, B=B, H=H, d=d, L=L, n=(chunks - 1) * L + tail, W=W, noalloc=rng.random() < 0.3)
                if 2 * B * H * case["n"] > (1 << 23):
                    case["noalloc"] = False
            elif kind == "stream":
                case = dict(kind=kind, B=B, H=H, d=d, L=L, c=chunks - 1, n_new=tail, cap=chunks * L + rng.choice([0, 64]))
            else:
                L = max(64, L // 8 * 8)
                case = dict(kind=kind, B=B, H=H, d=d, L=L, c=chunks - 1, n_new=min(tail, L), W=rng.choice([1, 1, 2, 3]))
        elif kind == "one_step":
            case = dict(kind=kind, n=_log_int(rng, 1 << 14, 1 << 26) + rng.randint(0, 7), bf16_out=rng.random() < 0.5)
        else:
            update = kind == "blend" and rng.random() < 0.5
            case = dict(kind=kind, B=rng.choice([1, 1, 2]), T=rng.randint(1, 12), Hg=_log_int(rng, 20, 140),
                        Wg=_log_int(rng, 20, 250), C=rng.choice([16, 48]) if update else rng.choice([256, 768, 1536]),
                        tile=rng.choice([32, 64]), overlap=rng.choice([8, 16]))
            if kind == "blend":
                case["update"] = update
        w = work(case)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return case


# ---------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------

def _intervals(case):
    """(first query row, end, first key row, end) of every query chunk of the call;
    key rows count from the first row of the sequence."""
    L = case["L"]
    if case["kind"] in ("attn", "bwd"):
        n, W = case["n"], case["W"]
        return [(c * L, min((c + 1) * L, n), max(0, c - W) * L if W >= 0 else 0, min((c + 1) * L, n))
                for c in range(-(-n // L))]
    c, n_new = case["c"], case["n_new"]
    lo = max(0, c - case["W"]) * L if case["kind"] == "ring" else 0
    return [(0, n_new, lo, c * L + n_new)]


def _tiles(case):
    ny, Ly = fastvr.tile_axis(case["Hg"], case["tile"], case["overlap"])
    nx, Lx = fastvr.tile_axis(case["Wg"], case["tile"], case["overlap"])
    return ny, Ly, nx, Lx


def work(case):
    kind = case["kind"]
    if kind == "one_step":
        return {"bytes": case["n"] * (4 + (2 if case["bf16_out"] else 4)), "flops": 2 * case["n"]}
    if kind in ("gather", "blend"):
        ny, Ly, nx, Lx = _tiles(case)
        field = case["B"] * case["T"] * case["Hg"] * case["Wg"] * case["C"]
        tiles = case["B"] * ny * nx * case["T"] * Ly * Lx * case["C"]
        if kind == "gather":
            return {"bytes": 2 * (field + tiles), "flops": 0}
        return {"bytes": 4 * (field + tiles) + (2 * field if case["update"] else 0), "flops": 2 * tiles + field}
    hd = case["H"] * case["d"]
    iv = _intervals(case)
    pairs = sum((b - a) * (e - s) for a, b, s, e in iv) * case["B"] * case["H"]
    nq = sum(b - a for a, b, _, _ in iv) * case["B"]
    nk = (max(e for _, _, _, e in iv) - min(s for _, _, s, _ in iv)) * case["B"]
    if kind == "bwd":
        # q, dO, dq and o of every query row, k, v, dk, dv of every key row, the LSE
        return {"bytes": nq * (hd * (2 + 2 + 4 + 4) + 4 * case["H"]) + nk * hd * (2 + 2 + 4 + 4),
                "flops": 10 * case["d"] * pairs}
    out = 2 if case.get("bf16_out") else 4
    extra = 4 * case["n_new"] * case["B"] * hd if kind in ("stream", "ring") else 0  # the cache rows written
    return {"bytes": nq * (hd * (2 + out) + 4 * case["H"]) + nk * hd * 4 + extra, "flops": 4 * case["d"] * pairs}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _randn(shape, g):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _qkv(B, n, H, d, g):
    """N(0, 1) queries and values; keys with a mean of their own per head, as trained projections have."""
    q = _randn((B, n, H, d), g).to(torch.bfloat16)
    k = (_randn((B, n, H, d), g) + 0.5 * _randn((H, d), g)).to(torch.bfloat16)
    v = _randn((B, n, H, d), g).to(torch.bfloat16)
    return q, k, v


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    st = {"case": case}
    if kind == "one_step":
        st["z"] = _randn((case["n"],), g).to(torch.bfloat16)
        st["v"] = _randn((case["n"],), g).to(torch.bfloat16)
        return st
    if kind in ("gather", "blend"):
        B, T, Hg, Wg, C = (case[x] for x in ("B", "T", "Hg", "Wg", "C"))
        if kind == "gather":
            st["x"] = _randn((B, T, Hg, Wg, C), g).to(torch.bfloat16)
        else:
            ny, Ly, nx, Lx = _tiles(case)
            st["tiles"] = _randn((B, ny * nx, T, Ly, Lx, C), g)
            if case["update"]:
                st["z"] = _randn((B, T, Hg, Wg, C), g).to(torch.bfloat16)
        return st
    B, H, d, L = case["B"], case["H"], case["d"], case["L"]
    if kind in ("attn", "bwd"):
        n = case["n"]
        q, k, v = _qkv(B, n, H, d, g)
        if kind == "attn":
            if case["packed"]:
                qkv = torch.stack((q, k, v), dim=2)  # [B, n, 3, H, d], one projection's output
                q, k, v = qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2]
            st.update(q=q, k=k, v=v)
        else:
            o, lse = fastvr.chunk_attn(q, k, v, chunk_len=L, window_chunks=case["W"])
            st.update(q=q, k=k, v=v, o=o, lse=lse, dout=_randn((B, n, H, d), g).to(torch.bfloat16))
            if case["noalloc"]:
                st["grads"] = [torch.empty((B, n, H, d), device="cuda", dtype=torch.float32) for _ in range(3)]
        return st
    c, n_new = case["c"], case["n_new"]
    q, k, v = _qkv(B, c * L + n_new, H, d, g)
    st["q"], st["k"], st["v"] = (x[:, c * L:].contiguous() for x in (q, k, v))
    if kind == "stream":
        st["kc"], st["vc"] = (torch.zeros((B, case["cap"], H, d), device="cuda", dtype=torch.bfloat16) for _ in range(2))
        st["kc"][:, :c * L], st["vc"][:, :c * L] = k[:, :c * L], v[:, :c * L]
    else:
        S = case["W"] + 1
        st["kr"], st["vr"] = (torch.zeros((B, S * L, H, d), device="cuda", dtype=torch.bfloat16) for _ in range(2))
        for s in range(max(0, c - case["W"]), c):
            st["kr"][:, s % S * L:(s % S + 1) * L] = k[:, s * L:(s + 1) * L]
            st["vr"][:, s % S * L:(s % S + 1) * L] = v[:, s * L:(s + 1) * L]
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

SIGMA = 0.7


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "attn":
        q = st["q"]
        out = torch.empty(q.shape, dtype=torch.bfloat16, device=q.device) if case["bf16_out"] else None
        return fastvr.chunk_attn(q, st["k"], st["v"], chunk_len=case["L"], window_chunks=case["W"], out=out)
    if kind == "stream":
        c, L = case["c"], case["L"]
        n = fastvr.kv_cache_append(st["kc"], st["vc"], st["k"], st["v"], c * L)
        o, lse = fastvr.chunk_attn(st["q"], st["kc"][:, :n], st["vc"][:, :n], chunk_len=L, q_chunk_offset=c)
        return o, lse, st["kc"], st["vc"]
    if kind == "ring":
        o, lse = fastvr.chunk_attn_ring_step(st["q"], st["k"], st["v"], st["kr"], st["vr"], chunk_len=case["L"],
                                             chunk_index=case["c"], window_chunks=case["W"])
        return o, lse, st["kr"], st["vr"]
    if kind == "bwd":
        args = (st["q"], st["k"], st["v"], st["o"], st["lse"], st["dout"])
        if case["noalloc"]:
            return fastvr.chunk_attn_bwd_noalloc(*args, *st["grads"], chunk_len=case["L"], window_chunks=case["W"])
        return fastvr.chunk_attn_bwd(*args, chunk_len=case["L"], window_chunks=case["W"])
    if kind == "gather":
        return fastvr.tile_gather(st["x"], tile=case["tile"], overlap=case["overlap"])
    if kind == "blend":
        return fastvr.tile_blend(st["tiles"], case["Hg"], case["Wg"], tile=case["tile"], overlap=case["overlap"],
                                 z_lq=st.get("z"), sigma=SIGMA)
    return fastvr.one_step_update(st["z"], st["v"], SIGMA, out_dtype=torch.bfloat16 if case["bf16_out"] else None)


def tolerance(case):
    # attention: P (and dS) are rounded to bf16 for the matrix cores; measured against 64 bits 1.4e-3 to 2.2e-3
    # (outputs; 2.3e-3 when stored as bf16) and 1.7e-3 to 2.4e-3 (gradients), four times that between two orders.
    # blend: 32-bit sums over at most 9 tiles (3e-8 measured; a weighted sum may round at every term).
    # The update of a bf16 latent in 32 bits is one correctly rounded step.
    kind = case["kind"]
    if kind == "gather" or kind == "one_step":
        return "exact"
    if kind == "blend":
        return {"rel": 5e-7}
    return {"rel": 1e-2}


# ---------------------------------------------------------------------------
# 64-bit results
# ---------------------------------------------------------------------------

def _scale(d):
    return float(torch.tensor(1.0 / math.sqrt(d), dtype=torch.float32))


def _softmax_rows(q, k, scale):
    s = (q @ k.t()) * scale
    lse = torch.logsumexp(s, dim=1)
    return s.sub_(lse[:, None]).exp_(), lse


def _exact_attn(q, k, v, rows, scale):
    """rows: list of (q rows a..b, key rows s..e); block by block in float64."""
    B, nq, H, d = q.shape
    o = torch.empty((B, nq, H, d), dtype=torch.float64, device=q.device)
    lse = torch.empty((B, H, nq), dtype=torch.float64, device=q.device)
    for b in range(B):
        for h in range(H):
            for a, e, s, t in rows:
                kk, vv = k[b, s:t, h].double().contiguous(), v[b, s:t, h].double().contiguous()
                for i in range(a, e, 2048):
                    j = min(e, i + 2048)
                    p, l = _softmax_rows(q[b, i:j, h].double().contiguous(), kk, scale)
                    o[b, i:j, h], lse[b, h, i:j] = p @ vv, l
    return o, lse


def _exact_bwd(q, k, v, dout, rows, scale):
    dq, dk, dv = (torch.zeros(x.shape, dtype=torch.float64, device=q.device) for x in (q, k, v))
    B, _, H, _ = q.shape
    for b in range(B):
        for h in range(H):
            for a, e, s, t in rows:
                kk, vv = k[b, s:t, h].double().contiguous(), v[b, s:t, h].double().contiguous()
                for i in range(a, e, 2048):
                    j = min(e, i + 2048)
                    qq, do = q[b, i:j, h].double().contiguous(), dout[b, i:j, h].double().contiguous()
                    p, _ = _softmax_rows(qq, kk, scale)
                    dv[b, s:t, h] += p.t() @ do
                    ds = do @ vv.t()
                    ds -= ((p @ vv) * do).sum(1, keepdim=True)
                    ds *= p
                    dq[b, i:j, h] = (ds @ kk) * scale
                    dk[b, s:t, h] += (ds.t() @ qq) * scale
    return dq, dk, dv


def _exact_blend(st):
    case = st["case"]
    ny, Ly, nx, Lx = _tiles(case)
    B, T, Hg, Wg, C = (case[x] for x in ("B", "T", "Hg", "Wg", "C"))
    R = max(case["overlap"], 1)

    def axis(n, L, size):
        org = [0 if n == 1 else (k * (size - L) + (n - 1) // 2) // (n - 1) for k in range(n)]
        return org, torch.tensor([min(i + 1, L - i, R) for i in range(L)], dtype=torch.float64, device="cuda")

    oy, wy = axis(ny, Ly, Hg)
    ox, wx = axis(nx, Lx, Wg)
    acc = torch.zeros((B, T, Hg, Wg, C), dtype=torch.float64, device="cuda")
    wsum = torch.zeros((Hg, Wg, 1), dtype=torch.float64, device="cuda")
    w = (wy[:, None] * wx[None, :])[..., None]
    for ty, y in enumerate(oy):
        for tx, x in enumerate(ox):
            acc[:, :, y:y + Ly, x:x + Lx] += st["tiles"][:, ty * nx + tx].double() * w
            wsum[y:y + Ly, x:x + Lx] += w
    acc /= wsum
    if case["update"]:
        acc = st["z"].double() - float(torch.tensor(SIGMA, dtype=torch.float32)) * acc
    return acc


def exact(case, seed):
    kind = case["kind"]
    if kind == "gather":
        return None
    if kind != "blend" and kind != "one_step" and work(case)["flops"] > 5e12:
        return None  # over about 20 seconds in 64 bits
    st = prepare(case, seed)
    if kind == "one_step":
        return st["z"].double() - float(torch.tensor(SIGMA, dtype=torch.float32)) * st["v"].double()
    if kind == "blend":
        return _exact_blend(st)
    scale = _scale(case["d"])
    if kind == "attn":
        return _exact_attn(st["q"], st["k"], st["v"], _intervals(case), scale)
    if kind == "bwd":
        return _exact_bwd(st["q"], st["k"], st["v"], st["dout"], _intervals(case), scale)
    c, L, n_new = case["c"], case["L"], case["n_new"]
    if kind == "stream":
        kc, vc = st["kc"].clone(), st["vc"].clone()
        kc[:, c * L:c * L + n_new], vc[:, c * L:c * L + n_new] = st["k"], st["v"]
        o, lse = _exact_attn(st["q"], kc, vc, [(0, n_new, 0, c * L + n_new)], scale)
        return o, lse, kc.double(), vc.double()
    S = case["W"] + 1
    first = max(0, c - case["W"])
    k = torch.cat([st["kr"][:, s % S * L:(s % S + 1) * L] for s in range(first, c)] + [st["k"]], dim=1)
    v = torch.cat([st["vr"][:, s % S * L:(s % S + 1) * L] for s in range(first, c)] + [st["v"]], dim=1)
    o, lse = _exact_attn(st["q"], k, v, [(0, n_new, 0, k.shape[1])], scale)
    kr, vr = st["kr"].clone(), st["vr"].clone()
    kr[:, c % S * L:c % S * L + n_new], vr[:, c % S * L:c % S * L + n_new] = st["k"], st["v"]
    return o, lse, kr.double(), vr.double()
