"""Workloads by which a change to this library is timed and checked.

Each case is one pass through the public entry points as an inference program calls them: the
tensors, the weights and every output buffer exist before the call (the library allocates
nothing), the pass enqueues its launches on the current stream and returns the buffers.

Inputs follow the distribution of the package's structured workloads: a per-slot, per-head
pattern shared by all frames plus per-frame noise, with queries that match the keys' pattern.
Token geometry is that of the package's workloads (37 x 37 patches + 5 special tokens, 16 heads
of 64) and of the paper's tables (28 x 37 patches), at 2 to 800 frames, and a 16 x 16 grid for the
smallest calls; other grids and head counts are generic.
"""
from __future__ import annotations

import math

import torch

from paper_2512_02541_amd import binding as agg
from paper_2512_02541_amd import harness, inputs

HEAD_DIM = 64
STRIDES = ((1, 2), (2, 2), (2, 3), (3, 3))  # sigma = 2, 4, 6, 9


def _case(kind, N, grid, strides=(2, 2), H=16, B=1, n_special=5, keep_first=1, name=None):
    c = {"kind": kind, "B": B, "N": N, "n_h": grid[0], "n_w": grid[1], "n_special": n_special,
         "H": H, "s_h": strides[0], "s_w": strides[1], "keep_first": keep_first}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: two small frames; launches and latency are all there is
        _case("layer", 2, (16, 16), (2, 2), name="layer_2f_16x16"),
        # a short clip (the paper's 10-frame setting): a few hundred workgroups
        _case("layer", 10, (37, 37), (1, 2), name="layer_10f"),
        # the everyday case of the paper and of the benchmark: one subsampled layer, 100 frames
        _case("layer", 100, (37, 37), (1, 2), name="layer_100f"),
        # the longest sequence of the paper's tables
        _case("layer", 800, (37, 37), (3, 3), name="layer_800f"),
        # the key/value pass alone over a long sequence, as a program that overlaps it calls it
        _case("subsample", 300, (37, 37), (2, 2), name="subsample_300f"),
        # attention through the index list, without compacted copies, all frames subsampled
        _case("indexed", 40, (37, 37), (2, 2), keep_first=0, name="indexed_40f"),
        # kept tokens chosen by magnitude (selection, list-driven pass, list-driven attention)
        _case("list", 60, (37, 37), (2, 2), name="list_60f"),
        # ordinary global attention, the baseline, on the wide grid and twelve heads
        _case("dense", 24, (28, 37), H=12, name="dense_24f_12h"),
        # an early global block's attention after its conversion to per-frame attention
        _case("frame", 90, (37, 37), name="frame_90f"),
        # whole blocks: projections and LayerNorm around per-frame attention, a long clip
        _case("block_frame", 100, (37, 37), name="block_frame_100f"),
        # ... around subsampled attention, a short clip
        _case("block_sga", 16, (37, 37), (2, 2), name="block_sga_16f"),
        # ... and the smallest whole block
        _case("block_sga", 2, (16, 16), (2, 2), name="block_sga_2f_16x16"),
    ]


# share of drawn cases and longest sequence (frames) of each kind
KINDS = (("layer", 0.34, 800), ("subsample", 0.08, 800), ("indexed", 0.08, 300), ("list", 0.08, 300),
         ("dense", 0.10, 150), ("frame", 0.12, 500), ("block_frame", 0.10, 333),
         ("block_sga", 0.10, 200))


def draw(rng):
    most = max(work(c)["flops"] for c in listed())
    while True:
        pick = rng.random()
        for kind, share, longest in KINDS:
            pick -= share
            if pick < 0:
                break
        N = int(round(2 ** rng.uniform(0.0, math.log2(longest))))
        grid = rng.choice(((37, 37), (37, 37), (28, 37), (16, 16),
                           (rng.randint(9, 40), rng.randint(9, 40))))
        # per-frame and whole-kept calls of one frame are ordinary; a subsampled one keeps none whole
        c = _case(kind, N, grid, rng.choice(STRIDES), H=rng.choice((16, 16, 16, 8, 12, 20)),
                  B=rng.choice((1, 1, 1, 2)), n_special=rng.choice((5, 5, 1)),
                  keep_first=rng.choice((1, 1, 0)) if N > 1 else 0)
        if work(c)["flops"] <= most:
            return c


def _shape(c):
    return agg.make_shape(c["B"], c["N"], c["n_h"], c["n_w"], c["n_special"], c["H"], HEAD_DIM,
                          c["s_h"], c["s_w"], c["keep_first"])


def _counts(c):
    """tokens per sequence, kept rows, dropped patches"""
    patches = c["n_h"] * c["n_w"]
    kept = -(-c["n_h"] // c["s_h"]) * -(-c["n_w"] // c["s_w"])
    sub = c["N"] - c["keep_first"]
    nq = c["N"] * (patches + c["n_special"])
    return nq, nq - sub * (patches - kept), sub * (patches - kept)


def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)


def _qkv(c, seed):
    B, N, H = c["B"], c["N"], c["H"]
    L = c["n_h"] * c["n_w"] + c["n_special"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    a_k, a_v = _normal(gen, L, H, HEAD_DIM), _normal(gen, L, H, HEAD_DIM)
    out = []
    for pattern in (a_k, a_k, a_v):
        t = torch.empty((B * N, L, H, HEAD_DIM), dtype=torch.bfloat16, device="cuda")
        for f in range(0, B * N, 64):
            n = min(64, B * N - f)
            t[f:f + n] = pattern + 0.5 * _normal(gen, n, L, H, HEAD_DIM)
        out.append(t.view(B, N * L, H, HEAD_DIM))
    return out


def _block_input(c, seed):
    nq, _, _ = _counts(c)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((c["B"], nq, c["H"] * HEAD_DIM), generator=gen, device="cuda",
                       dtype=torch.float32).to(torch.bfloat16)


def prepare(case, seed):
    c, kind = case, case["kind"]
    shape = _shape(c)
    st = {"kind": kind, "shape": shape}
    if kind in ("block_frame", "block_sga"):
        mode = agg.AGG_BLOCK_FRAME if kind == "block_frame" else agg.AGG_BLOCK_SGA
        x = _block_input(c, seed)
        w = inputs.block_weights(c["H"] * HEAD_DIM, seed, "cuda")
        packed = agg.make_block_weights(w["ln_gamma"], w["ln_beta"], w["ln_eps"], w["w_q"], w["w_k"],
                                        w["w_v"], w["w_o"], w["b_q"], w["b_k"], w["b_v"], w["b_o"])
        ws = torch.empty(agg.agg_block_workspace_bytes(shape, mode), dtype=torch.uint8, device="cuda")
        st.update(mode=mode, x=x, weights=w, packed=packed, ws=ws, y=torch.empty_like(x))
        return st
    q, k, v = _qkv(c, seed)
    st.update(q=q, k=k, v=v)
    B, H, nq = c["B"], c["H"], q.shape[1]
    if kind in ("layer", "subsample", "indexed"):
        st["buf"] = harness.alloc(shape, "cuda")
        return st
    st["O"] = torch.empty_like(q)
    # a frame's rows are contiguous in lse as [B*N, H, L]; the other calls give [B, H, N*L]
    st["lse"] = torch.empty((B * c["N"], H, nq // c["N"]) if kind == "frame" else (B, H, nq),
                            dtype=torch.float32, device="cuda")
    if kind == "list":
        m, _ = agg.agg_kv_count(shape)
        nbytes, _ = agg.agg_list_compact_bytes(shape, m)
        st.update(
            m=m, list=torch.empty((B, m), dtype=torch.int32, device="cuda"),
            Kc=torch.empty(nbytes // 2, dtype=torch.bfloat16, device="cuda"),
            Vc=torch.empty(nbytes // 2, dtype=torch.bfloat16, device="cuda"),
            kmean=torch.empty((B, H, HEAD_DIM), dtype=torch.float32, device="cuda"),
            vmean=torch.empty((B, H, HEAD_DIM), dtype=torch.float32, device="cuda"),
            bits=torch.empty((B, (nq + 31) // 32), dtype=torch.int32, device="cuda"),
            dropped=torch.empty((B,), dtype=torch.int32, device="cuda"),
            ws=torch.empty(agg.agg_list_workspace_bytes(shape), dtype=torch.uint8, device="cuda"))
    return st


def run(state):
    s, kind, shape = state, state["kind"], state["shape"]
    if kind in ("block_frame", "block_sga"):
        agg.agg_global_block_fwd(shape, s["mode"], s["packed"], s["x"], s["y"], s["ws"], s["ws"].numel())
        return {"y": s["y"]}
    q, k, v = s["q"], s["k"], s["v"]
    if kind == "layer":
        b = s["buf"]
        harness.subsample(b, k, v)
        harness.attend(b, q, k, v)
        return {"O": b.O, "lse": b.lse, "idx": b.idx, "kmean": b.kmean, "vmean": b.vmean}
    if kind == "subsample":
        b = s["buf"]
        harness.subsample(b, k, v)
        return {"idx": b.idx, "Kc": b.Kc, "Vc": b.Vc, "kmean": b.kmean, "vmean": b.vmean}
    if kind == "indexed":
        b = s["buf"]
        agg.agg_kv_subsample(shape, k, v, None, None, b.idx, b.kmean, b.vmean, b.workspace,
                             b.workspace.numel())
        harness.attend_idx(b, q, k, v)
        return {"O": b.O, "lse": b.lse, "idx": b.idx, "kmean": b.kmean, "vmean": b.vmean}
    if kind == "list":
        agg.agg_select_kv_indices(shape, agg.AGG_SELECT_HIGH, 0, k, s["list"])
        agg.agg_kv_subsample_list(shape, s["list"], s["m"], k, v, s["Kc"], s["Vc"], s["kmean"],
                                  s["vmean"], s["bits"], s["dropped"], s["ws"], s["ws"].numel())
        agg.agg_global_attn_fwd_list(shape, s["m"], q, k, v, s["Kc"], s["Vc"], s["kmean"],
                                     s["vmean"], s["bits"], s["dropped"], s["O"], s["lse"])
        return {"O": s["O"], "lse": s["lse"], "list": s["list"], "dropped": s["dropped"]}
    if kind == "dense":
        agg.agg_dense_global_attn_fwd(shape, q, k, v, s["O"], s["lse"])
    else:
        agg.agg_frame_attn_fwd(shape, q, k, v, s["O"], s["lse"])
    return {"O": s["O"], "lse": s["lse"]}


def work(case):
    """Operations and bytes a pass cannot do without: inputs read once, outputs written once;
    what passes between the launches of one pass is not counted."""
    c, kind = case, case["kind"]
    nq, m, nd = _counts(c)
    B, H = c["B"], c["H"]
    C = H * HEAD_DIM
    row = 2 * C          # bytes of one token's bf16 row
    tokens = B * nq
    if kind == "subsample":
        return {"bytes": 2 * tokens * row + 2 * B * m * row + 4 * m, "flops": 2 * B * nd * C}
    L = nq // c["N"]
    if kind in ("frame", "block_frame"):
        keys = L
    elif kind == "dense":
        keys = nq
    else:
        keys = m + 2     # kept rows, the self term, the mean term
    attn = 4 * tokens * keys * C
    if kind in ("block_frame", "block_sga"):
        return {"bytes": 2 * tokens * row + 4 * C * row, "flops": attn + 8 * tokens * C * C}
    return {"bytes": 4 * tokens * row + 4 * tokens * H, "flops": attn}


def tolerance(case):
    kind = case["kind"]
    if kind == "subsample":
        return {"rel": 1e-6}               # 32-bit sums of bf16 values, partials added in 64 bits
    if kind in ("block_frame", "block_sga"):
        return {"rel": 8e-3, "max": 0.05}  # five bf16 roundings on the way to a bf16 result
    if kind == "list":
        # a magnitude tie resolved the other way swaps one window's token
        return {"rel": 1e-2, "max": 0.5, "differ": 1e-3}
    # bf16 operands and probabilities, bf16 results: 1.9e-3 off the result in 64 bits
    return {"rel": 8e-3, "max": 0.05}


# ---- the same results in 64 bits, in plain torch ---------------------------------------------
def _kept_mask(c):
    keep = torch.zeros((c["N"], c["n_special"] + c["n_h"] * c["n_w"]), dtype=torch.bool, device="cuda")
    keep[:, :c["n_special"]] = True
    patches = keep[:, c["n_special"]:].view(c["N"], c["n_h"], c["n_w"])
    patches[:, ::c["s_h"], ::c["s_w"]] = True
    if c["keep_first"]:
        keep[0] = True
    return keep.view(-1)


def _softmax_rows(q, k, v, own=None, mean=None):
    """One head: q [n, 64], k/v [m, 64] in float64.  own = (k_i, v_i, present) per query,
    mean = (kmean, vmean); returns the output rows and the log-sum-exp of their logits."""
    scale = 1.0 / math.sqrt(HEAD_DIM)
    o, lse = torch.empty_like(q), torch.empty(q.shape[0], dtype=q.dtype, device=q.device)
    step = max(1, (1 << 27) // max(1, k.shape[0]))
    kt = k.t().contiguous()
    for i in range(0, q.shape[0], step):
        rows = slice(i, min(q.shape[0], i + step))
        s = (q[rows] @ kt).mul_(scale)
        top = s.max(dim=1).values
        extras = []
        if own is not None:
            d = (q[rows] * own[0][rows]).sum(1) * scale
            d = torch.where(own[2][rows], d, torch.full_like(d, -math.inf))
            extras.append((d, own[1][rows]))
        if mean is not None:
            d = (q[rows] @ mean[0]) * scale
            extras.append((d, mean[1].expand(d.shape[0], -1)))
        for d, _ in extras:
            top = torch.maximum(top, d)
        s.sub_(top[:, None]).exp_()
        total, acc = s.sum(1), s @ v
        for d, val in extras:
            w = (d - top).exp()
            total = total + w
            acc = acc + w[:, None] * val
        o[rows] = acc / total[:, None]
        lse[rows] = top + total.log()
    return o, lse


def _attention64(c, kind, q, k, v, kept=None):
    """q, k, v: float64 [B, NQ, H, 64] (a head at a time is taken).  kept: bool [B, NQ]."""
    B, nq, H, _ = q.shape
    O = torch.empty((B, nq, H, HEAD_DIM), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, H, nq), dtype=torch.float64, device="cuda")
    km = torch.zeros((B, H, HEAD_DIM), dtype=torch.float64, device="cuda")
    vm = torch.zeros_like(km)
    L = nq // c["N"]
    special = (torch.arange(nq, device="cuda") % L) < c["n_special"]
    for b in range(B):
        for h in range(H):
            qh, kh, vh = (t[b, :, h].double() for t in (q, k, v))
            if kind == "frame":
                for f in range(0, nq, L):
                    r = slice(f, f + L)
                    O[b, r, h], lse[b, h, r] = _softmax_rows(qh[r], kh[r], vh[r])
            elif kind == "dense":
                O[b, :, h], lse[b, h] = _softmax_rows(qh, kh, vh)
            else:
                keep = kept[b]
                out = ~keep & ~special
                mean = own = None
                if bool(out.any()):
                    km[b, h], vm[b, h] = kh[out].mean(0), vh[out].mean(0)
                    mean, own = (km[b, h], vm[b, h]), (kh, vh, ~keep)
                O[b, :, h], lse[b, h] = _softmax_rows(qh, kh[keep], vh[keep], own, mean)
    if kind == "frame":
        lse = lse.view(B, H, c["N"], L).permute(0, 2, 1, 3).reshape(B * c["N"], H, L)
    return O, lse, km, vm


def _compact(rows, m_pad, which):
    """Kept rows [B, M, H, 64] -> the 64-row tiles of the compacted tensors, zero padded."""
    B, M, H, D = rows.shape
    t = torch.zeros((B, m_pad, H, D), dtype=rows.dtype, device=rows.device)
    t[:, :M] = rows
    t = t.permute(0, 2, 1, 3)
    if which == "k":
        t = t.reshape(B, H, m_pad // 64, 2, 32, 4, 2, 8).permute(0, 1, 2, 3, 5, 6, 4, 7)
    else:
        t = t.reshape(B, H, m_pad // 64, 4, 2, 2, 4, 64).permute(0, 1, 2, 3, 5, 7, 4, 6)
    return t.reshape(-1)


def _largest_of_window(c, k):
    """Kept mask when the token of largest sum of squares stands for its window."""
    B, nq = k.shape[:2]
    mag = torch.stack([k[b].double().square().sum((1, 2)) for b in range(B)])
    mag = mag.view(B, c["N"], -1)
    kept = torch.zeros_like(mag, dtype=torch.bool)
    kept[:, :, :c["n_special"]] = True
    # grid padded to whole windows with -1, windows side by side
    gh, gw = -(-c["n_h"] // c["s_h"]), -(-c["n_w"] // c["s_w"])
    grid = torch.full((B, c["N"], gh * c["s_h"], gw * c["s_w"]), -1.0, dtype=torch.float64, device="cuda")
    grid[:, :, :c["n_h"], :c["n_w"]] = mag[:, :, c["n_special"]:].view(B, c["N"], c["n_h"], c["n_w"])
    win = grid.view(B, c["N"], gh, c["s_h"], gw, c["s_w"]).permute(0, 1, 2, 4, 3, 5)
    win = win.reshape(B, c["N"], gh, gw, c["s_h"] * c["s_w"])
    pick = torch.nn.functional.one_hot(win.argmax(-1), c["s_h"] * c["s_w"]).bool()
    pick = pick.view(B, c["N"], gh, gw, c["s_h"], c["s_w"]).permute(0, 1, 2, 4, 3, 5)
    pick = pick.reshape(B, c["N"], gh * c["s_h"], gw * c["s_w"])[:, :, :c["n_h"], :c["n_w"]]
    kept[:, :, c["n_special"]:] = pick.reshape(B, c["N"], -1)
    if c["keep_first"]:
        kept[:, 0] = True
    return kept.view(B, nq)


def exact(case, seed):
    c, kind = case, case["kind"]
    if work(c)["flops"] > 5e13:
        return None
    if kind in ("block_frame", "block_sga"):
        x = _block_input(c, seed)
        w = inputs.block_weights(c["H"] * HEAD_DIM, seed, "cuda")
        x64 = x.double()
        xn = torch.nn.functional.layer_norm(x64, (x64.shape[-1],), w["ln_gamma"].double(),
                                            w["ln_beta"].double(), w["ln_eps"])
        heads = (x.shape[0], x.shape[1], c["H"], HEAD_DIM)
        q, k, v = ((xn @ w["w_" + n].double().t().contiguous() + w["b_" + n].double()).view(heads)
                   for n in "qkv")
        if kind == "block_frame":
            O, _, _, _ = _attention64(c, "frame", q, k, v)
        else:
            O, _, _, _ = _attention64(c, "layer", q, k, v, _kept_mask(c).expand(c["B"], -1))
        return {"y": x64 + O.view(x.shape) @ w["w_o"].double().t().contiguous() + w["b_o"].double()}
    q, k, v = _qkv(c, seed)
    kept = _kept_mask(c)
    idx = kept.nonzero().view(-1).to(torch.int32)
    if kind == "subsample":
        m_pad = -(-idx.numel() // 64) * 64
        out = ~kept
        means = [torch.zeros((c["B"], c["H"], HEAD_DIM), dtype=torch.float64, device="cuda") for _ in "kv"]
        if bool(out.any()):
            for b in range(c["B"]):
                for h in range(c["H"]):
                    for t, mean in zip((k, v), means):
                        mean[b, h] = t[b, out, h].double().mean(0)
        return {"idx": idx, "Kc": _compact(k[:, kept], m_pad, "k").double(),
                "Vc": _compact(v[:, kept], m_pad, "v").double(), "kmean": means[0], "vmean": means[1]}
    if kind == "list":
        kept = _largest_of_window(c, k)
        O, lse, _, _ = _attention64(c, "layer", q, k, v, kept)
        return {"O": O, "lse": lse, "list": None, "dropped": None}
    O, lse, km, vm = _attention64(c, "layer" if kind == "indexed" else kind, q, k, v,
                                  kept.expand(c["B"], -1))
    if kind in ("layer", "indexed"):
        return {"O": O, "lse": lse, "idx": idx, "kmean": km, "vmean": vm}
    return {"O": O, "lse": lse}
