"""Performance cases of the DraftAttention2 path.

A case is one use of the library's public calls at sizes a program has for
them: the whole layer (draft map, ranking, operand preparation, attention),
or one of the four calls on its own, as a program makes it that reuses the
results of the others (the draft map and ranking of an earlier denoising step,
one set of operands under several budgets). Inputs are synthetic video-DiT
activations: per head a sum of low-frequency space-time waves and noise, Q and
K on shared wave vectors, made on the GPU from the seed.

Fields of a case: ``op`` (step, attn, draft, rank, prep), the problem (B, H, d,
T, Hg, Wg, partition), ``dtype`` of Q, K and V (the output has the same),
budgets ``num16``, ``num8``, ``num4`` of ``den``, ranking ``scope``, ``lam``,
4-bit encoding ``fmt4``, and ``token_major`` (Q, K, V and the output are
[B, H, N, d] views of [B, N, H, d] storage, as a fused QKV projection gives).
"""
import math

import numpy as np
import torch

from paper_2609_32628_amd import api

CAP = 64   # slots of a block
ETA = 2.0 ** -8.807


def _case(name, op, B, H, d, T, Hg, Wg, dtype="bf16", num16=0, num8=10, num4=30, den=100, scope="head", lam=0.2,
          fmt4="nvfp4", partition="tiles8", token_major=False):
    c = dict(op=op, B=B, H=H, d=d, T=T, Hg=Hg, Wg=Wg, dtype=dtype, num16=num16, num8=num8, num4=num4, den=den,
             scope=scope, lam=lam, fmt4=fmt4, partition=partition, token_major=token_major)
    return c if name is None else dict(name=name, **c)


def listed():
    mid = dict(B=1, H=12, d=128, T=21, Hg=30, Wg=52)     # 32,760 tokens: one layer of a mid-size video DiT
    wide = dict(B=1, H=40, d=128, T=21, Hg=45, Wg=80)    # 75,600 tokens, 40 heads: a large video DiT
    long = dict(B=1, H=24, d=128, T=33, Hg=45, Wg=80)    # 118,800 tokens: a long or high-resolution clip
    return [
        # a layer over two small latent frames: launches and latency are the time
        _case("step-tiny", "step", 1, 2, 64, 2, 16, 16, dtype="fp32", num8=25, num4=25, scope="row"),
        # a short low-resolution clip, two samples (guidance pair), ragged edges everywhere
        _case("step-small-ragged", "step", 2, 6, 64, 5, 23, 37, scope="row", partition="ragged"),
        # the ordinary layer of one denoising step
        _case("step-mid", "step", **mid),
        # the same with the 4-bit encoding that the matrix cores scale natively
        _case("step-mid-mxfp4", "step", fmt4="mxfp4", **mid),
        # a quality setting: the first tenth of the pairs in 16 bits, regions with little padding,
        # tensors as the QKV projection leaves them
        _case("step-mid-16bit", "step", num16=10, partition="ragged", token_major=True, **mid),
        # the largest layer
        _case("step-wide", "step", **wide),
        # attention alone, as for further budgets on prepared operands: 4-bit pairs only (the cheapest setting) ...
        _case("attn-4bit", "attn", num8=0, num4=40, **mid),
        # ... and every pair in 8 bits (a dense layer, as in the first denoising steps)
        _case("attn-8bit", "attn", num8=100, num4=0, **mid),
        # the draft map of a large layer
        _case("draft-wide", "draft", **wide),
        # the ranking of a long clip's layer, e.g. under new budgets on the draft map of an earlier step
        _case("rank-long", "rank", num8=5, num4=25, **long),
        # operand preparation where routing is reused from an earlier step
        _case("prep-mid", "prep", **mid),
        # ... in float32 with the 16-bit and MXFP4 sections, head width 64
        _case("prep-fp32-mxfp4", "prep", 1, 20, 64, 13, 32, 56, dtype="fp32", num16=10, fmt4="mxfp4"),
    ]


def _regions(c):
    """Regions of one frame."""
    if c["partition"] == "ragged":
        return -(-c["Hg"] * c["Wg"] // CAP)
    return -(-c["Hg"] // 8) * -(-c["Wg"] // 8)


def _tiles(c):
    """Retained 64 x 64 tiles of a pass."""
    R = c["T"] * _regions(c)
    return c["B"] * c["H"] * R * R * (c["num16"] + c["num8"] + c["num4"]) / c["den"]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        # each op at the shares the listed cases have, over frame counts, frame sizes and heads on a log scale
        op = rng.choice(["step"] * 6 + ["attn"] * 2 + ["draft", "rank", "prep", "prep"])
        den = rng.choice([100, 100, 1000, 64])
        n16 = rng.choice([0, 0, 0, rng.randint(1, den // 8)])
        n8 = rng.choice([0, rng.randint(1, den // 2), den // 10, den // 20])
        n4 = rng.choice([0, rng.randint(1, den // 2), 3 * den // 10, den // 4])
        c = _case(None, op, rng.choice([1, 1, 1, 2]), log(1, 40), rng.choice([64, 128, 128]), log(1, 33), log(8, 60),
                  log(8, 104), dtype=rng.choice(["bf16", "bf16", "fp32"]), num16=n16, num8=n8, num4=n4, den=den,
                  scope=rng.choice(["head", "head", "row"]), lam=rng.choice([0.2, 0.2, 0.0, 1.0, 0.35]),
                  fmt4=rng.choice(["nvfp4", "nvfp4", "mxfp4"]), partition=rng.choice(["tiles8", "ragged"]),
                  token_major=rng.random() < 0.4)
        R = c["T"] * _regions(c)
        if n16 + n8 + n4 == 0 or n16 + n8 + n4 > den or R > 2000:
            continue
        # no more than the largest listed layer: its tokens and a third of its tiles (tiles of drawn cases may be dense)
        if c["B"] * c["H"] * c["T"] * c["Hg"] * c["Wg"] <= 2.0e6 and _tiles(c) <= 8e6:
            return c


# ---- inputs ------------------------------------------------------------------
def _field(gen, waves, T, Hg, Wg, d, scale):
    """One head of one tensor, [T Hg Wg, d] float32: four waves and noise per channel."""
    dev = gen.device
    kt, ky, kx = waves
    amp = torch.randn(4, d, generator=gen, device=dev) * scale
    phi = torch.rand(4, d, generator=gen, device=dev) * (2 * math.pi)
    drift = (torch.rand(4, d, generator=gen, device=dev) - 0.5) * (math.pi / 8)
    t = torch.arange(T, device=dev, dtype=torch.float32)[:, None]
    y = torch.arange(Hg, device=dev, dtype=torch.float32)[:, None]
    x = torch.arange(Wg, device=dev, dtype=torch.float32)[:, None]
    out = 0.1 * torch.randn(T, Hg, Wg, d, generator=gen, device=dev)
    for k in range(4):
        pt = phi[k] + t * (kt[k] * (2 * math.pi / T) + drift[k])
        py, px = y * (ky[k] * (2 * math.pi / Hg)), x * (kx[k] * (2 * math.pi / Wg))
        pty = (pt[:, None] + py[None, :])[:, :, None]          # [T, Hg, 1, d]
        out += (amp[k] * torch.sin(pty)) * torch.cos(px) + (amp[k] * torch.cos(pty)) * torch.sin(px)
    return out.reshape(T * Hg * Wg, d)


def _inputs(c, seed, device, tensors=3, grid=None):
    """Q, K and V ([B, H, N, d]) of the case, the first ``tensors`` of them."""
    B, H, d = c["B"], c["H"], c["d"]
    T, Hg, Wg = grid or (c["T"], c["Hg"], c["Wg"])
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    N = T * Hg * Wg
    shape = (B, N, H, d) if c["token_major"] else (B, H, N, d)
    xs = [torch.empty(shape, dtype=dt, device=device) for _ in range(tensors)]
    xs = [x.transpose(1, 2) if c["token_major"] else x for x in xs]
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)

    def waves():
        return [torch.randint(0, n, (4, d), generator=gen, device=device).float() for n in (3, 4, 4)]

    for b in range(B):
        for h in range(H):
            scale = (0.5 + 1.5 * torch.rand(3, generator=gen, device=device))
            w_qk, w_v = waves(), waves()
            for i, x in enumerate(xs):
                x[b, h] = _field(gen, w_qk if i < 2 else w_v, T, Hg, Wg, d, scale[i])
    return xs


def _pooled_map(c, seed, device):
    """A draft map for the ranking alone: softmaxes of descriptors drawn on the grid of the regions."""
    nI, nJ = -(-c["Hg"] // 8), -(-c["Wg"] // 8)
    if c["partition"] == "ragged":
        nI, nJ = 1, _regions(c)
    g = dict(c, dtype="fp32", token_major=False)
    Q, K = _inputs(g, seed, device, 2, (c["T"], nI, nJ))
    A = torch.empty((c["B"], c["H"], Q.shape[2], Q.shape[2]), dtype=torch.float32, device=device)
    for b in range(c["B"]):
        for h in range(c["H"]):
            q, k = Q[b, h].double(), K[b, h].double()
            A[b, h] = torch.softmax(q @ k.T.contiguous() / math.sqrt(c["d"]), dim=1).float()
    return A


def prepare(case, seed):
    c = case
    p = api.problem(c["B"], c["H"], c["d"], c["T"], c["Hg"], c["Wg"], c["partition"])
    buf = api.alloc(p, c["scope"], fmt4=c["fmt4"], with16=c["num16"] > 0)
    for x in (buf.A, buf.cls, buf.stats, buf.lists, buf.ops):
        x.zero_()   # bytes that a call leaves alone compare equal
    s = dict(c=c, p=p, buf=buf, budgets=(c["num8"], c["num4"], c["den"]), with16=int(c["num16"] > 0))
    if c["op"] == "rank":
        buf.A.copy_(_pooled_map(c, seed, "cuda"))
        return s
    Q, K, V = _inputs(c, seed, "cuda")
    s.update(Q=Q, K=K, V=V)
    if c["op"] in ("step", "attn"):
        s["O"] = torch.empty_strided(Q.shape, Q.stride(), dtype=Q.dtype, device="cuda")
    if c["op"] in ("attn", "prep"):
        api.da2_draft_map(Q, K, buf.layout, p, c["lam"], buf.A, buf.stats, buf.ws_draft)
    if c["op"] == "attn":
        api.da2_rank_assign(buf.A, p, c["num16"], *s["budgets"], c["scope"], buf.cls, buf.lists, buf.ws_rank)
        api.da2_prep_operands(Q, K, V, buf.layout, p, s["with16"], c["fmt4"], buf.stats, buf.ops, None)
    return s


def _stats(s):
    c = s["c"]
    return s["buf"].stats.view(torch.float32).view(c["B"] * c["H"], 4 + c["d"])


def run(state):
    s = state
    c, p, buf = s["c"], s["p"], s["buf"]
    op = c["op"]
    if op == "step":
        api.attention(s["Q"], s["K"], s["V"], buf, c["lam"], s["budgets"], s["O"], num16=c["num16"])
        return {"O": s["O"], "A": buf.A, "cls": buf.cls}
    if op == "attn":
        api.da2_mixed_attn(buf.ops, buf.lists, buf.layout, p, s["O"], fmt4=c["fmt4"])
        return {"O": s["O"]}
    if op == "draft":
        api.da2_draft_map(s["Q"], s["K"], buf.layout, p, c["lam"], buf.A, buf.stats, buf.ws_draft)
        return {"A": buf.A, "stats": _stats(s)}
    if op == "rank":
        api.da2_rank_assign(buf.A, p, c["num16"], *s["budgets"], c["scope"], buf.cls, buf.lists, buf.ws_rank)
        lo = api.da2_lists_offsets(p)
        n, R = c["B"] * c["H"] * buf.sizes["R"], buf.sizes["R"]
        return {"cls": buf.cls, "keys": buf.lists[lo[0]:lo[0] + 2 * n * R].view(torch.int16),
                "counts": buf.lists[lo[1]:lo[1] + 16 * n].view(torch.int32)}
    api.da2_prep_operands(s["Q"], s["K"], s["V"], buf.layout, p, s["with16"], c["fmt4"], buf.stats, buf.ops, None)
    return {"ops": buf.ops, "stats": _stats(s)}


def work(case):
    c = case
    BH, R, d = c["B"] * c["H"], c["T"] * _regions(c), c["d"]
    x = BH * c["T"] * c["Hg"] * c["Wg"] * d * (2 if c["dtype"] == "bf16" else 4)   # bytes of Q (of K, V, O)
    slots = BH * R * CAP * d
    A, cls, keys = 4 * BH * R * R, BH * R * R, 2 * _tiles(c)
    q4 = 4.5 / 8 if c["fmt4"] == "nvfp4" else (d / 32 + 1) / (d / 32) / 2
    ops = 3 * slots * (1 + q4 + (2 if c["num16"] else 0))
    # the encodings that some pair uses
    used = 3 * slots * ((1 if c["num8"] else 0) + (q4 if c["num4"] else 0) + (2 if c["num16"] else 0))
    attn = 4.0 * CAP * CAP * d * _tiles(c)
    draft = 4.0 * BH * R * R * d
    return {"step": {"bytes": 4 * x + A + cls, "flops": attn + draft},
            "attn": {"bytes": used + keys + x, "flops": attn},
            "draft": {"bytes": 2 * x + A, "flops": draft},
            "rank": {"bytes": A + cls + keys, "flops": 0},
            "prep": {"bytes": 3 * x + ops, "flops": 0}}[c["op"]]


def tolerance(case):
    if case["op"] in ("rank", "prep"):
        return "exact"          # classes, lists, encoded bytes and maxima
    if case["op"] == "draft":
        return {"rel": 1e-7}    # float64 sums, rounded once to float32
    # a weight whose float32 value lies near a rounding midpoint of its 4- or 8-bit
    # format may round the other way; bf16 outputs add a flip of their own last bit.
    # The draft map is as above; a class may differ at a tie of the float32 scores.
    return {"rel": 1e-3 if case["dtype"] == "bf16" else 2e-4, "max": 0.25, "differ": 1e-6}


# ---- the same in 64 bits -----------------------------------------------------------
def _f32(x):
    return x.float().double()


def _e4m3(x):
    return x.clamp(-448.0, 448.0).float().to(torch.float8_e4m3fn).double()


def _e2m1(x):
    a = x.abs()
    r = torch.where(a < 2, torch.round(a * 2) / 2, torch.where(a < 4, torch.round(a), torch.round(a / 2) * 2))
    return torch.copysign(r.clamp(max=6.0), x)


def _ragged_frame(H, W):
    """Region of every cell: the run partition of smallest perimeter (row bands first, fewer bands first)."""
    best = None
    for turn in (0, 1):
        h, w = (W, H) if turn else (H, W)
        for nb in range(1, h + 1):
            heights = [h // nb + (i < h % nb) for i in range(nb)]
            runs = [-(-q * w // CAP) for q in heights]
            if sum(runs) != -(-H * W // CAP):
                continue
            lab, y0, first = np.empty((h, w), np.int64), 0, 0
            for q, r in zip(heights, runs):
                # down one column and up the next, cut into runs of balanced size
                ys = np.concatenate([np.arange(q) if x % 2 == 0 else np.arange(q)[::-1] for x in range(w)]) + y0
                xs = np.repeat(np.arange(w), q)
                lab[ys, xs] = first + np.repeat(np.arange(r), [q * w // r + (k < q * w % r) for k in range(r)])
                y0, first = y0 + q, first + r
            cut = int((lab[:, 1:] != lab[:, :-1]).sum() + (lab[1:] != lab[:-1]).sum())
            if best is None or cut < best[0]:
                best = (cut, lab.T if turn else lab)
    return best[1]


def _slots(c):
    """Token of every slot [R, 64] (-1: padding)."""
    Hg, Wg, T = c["Hg"], c["Wg"], c["T"]
    if c["partition"] == "ragged":
        lab = _ragged_frame(Hg, Wg)
    else:
        lab = (np.arange(Hg)[:, None] // 8) * -(-Wg // 8) + np.arange(Wg)[None, :] // 8
    frame = np.full((int(lab.max()) + 1, CAP), -1, np.int64)
    for r in range(frame.shape[0]):
        toks = np.flatnonzero(lab.reshape(-1) == r)
        frame[r, :toks.size] = toks
    every = [np.where(frame >= 0, frame + t * Hg * Wg, -1) for t in range(T)]
    return torch.from_numpy(np.concatenate(every))


def _draft64(q, k, valid, lam):
    """Draft map of one head; q, k: [R, 64, d] float64 by slot, valid [R, 64]."""
    d, n = q.shape[2], valid.sum(1, keepdim=True)
    out = 0
    for w, pool in ((1.0 - lam, lambda x: (x * valid[..., None]).sum(1) / n),
                    (lam, lambda x: torch.where(valid[..., None], x, -math.inf).amax(1))):
        s = pool(q) @ pool(k).T.contiguous() / math.sqrt(d)
        out = out + w * torch.softmax(s, dim=1)
    return out


def _classes(A, c):
    """Class of every pair of one head from its float32 scores: a stable sort, best first."""
    R = A.shape[0]
    rows = A.reshape(1, -1) if c["scope"] == "head" else A
    M = rows.shape[1]
    n16, n8, n4, den = c["num16"], c["num8"], c["num4"], c["den"]
    cuts = [(2 * n * M + den) // (2 * den) for n in (n16, n16 + n8, n16 + n8 + n4)]
    rank = torch.empty(rows.shape, dtype=torch.int64, device=A.device)
    rank.scatter_(1, torch.sort(rows, dim=1, descending=True, stable=True).indices,
                  torch.arange(M, device=A.device).expand(rows.shape[0], M))
    cls = torch.where(rank < cuts[0], 16, torch.where(rank < cuts[1], 8, torch.where(rank < cuts[2], 4, 0)))
    return cls.reshape(R, R).to(torch.uint8)


def _groups(x, size):
    """x [R, 64, d] -> [R, 64, d / size, size] (channel groups)."""
    return x.reshape(x.shape[0], x.shape[1], -1, size)


def _nvfp4(x, amax, along_slots):
    """NVFP4 values in original units (groups of 16 channels, or of 16 slots)."""
    if along_slots:
        return _nvfp4(x.transpose(1, 2), amax, False).transpose(1, 2)
    g = _f32(amax / 2688.0)
    g = torch.where(g == 0, 1.0, g)
    y = _groups(x, 16)
    sigma = _e4m3(_f32(y.abs().amax(-1, keepdim=True) / _f32(6.0 * g)))
    inv = _f32(1.0 / _f32(g * torch.where(sigma == 0, 1.0, sigma)))
    return torch.where(sigma == 0, 0.0, g * sigma * _e2m1(_f32(y * inv))).reshape(x.shape)


def _mx_exponent(amax):
    e = torch.frexp(torch.where(amax > 0, amax, 1.0)).exponent.double() - 3
    return torch.where(amax > 0, e.clamp(-127, 127), -127.0)


def _mxfp4(x, along_slots):
    if along_slots:
        return _mxfp4(x.transpose(1, 2), False).transpose(1, 2)
    y = _groups(x, 32)
    X = torch.exp2(_mx_exponent(y.abs().amax(-1, keepdim=True)))
    return (X * _e2m1(y / X)).reshape(x.shape)


def _int8(x):
    delta = _f32(_f32(x.abs().amax((1, 2), keepdim=True) / 127.0) + float(np.float32(1e-7)))
    y = _f32(x * _f32(1.0 / delta))
    return delta * torch.copysign(torch.floor(y.abs() + 0.5), y).clamp(-127, 127)


def _e4m3_v(v):
    delta = _f32(v.abs().amax((0, 1)) / 2.25)
    inv = torch.where(delta == 0, 0.0, _f32(1.0 / torch.where(delta == 0, 1.0, delta)))
    return delta * _e4m3(_f32(v * inv))


def _weights(P, phase, mx):
    """Quantized weights of the unnormalized ones P [..., 64]."""
    if phase == 16:
        return P.half().double()
    if phase == 8:
        return ETA * _e4m3(P / ETA)
    if mx:
        g = P.reshape(P.shape[:-1] + (2, 32))
        X = torch.exp2(_mx_exponent(g.amax(-1, keepdim=True)))
        return (X * _e2m1(g / X)).reshape(P.shape)
    g = P.reshape(P.shape[:-1] + (4, 16))
    sigma = _e4m3(448.0 * g.amax(-1, keepdim=True))
    w = sigma / 2688.0 * _e2m1(2688.0 * g / torch.where(sigma == 0, 1.0, sigma))
    return torch.where(sigma == 0, 0.0, w).reshape(P.shape)


def _attend64(q, k, v, valid, cls, c):
    """One head: [R, 64, d] outputs by slot."""
    R, _, d = q.shape
    mx = c["fmt4"] == "mxfp4"
    ph = {}
    if c["num4"]:
        ph[4] = ((_mxfp4(q, False), _mxfp4(k, False), _mxfp4(v, True)) if mx else
                 tuple(_nvfp4(x, x.abs().max(), x is v) for x in (q, k, v)))
    if c["num8"]:
        ph[8] = (_int8(q), _int8(k), _e4m3_v(v))
    if c["num16"]:
        ph[16] = tuple(x.half().double() for x in (q, k, v))
    out = torch.zeros_like(q)
    turn = torch.where(cls == 4, 0, torch.where(cls == 8, 1, torch.where(cls == 16, 2, 3)))
    order = torch.sort(turn, dim=1, stable=True)
    count = (cls > 0).sum(1)
    step = max(1, min(R, int(2.5e8 / (CAP * CAP * max(1, int(count.max()))))))
    for a in range(0, R, step):
        rows = slice(a, min(R, a + step))
        n = int(count[rows].max())
        if n == 0:
            continue
        idx, t = order.indices[rows, :n], order.values[rows, :n]
        m = idx.shape[0]
        S = torch.full((m, CAP, n, CAP), -math.inf, dtype=torch.float64, device=q.device)
        use = {p: (t == i)[:, None, :, None] for i, p in enumerate((4, 8, 16)) if p in ph}
        for p, on in use.items():
            K = ph[p][1][idx].reshape(m, n * CAP, d)
            s = torch.bmm(ph[p][0][rows], K.transpose(1, 2).contiguous()).reshape(m, CAP, n, CAP) / math.sqrt(d)
            S = torch.where(on & valid[idx][:, None], s, S)
        top = torch.cummax(S.amax(3), dim=2).values                     # running maximum, [m, 64, n]
        P = torch.exp(S - top[..., None])
        f = torch.exp(top - top[..., -1:])
        den = (f * P.sum(3)).sum(2)
        num = 0
        for p, on in use.items():
            w = torch.where(on, _weights(P, p, mx), 0.0) * f[..., None]
            num = num + torch.bmm(w.reshape(m, CAP, n * CAP), ph[p][2][idx].reshape(m, n * CAP, d))
        out[rows] = torch.where(count[rows][:, None, None] > 0, num / den[..., None], 0.0)
    return out


def exact(case, seed):
    c = case
    BH, T, N, d = c["B"] * c["H"], c["T"], c["T"] * c["Hg"] * c["Wg"], c["d"]
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if c["op"] == "rank":
        A = _pooled_map(c, seed, dev)
        R = A.shape[2]
        cls = torch.stack([_classes(A[b, h], c) for b in range(c["B"]) for h in range(c["H"])])
        turn = torch.where(cls == 4, 0, torch.where(cls == 8, 1, torch.where(cls == 16, 2, 3))).to(torch.uint8)
        o = torch.sort(turn, dim=2, stable=True)
        keys = torch.where(o.values < 3, o.indices, 0).to(torch.int16)
        n = torch.stack([(cls == v).sum(2) for v in (4, 8, 16)] + [torch.zeros_like(cls[..., 0]).long()], dim=2)
        return {"cls": cls.reshape(A.shape), "keys": keys.reshape(-1), "counts": n.to(torch.int32).reshape(-1)}
    if c["op"] in ("step", "attn") and _tiles(c) > 5e6:
        return None   # over twenty seconds
    Q, K, V = _inputs(c, seed, dev)
    if c["op"] == "prep":
        top = [x.float().abs().amax((2, 3)).reshape(BH) for x in (Q, K, V)]
        stats = torch.cat([torch.stack(top + [torch.zeros_like(top[0])], 1), V.float().abs().amax(2).reshape(BH, d)], 1)
        return {"ops": None, "stats": stats.double()}
    slots = _slots(c).to(dev)
    valid, at = slots >= 0, slots.clamp(min=0)
    R = slots.shape[0]
    A = torch.empty((BH, R, R), dtype=torch.float64, device=dev)
    cls = torch.empty((BH, R, R), dtype=torch.uint8, device=dev)
    O = torch.empty((BH, N, d), dtype=torch.float64, device=dev)
    stats = torch.zeros((BH, 4 + d), dtype=torch.float64, device=dev)
    for i in range(BH):
        b, h = divmod(i, c["H"])
        q, k, v = (torch.where(valid[..., None], x[b, h].double()[at], 0.0) for x in (Q, K, V))
        A[i] = _draft64(q, k, valid, c["lam"])
        if c["op"] == "draft":
            stats[i, 0], stats[i, 1] = q.abs().max(), k.abs().max()
            continue
        cls[i] = _classes(A[i].float(), c)
        O[i, slots[valid]] = _attend64(q, k, v, valid, cls[i], c)[valid]
    A = A.reshape(c["B"], c["H"], R, R)
    if c["op"] == "draft":
        return {"A": A, "stats": stats}
    O = O.reshape(c["B"], c["H"], N, d)
    if c["op"] == "attn":
        return {"O": O}
    return {"O": O, "A": A, "cls": cls.reshape(A.shape)}
