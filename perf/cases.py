"""Timed cases of the library's public entry points.

A case is one call (or one denoising step: mask build, then attention) of the
kind a video diffusion program makes: self-attention of one transformer layer
over T latent frames of P = h*w tokens plus optional text tokens, in one of
the forms the library offers:

    block   block-sparse attention over an LVSA block mask
    exact   token-exact attention (the LVSA frame sets token for token)
    dense   dense attention
    mask    the device mask builder alone (block form and token-exact form)

Options: block size B (64 or 128), head count H, the tensor layout (`hnd`:
[H, N, 128] contiguous; `nhd`: Q, K and V are views of one fused projection
[N, 3, H, 128]), and where the mask comes from (`given`: built before the
call and shared by the layers of a step; `device`: the device builder on the
stream in front of the attention; `host`: the host builder plus its upload).

The shapes are those of the repository's workloads (Wan 2.1 1.3B and 14B, 30x52
latents, 21 frames at the training horizon, 121 at six times it;
HunyuanVideo 1.5, 30x53 latents, 65 frames at twice the horizon, 512 text
tokens), a few heads of them as one GPU of a head-sharded layer holds, and
short clips.  Values are N(0, 1) rounded to bf16, the repository's recipe.
"""
import math
import random

import numpy as np
import torch

import paper_2605_31057_amd as lvsa

D = 128


def _case(name, form, H, T, P, B=128, text=0, C=21, W=6, tper=0, step=10, mask="given",
          layout="hnd", entry="attention"):
    c = dict(form=form, H=H, T=T, P=P, B=B, text=text, C=C, W=W, tper=tper, step=step,
             mask=mask, layout=layout, entry=entry)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The repository's smallest workload (4 frames of 16x16, one head, block
        # 64) as a whole denoising step: launches and latency count.
        _case("tiny_step", "block", 1, 4, 256, B=64, C=2, W=0, tper=4, step=1, mask="device"),
        # One latent frame (an image, or a first frame) through dense attention.
        _case("image_dense", "dense", 12, 1, 1560),
        # A short, small preview clip with odd sizes, its token-exact mask
        # built on the host for this step and uploaded.
        _case("clip_host_exact", "exact", 12, 9, 391, C=7, W=2, step=3, mask="host"),
        # The mask of one step at the long horizon, both forms, as a denoising
        # loop builds it in front of its layers.
        _case("mask_wan_6x", "mask", 0, 121, 1560),
        # Wan 1.3B at the training horizon, Q, K, V straight from the fused
        # projection (strided).
        _case("wan13_1x_nhd", "block", 12, 21, 1560, layout="nhd"),
        # The dense layer that LVSA replaces, at the training horizon, for the
        # 5 of 40 heads that one of 8 GPUs holds of a head-sharded 14B layer.
        _case("wan14_1x_dense_5h", "dense", 5, 21, 1560),
        # Wan 1.3B at twice the horizon with 64-token blocks (a block mask
        # closer to the frame mask).
        _case("wan13_2x_b64", "block", 12, 41, 1560, B=64),
        # HunyuanVideo 1.5, twice the horizon: the 2 of 16 heads that one of 8
        # GPUs holds.
        _case("hv15_2x_2h", "block", 2, 65, 1590, C=33),
        # The whole HunyuanVideo layer with its text tokens, token-exact.
        _case("hv15_2x_text_exact", "exact", 16, 65, 1590, text=512, C=33),
        # The main workload: Wan 1.3B at six times the horizon, one denoising
        # step with its mask built on the device.
        _case("wan13_6x_step", "block", 12, 121, 1560, mask="device"),
        # The same horizon in the token-exact form.
        _case("wan13_6x_exact", "exact", 12, 121, 1560),
        # The largest: a whole Wan 14B layer at six times the horizon.
        _case("wan14_6x", "block", 40, 121, 1560),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    cap = work(listed()[-1])["flops"]
    while True:
        form = rng.choice(["block", "block", "block", "exact", "exact", "dense", "mask"])
        T = _log_int(rng, 1, 121)
        P = _log_int(rng, 8, 34) * _log_int(rng, 8, 60)
        H = _log_int(rng, 1, 40) if form != "mask" else 0
        B = rng.choice([128, 128, 64])
        W = rng.randint(0, 6)
        C = 2 * W + 1 + rng.randint(1, 12)
        text = _log_int(rng, 1, 512) if rng.random() < 0.25 else 0
        if form == "dense":
            text = 0
        if form == "mask":
            T = _log_int(rng, 24, 121)
            W = rng.randint(1, 6)
            C = 2 * W + 1 + rng.randint(5, 12)
        c = _case(None, form, H, T, P, B=B, text=text, C=C, W=W, step=rng.randint(0, 49),
                  mask=rng.choice(["given", "given", "device", "host"]),
                  layout=rng.choice(["hnd", "nhd"]),
                  entry="noalloc" if form == "block" and rng.random() < 0.25 else "attention")
        if form in ("exact", "mask") and P < B:
            continue
        w = work(c)
        if w["flops"] > cap or (form != "mask" and w["flops"] < 1e8):
            continue
        return c


# ---------------------------------------------------------------- frame sets

def _frame_sets(c):
    """A(t) of every frame t as a boolean [T, T] array, in the paper's own
    order: anchors of Eq. 3, the adaptive window, Alg. 1 one frame at a time."""
    T, W, E = c["T"], c["W"], c.get("E", 0)
    tper = c["tper"] or -(-T // (c["C"] - (2 * W + 1) - E))
    s = c["step"] % tper
    anchors = {(s + i * tper) % T for i in range(-(-T // tper))} | set(range(min(E, T)))
    A = np.zeros((T, T), dtype=bool)
    target = min(2 * W + 1, T - len(anchors))
    for t in range(T):
        lo = max(0, min(t - W, T - 1 - 2 * W))
        hi = min(T - 1, max(t + W, 2 * W))
        while sum(f not in anchors for f in range(lo, hi + 1)) < target and (lo > 0 or
                                                                           hi < T - 1):
            if lo >= T - 1 - hi and lo > 0:
                lo -= 1
            else:
                hi += 1
        A[t, lo:hi + 1] = True
        A[t, sorted(anchors)] = True
    return A


def _segments(c):
    """Attended-segment matrix (frames, then the text as one more segment)
    and each segment's first token, with N at the end."""
    A = _frame_sets(c)
    T, P, L = c["T"], c["P"], c["text"]
    edges = [t * P for t in range(T + 1)]
    if L:
        A = np.pad(A, ((0, 1), (0, 1)), constant_values=True)
        edges.append(T * P + L)
    return A, np.asarray(edges)


def _tokens(c):
    return c["T"] * c["P"] + c["text"]


def _blocks(c):
    """Kept blocks [nb, nb] (any attended segment pair), and segment bounds of
    every block."""
    A, edges = _segments(c)
    N, B = _tokens(c), c["B"]
    nb = -(-N // B)
    first = np.arange(nb) * B
    last = np.minimum(first + B, N) - 1
    s0 = np.searchsorted(edges, first, side="right") - 1
    s1 = np.searchsorted(edges, last, side="right") - 1
    touch = (np.arange(A.shape[0])[None] >= s0[:, None]) & (np.arange(A.shape[0])[None] <=
                                                            s1[:, None])
    t = touch.astype(np.float32)
    return (t @ A.astype(np.float32) @ t.T) > 0, s0, s1


def _csr_and_entries(c):
    keep, s0, s1 = _blocks(c)
    A, edges = _segments(c)
    B = c["B"]
    row_ptr = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int32)
    qb, kb = np.nonzero(keep)
    straddles = s1[kb] > s0[kb]
    kfirst = np.where(straddles, edges[s0[kb] + 1] - kb * B, B)
    pat = (A[s0[qb], s0[kb]] * 1 + A[s0[qb], s1[kb]] * 2 + A[s1[qb], s0[kb]] * 4 +
           A[s1[qb], s1[kb]] * 8)
    return row_ptr, kb.astype(np.int32), (kb | (kfirst << 16) | (pat << 24)).astype(np.int64)


# ---------------------------------------------------------------- one case

def _params(c):
    return lvsa.Params(budget_frames=c["C"], window=c["W"], tper=c["tper"],
                       extra_anchors=c.get("E", 0), text_tokens=c["text"])


def _seeded_mask(c, seed):
    """The mask form's inputs are its step and pattern: a seed takes another
    step of the loop, up to three dedicated first anchors and a window one
    frame narrower or not (the kept share moves by a few percent)."""
    r = random.Random(seed)
    return dict(c, step=r.randint(0, 49), E=r.randint(0, 3), W=c["W"] - r.randint(0, 1))


def prepare(case, seed):
    c = _seeded_mask(case, seed) if case["form"] == "mask" else case
    N, B, H = _tokens(c), c["B"], c["H"]
    nb = -(-N // B)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    s = {"case": c, "params": _params(c), "step": c["step"]}
    if c["form"] == "mask":
        s["row_ptr"] = torch.zeros(nb + 1, dtype=torch.int32, device="cuda")
        s["row_ptr_x"] = torch.zeros_like(s["row_ptr"])
        s["col_idx"] = torch.zeros(nb * nb, dtype=torch.int32, device="cuda")
        s["entry"] = torch.zeros(nb * nb, dtype=torch.int32, device="cuda")
        return s
    if c["layout"] == "nhd":
        qkv = torch.empty((N, 3, H, D), dtype=torch.bfloat16, device="cuda")
        s["qkv"] = [qkv[:, i].transpose(0, 1) for i in range(3)]
        s["out"] = torch.empty((N, H, D), dtype=torch.bfloat16, device="cuda").transpose(0, 1)
    else:
        s["qkv"] = [torch.empty((H, N, D), dtype=torch.bfloat16, device="cuda")
                    for _ in range(3)]
        s["out"] = torch.empty((H, N, D), dtype=torch.bfloat16, device="cuda")
    for h in range(H):
        for x in s["qkv"]:
            x[h].copy_(torch.randn((N, D), generator=g, device="cuda"))
    if c["form"] == "dense":
        return s
    exact = c["form"] == "exact"
    if c["mask"] == "given":
        s["csr"] = lvsa.build_mask(c["T"], c["P"], B, c["step"], s["params"], exact=exact)
        s["csr"].upload()
        s["view"] = s["csr"].exact_mask() if exact else s["csr"].device_mask()
    elif c["mask"] == "device":
        s["row_ptr"] = torch.empty(nb + 1, dtype=torch.int32, device="cuda")
        s["rows"] = torch.empty(nb * nb, dtype=torch.int32, device="cuda")
    return s


def run(state):
    s, c = state, state["case"]
    T, P, B, step, p = c["T"], c["P"], c["B"], s["step"], s["params"]
    if c["form"] == "mask":
        lvsa.build_mask_device(T, P, B, step, s["row_ptr"], s["col_idx"], params=p)
        lvsa.build_exact_mask_device(T, P, B, step, s["row_ptr_x"], s["entry"], params=p)
        return s["row_ptr"], s["col_idx"], s["row_ptr_x"], s["entry"]
    q, k, v = s["qkv"]
    if c["form"] == "dense":
        return lvsa.dense_attention(q, k, v, block=B, out=s["out"])
    exact = c["form"] == "exact"
    if c["mask"] == "device":
        build = lvsa.build_exact_mask_device if exact else lvsa.build_mask_device
        m = build(T, P, B, step, s["row_ptr"], s["rows"], params=p)
    elif c["mask"] == "host":
        # The handle of the step before is freed once this step's is built.
        s["csr"] = lvsa.build_mask(T, P, B, step, p, exact=exact)
        s["csr"].upload()
        m = s["csr"].exact_mask() if exact else s["csr"].device_mask()
    else:
        m = s["view"]
    if exact:
        return lvsa.attention_exact(q, k, v, m, out=s["out"])
    if c["entry"] == "noalloc":
        return lvsa.attention_noalloc(q, k, v, m, s["out"])
    return lvsa.attention(q, k, v, m, out=s["out"])


def work(case):
    """Kept (query, key) token pairs at 4*D FLOP each; Q, K and V read and the
    output written once, plus the mask where the pass builds or reads one."""
    c = case
    N, H, B = _tokens(c), c["H"], c["B"]
    nb = -(-N // B)
    if c["form"] == "mask":
        nnz = int(_blocks(c)[0].sum())
        return {"bytes": 8 * (nb + 1) + 8 * nnz, "flops": 0}
    if c["form"] == "dense":
        return {"bytes": 8 * H * N * D, "flops": 4 * D * H * N * N}
    keep, _, _ = _blocks(c)
    if c["form"] == "exact":
        A, edges = _segments(c)
        size = np.diff(edges).astype(np.float64)
        pairs = float(size @ A.astype(np.float64) @ size)
    else:
        size = np.full(nb, float(B))
        size[-1] = N - B * (nb - 1)
        pairs = float(size @ keep.astype(np.float64) @ size)
    return {"bytes": 8 * H * N * D + 4 * (nb + 1 + int(keep.sum())),
            "flops": 4 * D * H * pairs}


def tolerance(case):
    """bf16 probabilities and a bf16 result.  Measured: against float64 the
    result is off by 2.4e-3 of its 2-norm (rounding float64 itself to bf16:
    1.7e-3), the largest difference 1.2e-2 of the root mean square or of the
    value; walking the keys in the other order moves it by 3.1e-3 and at most
    1.8e-2.  Four times the latter.  Masks are integers."""
    if case["form"] == "mask":
        return "exact"
    return {"rel": 1.25e-2, "max": 7e-2}


def exact(case, seed):
    """The same pass in float64 from the same inputs with plain torch."""
    c = case
    if c["form"] == "mask":
        rp, ci, ent = _csr_and_entries(_seeded_mask(c, seed))
        nb = len(rp) - 1
        full = np.zeros((2, nb * nb), dtype=np.int64)
        full[0, :len(ci)] = ci
        full[1, :len(ci)] = ent
        return rp, full[0].astype(np.int32), rp, full[1].astype(np.int32)
    if work(c)["flops"] > 5e13:
        return None
    N, H, B = _tokens(c), c["H"], c["B"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    # Runs of query tokens that share one key set, and that set.
    if c["form"] == "dense":
        runs = [(0, N, torch.arange(N, device="cuda"))]
    elif c["form"] == "exact":
        A, edges = _segments(c)
        runs = []
        for t in range(A.shape[0]):
            keys = np.concatenate([np.arange(edges[u], edges[u + 1]) for u in np.nonzero(A[t])[0]])
            runs.append((int(edges[t]), int(edges[t + 1]), torch.from_numpy(keys).cuda()))
    else:
        keep, _, _ = _blocks(c)
        runs, qb = [], 0
        while qb < keep.shape[0]:
            end = qb + 1
            while end < keep.shape[0] and (keep[end] == keep[qb]).all():
                end += 1
            keys = (np.nonzero(keep[qb])[0][:, None] * B + np.arange(B)).ravel()
            runs.append((qb * B, min(end * B, N), torch.from_numpy(keys[keys < N]).cuda()))
            qb = end
    out = torch.empty((H, N, D), dtype=torch.float64, device="cuda")
    for h in range(H):
        q, k, v = (torch.randn((N, D), generator=g, device="cuda").bfloat16().double()
                   for _ in range(3))
        for a, b, keys in runs:
            ks, vs = k[keys].t().contiguous(), v[keys]
            for i in range(a, b, 2048):
                p = torch.softmax(q[i:min(i + 2048, b)] @ ks * (D ** -0.5), dim=-1)
                out[h, i:min(i + 2048, b)] = p @ vs
    return out
