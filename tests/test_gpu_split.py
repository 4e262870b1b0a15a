"""GPU parity of the launch plans: a launch's tiles run whole (256 query rows)
or split over the key groups of a workgroup (128 or 64 rows), or whole rounds
whole and the rest split, by the number of tiles; 64-token blocks take two key
blocks per step and four query blocks per whole tile.  Shapes on both sides of
each line of the plan (256 CUs), with ragged ends, over random caller CSRs
whose rows differ within a tile (some empty), the token-exact form and dense
attention, against the fp32 oracle on the first and last heads (whole tiles
come first, split ones last)."""
import sys

import numpy as np
import pytest
import torch

import paper_2605_31057_amd as L
from paper_2605_31057_amd.inputs import make_qkv
from oracle import attention as OA
from oracle import mask as M
from tests.gpu_util import assert_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    L.lib()


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _check(out, ref, heads, N, block):
    """Heads `heads` of out against block-wise reference rows."""
    worst, total, count = 0.0, 0.0, 0
    for (h, qb), r in ref.items():
        g = out[heads[h], qb * block: qb * block + r.shape[0]].float().cpu().numpy()
        assert np.isfinite(g).all()
        err = np.abs(g - r)
        worst, total, count = max(worst, float(err.max())), total + float(err.sum()), count + err.size
    assert_close(worst, total / count)


def _random_csr(nb, seed, empty):
    rng = np.random.default_rng(seed)
    rows = []
    for qb in range(nb):
        n = 0 if qb in empty else int(rng.integers(1, nb + 1))
        rows.append(sorted(rng.choice(nb, size=n, replace=False).tolist()))
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    return rp, np.asarray([k for r in rows for k in r], dtype=np.int32)


# heads, tokens: 256-row tiles per launch, and what the plan makes of them.
SHAPES = [
    (2, 1),        #   2: 64-row parts, one token
    (8, 2049),     #  72: 128-row parts, the last part one row
    (64, 1000),    # 256: whole
    (37, 1740),    # 259: whole and 64-row parts
    (40, 2055),    # 360: whole and 128-row parts
    (66, 1793),    # 528: two rounds whole, 64-row parts
]


@pytest.mark.parametrize("block", [128, 64])
@pytest.mark.parametrize("H,N", SHAPES)
def test_random_csr_by_plan(H, N, block):
    _say(f"[split] block form H={H} N={N} B={block}")
    q, k, v = make_qkv(H, N, seed=H + N)
    nb = -(-N // block)
    empty = {nb // 2} if nb > 2 else set()
    rp, ci = _random_csr(nb, H + block, empty)
    m = L.csr_mask(torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), N, block)
    out = torch.full((H, N, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    L.attention(q.cuda(), k.cuda(), v.cuda(), m, out=out)
    dense = L.dense_attention(q.cuda(), k.cuda(), v.cuda(), block=block)
    torch.cuda.synchronize()
    heads = sorted({0, H - 1})
    qs, ks, vs = (x[heads].float().numpy() for x in (q, k, v))
    ref = OA.block_sparse_attention(qs, ks, vs, rp.tolist(), ci.tolist(), block,
                                    q_blocks=[qb for qb in range(nb) if qb not in empty])
    _check(out, ref, heads, N, block)
    frp, fci = [i * nb for i in range(nb + 1)], list(range(nb)) * nb
    _check(dense, OA.block_sparse_attention(qs, ks, vs, frp, fci, block), heads, N, block)
    for qb in empty:
        assert bool((out[:, qb * block:(qb + 1) * block] == 0).all())


@pytest.mark.parametrize("H,N", [(16, 4089), (21, 3200), (22, 3999)])
def test_four_blocks_with_little_in_common(H, N):
    """64-token blocks: whole tiles whose four rows are alike, alike in pairs, or
    disjoint, some empty, side by side; those with little in common are worked in
    parts.  256 whole tiles (no counters), whole tiles beside 64-row parts, and
    beside 128-row parts."""
    _say(f"[split] rows with little in common H={H} N={N}")
    block = 64
    q, k, v = make_qkv(H, N, seed=N)
    nb = -(-N // block)
    rng = np.random.default_rng(N)
    rows = []
    for qb in range(nb):
        i, kind = qb % 4, qb // 4 % 4
        if i == 0:
            base = rng.permutation(nb)
        cols = {0: base[: nb // 2], 1: base[i // 2::2], 2: base[i::4],
                3: base[i::2] if i < 3 else []}[kind]
        rows.append(sorted(int(x) for x in cols))
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.asarray([x for r in rows for x in r], dtype=np.int32)
    m = L.csr_mask(torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), N, block)
    out = torch.full((H, N, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    L.attention(q.cuda(), k.cuda(), v.cuda(), m, out=out)
    torch.cuda.synchronize()
    heads = sorted({0, H // 2, H - 1})
    qs, ks, vs = (x[heads].float().numpy() for x in (q, k, v))
    full = [qb for qb in range(nb) if rows[qb]]
    ref = OA.block_sparse_attention(qs, ks, vs, rp.tolist(), ci.tolist(), block, q_blocks=full)
    _check(out, ref, heads, N, block)
    for qb in set(range(nb)) - set(full):
        assert bool((out[:, qb * block:(qb + 1) * block] == 0).all())
    assert bool(torch.isfinite(out.float()).all())


@pytest.mark.parametrize("block", [128, 64])
@pytest.mark.parametrize("tiles", [2, 84])
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5])
def test_short_walks_of_split_tiles(steps, tiles, block):
    """64-row parts (few tiles) and 128-row parts whose walks are as short as
    the pipeline of tile loads is deep, and one or two steps longer."""
    N = 128 * steps - 5
    H = max(1, tiles // -(-N // 256))
    _say(f"[split] short walks H={H} N={N} B={block}")
    q, k, v = make_qkv(H, N, seed=steps + tiles)
    nb = -(-N // block)
    rp, ci = _random_csr(nb, 7 * steps + block, set())
    m = L.csr_mask(torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), N, block)
    out = L.attention(q.cuda(), k.cuda(), v.cuda(), m)
    dense = L.dense_attention(q.cuda(), k.cuda(), v.cuda(), block=block)
    torch.cuda.synchronize()
    heads = sorted({0, H - 1})
    qs, ks, vs = (x[heads].float().numpy() for x in (q, k, v))
    _check(out, OA.block_sparse_attention(qs, ks, vs, rp.tolist(), ci.tolist(), block), heads, N,
           block)
    frp, fci = [i * nb for i in range(nb + 1)], list(range(nb)) * nb
    _check(dense, OA.block_sparse_attention(qs, ks, vs, frp, fci, block), heads, N, block)


@pytest.mark.parametrize("block", [128, 64])
@pytest.mark.parametrize("H,T,P,text", [(3, 5, 131, 0), (37, 9, 193, 3), (66, 8, 201, 60)])
def test_exact_by_plan(H, T, P, text, block):
    _say(f"[split] exact form H={H} T={T} P={P} text={text} B={block}")
    N = T * P + text
    q, k, v = make_qkv(H, N, seed=H + N)
    csr = L.build_mask(T, P, block, 3, L.Params(window=1, tper=4, text_tokens=text), exact=True)
    csr.upload()
    out = L.attention_exact(q.cuda(), k.cuda(), v.cuda(), csr.exact_mask())
    torch.cuda.synchronize()
    _, _, A = M.attended_frames(T, 3, W=1, tper=4)
    seg = np.minimum(np.arange(N) // P, T)
    att = np.ones((T + 1, T + 1), dtype=bool)
    for t in range(T):
        att[t, :T] = [u in A[t] for u in range(T)]
    keep = att[seg][:, seg]
    worst, total, count = 0.0, 0.0, 0
    for h in (0, H - 1):
        s = (q[h].float() @ k[h].float().t()).numpy() / np.sqrt(128.0)
        s = np.where(keep, s, -np.inf)
        p = np.exp(s - s.max(1, keepdims=True))
        err = np.abs(out[h].float().cpu().numpy() -
                     (p / p.sum(1, keepdims=True)) @ v[h].float().numpy())
        worst, total, count = max(worst, float(err.max())), total + float(err.sum()), count + err.size
    assert_close(worst, total / count)


@pytest.mark.parametrize("block", [128, 64])
@pytest.mark.parametrize("H,N", SHAPES)
def test_weights_add_up_to_one(H, N, block):
    """The same V row at every token comes back bit for bit from every kind of
    tile: the row sums are those of the bf16 probabilities that multiply V, so
    only the fp32 accumulation (relative error below N * 2^-24 <= 2^-12) and the
    exact value's rounding to itself stand between.  Wide logits, whose
    probabilities fall anywhere between two bf16 values."""
    _say(f"[split] constant V H={H} N={N} B={block}")
    q, k, _ = make_qkv(H, N, seed=H + N)
    row = torch.randn(128, generator=torch.Generator().manual_seed(H)).to(torch.bfloat16)
    qd, kd, vd = (q * 4).cuda(), k.cuda(), row.expand(H, N, 128).contiguous().cuda()
    nb = -(-N // block)
    rp, ci = _random_csr(nb, H + block, set())
    m = L.csr_mask(torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), N, block)
    outs = [L.attention(qd, kd, vd, m), L.dense_attention(qd, kd, vd, block=block)]
    P = max(N // 3, block)
    if N > P:
        csr = L.build_mask(N // P, P, block, 0, L.Params(window=0, tper=3, text_tokens=N % P),
                           exact=True)
        csr.upload()
        outs.append(L.attention_exact(qd, kd, vd, csr.exact_mask()))
    torch.cuda.synchronize()
    for out in outs:
        assert torch.equal(out, vd)


@pytest.mark.parametrize("peak", [0.0, 400.0])
def test_reference_is_raised_within_a_walk(peak):
    """Scores that grow along the walk (the walk goes from the last key block
    to the first): the reference is raised by far more than its headroom, step
    after step, and again for one outlying key near the end."""
    H, N = 3, 1500
    q, k, v = make_qkv(H, N, seed=4)
    k *= torch.linspace(40.0, 0.1, N).view(1, N, 1).to(torch.bfloat16)
    if peak:
        k[:, 7] = (q[:, 700] * (peak / 128.0)).to(torch.bfloat16)
    out = L.dense_attention(q.cuda(), k.cuda(), v.cuda())
    torch.cuda.synchronize()
    nb = -(-N // 128)
    ref = OA.block_sparse_attention(q.float().numpy(), k.float().numpy(), v.float().numpy(),
                                    [i * nb for i in range(nb + 1)], list(range(nb)) * nb, 128)
    _check(out, ref, list(range(H)), N, 128)


@pytest.mark.parametrize("H,P,ramp,v_exp", [(64, 333, 30.0, 0), (64, 333, 30.0, -90),
                                            (16, 1363, 350.0, 0), (1, 1363, 350.0, 0)])
@pytest.mark.parametrize("form,block", [("dense", 128), ("block", 128), ("block", 64),
                                        ("exact", 128), ("exact", 64)])
def test_reference_is_raised_in_whole_tiles(form, block, H, P, ramp, v_exp):
    """The same in launches of whole tiles (256 of 256 rows; token-exact with
    64-token blocks 512 of 128): rows whose reference rises by more than either
    headroom, step after step, beside rows that never raise it; V down to
    2^-90, whose products with the smallest references still are normal
    numbers; and walks of 32 steps that would redo nearly all of them (a wave
    takes the row maximum first after 12), also in 64-row parts (one head)."""
    T = 3
    N = P * T + 1
    _say(f"[split] raised reference, {form} B={block} H={H} N={N} V*2^{v_exp}")
    q, k, v = make_qkv(H, N, seed=4)
    q[:, 1::3] *= 0.02
    k *= torch.linspace(ramp, 0.1, N).view(1, N, 1).to(torch.bfloat16)
    k[:, 7] = (q[:, 702] * 3).to(torch.bfloat16)
    vd = (v.float() * 2.0 ** v_exp).to(torch.bfloat16).cuda()
    heads, nb = sorted({0, H - 1}), -(-N // block)
    qs, ks, vs = (x[heads].float().numpy() for x in (q, k, v))
    if form == "exact":
        p = L.Params(window=0, tper=3, text_tokens=1)
        csr = L.build_mask(T, P, block, 0, p, exact=True)
        csr.upload()
        out = L.attention_exact(q.cuda(), k.cuda(), vd, csr.exact_mask())
        _, _, A = M.attended_frames(T, 0, W=0, tper=3)
        seg = np.minimum(np.arange(N) // P, T)
        att = np.ones((T + 1, T + 1), dtype=bool)
        for t in range(T):
            att[t, :T] = [u in A[t] for u in range(T)]
        s = np.where(att[seg][:, seg], qs @ ks.transpose(0, 2, 1) / np.sqrt(128.0), -np.inf)
        pr = np.exp(s - s.max(-1, keepdims=True))
        full = (pr / pr.sum(-1, keepdims=True)) @ vs
        ref = {(h, qb): full[h, qb * block:(qb + 1) * block]
               for h in range(len(heads)) for qb in range(nb)}
    else:
        if form == "block":
            rp, ci = _random_csr(nb, block, set())
            m = L.csr_mask(torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), N, block)
            out = L.attention(q.cuda(), k.cuda(), vd, m)
            rp, ci = rp.tolist(), ci.tolist()
        else:
            rp, ci = [i * nb for i in range(nb + 1)], list(range(nb)) * nb
            out = L.dense_attention(q.cuda(), k.cuda(), vd, block=block)
        ref = OA.block_sparse_attention(qs, ks, vs, rp, ci, block)
    torch.cuda.synchronize()
    _check(out.float() * 2.0 ** -v_exp, ref, heads, N, block)


@pytest.mark.parametrize("form,block", [("block", 128), ("block", 64), ("exact", 128),
                                        ("exact", 64)])
@pytest.mark.parametrize("H,nb128", [(64, 8), (40, 15), (8, 17), (44, 16), (2, 8)])
def test_unkept_key_blocks_do_not_reach_a_query_block(H, nb128, form, block):
    """K and V of a key block may hold anything where a query block does not keep
    it, in every kind of tile: whole ones (256 tiles), whole ones beside 64-row parts,
    128-row parts, whole ones beside 128-row parts, 64-row parts.  Block form:
    key block 5 is kept by the first of every four query blocks only; token-exact
    form: frames of one block, of which frame 5 is attended by itself only."""
    nb = nb128 * 128 // block
    N = nb * block
    _say(f"[split] unkept V {form} B={block} H={H} N={N}")
    q, k, v = (x.cuda() for x in make_qkv(H, N, seed=8))
    for x in (k, v):
        x[:, 5 * block:6 * block] = float("nan")
    if form == "block":
        keep = [[kb for kb in range(nb) if kb != 5 or qb % 4 == 0] for qb in range(nb)]
        rp = torch.tensor([0] + np.cumsum([len(r) for r in keep]).tolist(), dtype=torch.int32)
        ci = torch.tensor([kb for r in keep for kb in r], dtype=torch.int32)
        out = L.attention(q, k, v, L.csr_mask(rp.cuda(), ci.cuda(), N, block))
        keeps = [qb % 4 == 0 for qb in range(nb)]
    else:
        csr = L.build_mask(nb, block, block, 0, L.Params(window=0, window_mode=L.WINDOW_BASIC,
                                                         tper=4), exact=True)
        csr.upload()
        out = L.attention_exact(q, k, v, csr.exact_mask())
        keeps = [qb == 5 for qb in range(nb)]
    torch.cuda.synchronize()
    nan = torch.isnan(out.float()).view(H, nb, block * 128)
    want = torch.tensor(keeps, device="cuda").expand(H, nb)
    assert torch.equal(nan.all(-1), want)    # its own query blocks, in every head
    assert torch.equal(nan.any(-1), want)    # and no other


def test_counted_launches_in_graphs_and_streams():
    """A launch of more tiles than CUs takes tile counters: captured and
    replayed it gives the eager bits, also beside eager launches on another
    stream."""
    H, N, block = 70, 1000, 128
    q, k, v = (x.cuda() for x in make_qkv(H, N, seed=12))
    nb = -(-N // block)
    rp, ci = _random_csr(nb, 5, set())
    m = L.csr_mask(torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), N, block)
    want = L.attention(q, k, v, m)
    out, other = torch.empty_like(q), torch.empty_like(q)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        L.attention(q, k, v, m, out=out, stream=torch.cuda.current_stream())
    for rep in range(4):
        out.fill_(float("nan"))
        other.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        L.attention(q, k, v, m, out=other, stream=side)
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"replay {rep}"
        assert torch.equal(other, want), f"eager launch beside replay {rep}"
