"""GPU: kernels and dispatch branches at the sizes where they can go wrong (edges of tiles and chunks, remainders, the
smallest and largest shapes of their range), through the C ABI, against the CPU oracle on the same inputs."""
import numpy as np
import pytest
import torch

from oracle import madakv_oracle as O
from paper_2506_15724_amd import binding as MB
from paper_2506_15724_amd import workloads as WL
from tests import parity_utils as PU

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(msg):
    print(f"[kernels] {msg}", flush=True)


def workload(name, **kw):
    base = dict(name=name, n_layers=1, batch=1, n_images=1, decode_steps=2)
    L = kw["ctx_len"]
    base.update(image_tokens=(max(1, L // 4), max(1, L // 4)), text_tokens=(1, max(2, L // 8)))
    base.update(kw)
    return WL.CONFIGS["llava_layer"].scaled(**base)


def engine(wl, **kw):
    args = dict(n_layers=wl.n_layers, batch=wl.batch, n_q_heads=wl.n_q_heads, n_kv_heads=wl.n_kv_heads, head_dim=wl.head_dim,
                ctx_len=wl.ctx_len, window=wl.window, budget=wl.budget, dtype=wl.dtype, pool_k=wl.pool_k,
                max_new_tokens=wl.decode_steps, out_fp32=1, device=DEV)
    args.update(kw)
    return MB.MadaKV(**args)


def check_psi(eng, wl, q, k):
    G = wl.n_q_heads // wl.n_kv_heads
    qh, kh, scale = WL.to_f64(q), WL.to_f64(k), PU.oracle_params(wl).scale
    psi_o = np.stack([np.stack([O.window_scores(qh[l, b], kh[l, b], scale) for b in range(wl.batch)]) for l in range(wl.n_layers)])
    nbad, worst = PU.psi_close(eng.psi.cpu().numpy(), psi_o, G, wl.window, wl.ctx_len)
    assert nbad == 0, (wl.name, nbad, worst)
    return worst


@pytest.mark.parametrize("kw", [
    dict(head_dim=64, n_q_heads=2, n_kv_heads=2, window=16, ctx_len=40, budget=24),          # less than one wave's subtiles
    dict(head_dim=64, n_q_heads=3, n_kv_heads=3, window=16, ctx_len=512, budget=64),         # exactly one chunk: no exchange
    dict(head_dim=64, n_q_heads=3, n_kv_heads=3, window=17, ctx_len=513, budget=64),         # one key in the second chunk
    dict(head_dim=128, n_q_heads=2, n_kv_heads=1, window=32, ctx_len=1100, budget=100),      # two row blocks, 128 dims
    dict(head_dim=128, n_q_heads=3, n_kv_heads=1, window=32, ctx_len=900, budget=100),       # 96 rows: two blocks of 64 rows
    dict(head_dim=64, n_q_heads=6, n_kv_heads=2, window=64, ctx_len=700, budget=100),        # 192 rows: three blocks
    dict(head_dim=64, n_q_heads=1, n_kv_heads=1, window=8, ctx_len=32768, budget=300),       # the longest head of the one-sweep kernel
    dict(head_dim=64, n_q_heads=1, n_kv_heads=1, window=8, ctx_len=32769, budget=300),       # one key more: the plain kernels
], ids=lambda kw: f"d{kw['head_dim']}_q{kw['n_q_heads']}_w{kw['window']}_L{kw['ctx_len']}")
def test_fp32_scores(kw, monkeypatch):
    """fp32 queries and keys on the fp32 matrix instructions, all sums in fp32: the tolerance of every psi check
    (1e-3 relative) holds with three digits to spare (fp32 sums of <= 128 products: 1e-5 on a logit)."""
    wl = workload("fp32_scores", dtype="fp32", **kw)
    q, k, v, mask, masks = PU.make_inputs(wl, DEV)
    eng = engine(wl)
    eng.score(0, wl.n_layers, q, k, mask)
    torch.cuda.synchronize()
    worst = check_psi(eng, wl, q, k)
    say(f"{kw}: psi worst scaled error {worst:.2e}")
    assert worst < 1e-4
    one = eng.psi.clone()
    monkeypatch.setenv("MADAKV_SCORE_SPIN_LIMIT", "1")          # workgroups that compute a head's row statistics alone
    eng.score(0, wl.n_layers, q, k, mask)
    torch.cuda.synchronize()
    assert torch.allclose(eng.psi, one, rtol=2e-5, atol=1e-12)
    eng.close()


@pytest.mark.parametrize("kw,lens", [
    # many heads on a small budget: at most two pieces per head, so a long head takes long pieces
    (dict(batch=8, n_q_heads=64, n_kv_heads=64, head_dim=64, ctx_len=6000, budget=128), [5001, 512, 513, 511, 1, 31, 0, 545]),
    (dict(batch=8, n_q_heads=64, n_kv_heads=64, head_dim=128, ctx_len=6000, budget=128, cache_fp8=1), [5001, 512, 513, 511, 1, 32, 0, 545]),
    (dict(batch=8, n_q_heads=128, n_kv_heads=64, head_dim=64, ctx_len=6000, budget=128), [5001, 512, 513, 511, 1, 33, 0, 545]),
    # few heads, grouped queries: pieces of 128 rows; more pieces than the merge has in flight at once
    (dict(n_q_heads=28, n_kv_heads=4, head_dim=128, ctx_len=9000, budget=2000), [6001, 128, 127, 129]),
    (dict(n_q_heads=8, n_kv_heads=1, head_dim=64, ctx_len=9000, budget=4500), [4499]),
    (dict(n_q_heads=12, n_kv_heads=2, head_dim=128, ctx_len=5000, budget=1000, cache_fp8=1), [1700, 159]),
    # grouped queries of 64 dims in large launches: tiles of 32 rows, in longer pieces and, with many heads, in those of 128
    (dict(batch=2, n_q_heads=64, n_kv_heads=8, head_dim=64, ctx_len=9000, budget=4300), [8000, 511, 512, 513, 543, 544, 545, 31, 32, 33, 0, 1]),
    (dict(batch=2, n_q_heads=56, n_kv_heads=8, head_dim=64, ctx_len=9000, budget=4300, cache_fp8=1), [8000, 511, 512, 513, 543, 544, 545, 31, 32, 33, 0, 1]),
    (dict(batch=4, n_q_heads=128, n_kv_heads=64, head_dim=64, ctx_len=2000, budget=200), [1500, 127, 128, 129, 159, 160, 161, 31, 32, 33, 0, 1]),
    (dict(batch=4, n_q_heads=192, n_kv_heads=64, head_dim=64, ctx_len=2000, budget=200, cache_fp8=1), [1500, 127, 128, 129, 159, 160, 161, 31, 32, 33, 0, 1]),
    (dict(n_q_heads=3, n_kv_heads=1, head_dim=128, ctx_len=12000, budget=11000, dtype="fp32"), [10999]),
    (dict(n_q_heads=2, n_kv_heads=2, head_dim=64, ctx_len=400, budget=300, dtype="fp32"), [299, 255]),
    # single queries, little to read: pieces of 128 rows in one trip (by the bytes of a row), heads at their edges and longer than all of them
    (dict(batch=2, n_q_heads=5, n_kv_heads=5, head_dim=128, ctx_len=3000, budget=700), [127, 128, 129, 255, 256, 0, 1, 2990]),
    (dict(batch=2, n_q_heads=5, n_kv_heads=5, head_dim=64, ctx_len=3000, budget=700), [126, 127, 128, 31, 32, 0, 1, 2990]),
    (dict(batch=2, n_q_heads=5, n_kv_heads=5, head_dim=64, ctx_len=3000, budget=700, cache_fp8=1), [126, 127, 128, 63, 64, 0, 1, 2990]),
    (dict(batch=2, n_q_heads=5, n_kv_heads=5, head_dim=128, ctx_len=3000, budget=700, dtype="fp32"), [126, 127, 128, 15, 16, 0, 1, 2990]),
    # long pieces (768 rows): eight rows in flight
    (dict(batch=4, n_q_heads=64, n_kv_heads=64, head_dim=64, ctx_len=7000, budget=6200), [6190, 769, 768, 767, 1]),
], ids=lambda x: f"q{x['n_q_heads']}_kv{x['n_kv_heads']}_d{x['head_dim']}_L{x['ctx_len']}_{x.get('dtype', 'bf16')}" if isinstance(x, dict) else "")
@pytest.mark.parametrize("out_fp32", [1, 0])
def test_decode_pieces(kw, lens, out_fp32):
    """Heads cut into pieces in every way the plan has, an appended row at the edges of pieces and tiles, against a 64-bit
    attention over the rows the cache then holds.  Bound: outputs are means of N(0, 1) rows; a logit of <= 128 fp32
    products (|logit| < 8) is within 1e-5, P as two bf16 parts within 2^-17: 1e-4 covers both; a bf16 output adds half
    a unit of its last place (2^-9 of the value)."""
    args = dict(n_layers=1, batch=1, window=8, dtype="bf16", pool_k=1, max_new_tokens=2, out_fp32=out_fp32)
    args.update(kw)
    eng = MB.MadaKV(device=DEV, **args)
    B, H, Hq, d = args["batch"], args["n_kv_heads"], args["n_q_heads"], args["head_dim"]
    g = torch.Generator().manual_seed(7)
    ln = torch.zeros(B * H, dtype=torch.int32)
    ln[torch.randperm(B * H, generator=g)[:len(lens)]] = torch.tensor(lens, dtype=torch.int32)
    off = torch.cumsum(ln.long() + args["max_new_tokens"], 0) - ln.long() - args["max_new_tokens"]
    used = int(off[-1] + ln[-1]) + args["max_new_tokens"]
    assert used <= eng.capacity
    eng.kv_off.view(-1).copy_(off); eng.kv_len.view(-1).copy_(ln)
    rows = torch.randn(2, used, d, generator=g).to(DEV)
    if args.get("cache_fp8"):
        eng.k_c[:used] = rows[0].to(torch.float8_e4m3fn).view(torch.uint8); eng.v_c[:used] = rows[1].to(torch.float8_e4m3fn).view(torch.uint8)
    else:
        eng.k_c[:used] = rows[0]; eng.v_c[:used] = rows[1]
    f64 = lambda t: (t.view(torch.float8_e4m3fn) if args.get("cache_fp8") else t).cpu().double()
    q, kn, vn = (torch.randn(1, B, h, d, generator=g).to(DEV, eng.tdtype) for h in (Hq, H, H))
    out = torch.empty(1, B, Hq, d, dtype=torch.float32 if out_fp32 else eng.tdtype, device=DEV)
    worst = 0.0
    for step in range(2):
        say(f"{kw} out_fp32={out_fp32} step {step}")
        eng.decode_attn(0, 1, q, kn, vn, out)
        torch.cuda.synchronize()
        assert torch.equal(eng.kv_len.view(-1).cpu(), torch.where(ln > 0, ln + step + 1, ln))
        res = out.view(B * H, Hq // H, d).cpu().double()
        for h in range(B * H):
            n = int(ln[h])
            if n == 0:
                assert torch.isnan(res[h]).all()
                continue
            lo, hi = int(off[h]), int(off[h]) + n + step + 1
            k, v = f64(eng.k_c[lo:hi]), f64(eng.v_c[lo:hi])
            if not args.get("cache_fp8"):
                assert torch.equal(k[-1], kn.view(-1, d)[h].cpu().double()) and torch.equal(v[-1], vn.view(-1, d)[h].cpu().double())
            ref = torch.softmax(q.view(B * H, Hq // H, d)[h].cpu().double() @ k.T / d ** 0.5, -1) @ v
            err = ((res[h] - ref).abs() - (0 if out_fp32 or eng.tdtype == torch.float32 else ref.abs() * 2.0 ** -8)).max()
            worst = max(worst, float(err))
    say(f"worst {worst:.2e}")
    assert worst < 1e-4
    eng.close()


@pytest.mark.parametrize("Hq,H", [(2, 1), (9, 3), (28, 4), (16, 2)])
@pytest.mark.parametrize("kw", [dict(head_dim=128), dict(head_dim=64), dict(head_dim=128, cache_fp8=1), dict(head_dim=64, cache_fp8=1)])
def test_decode_of_grouped_queries_at_tile_edges(Hq, H, kw):
    """Heads whose last tile of 16 rows, last wave and last piece of 128 rows are full, hold one row or are one row short, the
    appended row the first, the last or alone in them: against 64-bit attention over the same rows (the bound of
    test_decode_pieces)."""
    test_decode_pieces(dict(n_q_heads=Hq, n_kv_heads=H, batch=4, ctx_len=2000, budget=300, **kw), [15, 16, 17, 126, 127, 128, 143, 144, 255, 256, 257, 1][:4 * H], 1)


@pytest.mark.parametrize("L,W,M,pool_k,avg", [
    (9, 8, 2, 7, 0), (13, 8, 2, 3, 1), (200, 5, 2, 7, 1), (4096 + 8, 8, 2, 7, 0), (4097 + 8, 8, 3, 5, 0), (16383 + 8, 8, 2, 7, 0),
    (16384 + 8, 8, 4, 1, 0), (16385 + 8, 8, 2, 9, 0), (20483 + 1, 1, 2, 7, 0), (70001, 8, 2, 7, 0), (70001, 8, 3, 5, 1)])
def test_statistics_at_edges(L, W, M, pool_k, avg):
    """Candidate counts at and around the groups, workgroups and chunks of the statistics kernel; one modality's keys point
    away from the queries, so that its masses are tiny (the descent's open lowest bin).  The rules of the stage-wise tests:
    masses on the same psi bits, counts that cross theta within 1e-4, pooled maxima bit for bit (averages of up to nine
    fp32 values: 1e-6 relative)."""
    H, d, nc = 3, 64, L - W
    g = torch.Generator().manual_seed(L + M)
    mask_h = torch.randint(0, M, (1, L), generator=g).to(torch.uint8)
    q = (torch.randn(1, 1, H, W, d, generator=g) + 1.0)
    k = torch.randn(1, 1, H, L, d, generator=g)
    k[0, 0, 1:][:, mask_h[0] == M - 1] -= torch.tensor([1.0, 3.0])[:, None, None]
    q, k, mask = q.to(DEV, torch.bfloat16), k.to(DEV, torch.bfloat16), mask_h.to(DEV)
    eng = MB.MadaKV(n_layers=1, batch=1, n_q_heads=H, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=W + max(1, nc // 3) if nc > 1 else L,
                    dtype="bf16", pool_k=pool_k, pool_mode=avg, n_modalities=M, device=DEV)
    say(f"statistics L={L} W={W} M={M}")
    eng.score(0, 1, q, k, mask)
    torch.cuda.synchronize()
    psi = eng.psi[0, 0].cpu().numpy().astype(np.float64)
    w_g, k_g = eng.stats_host()
    mh = mask_h[0].numpy()
    w_o, k_o, n_o = O.modality_stats(psi, mh, W, 0.9, 0, M)
    assert tuple(eng.n_mod.cpu().numpy()[0]) == tuple(n_o)
    PU.assert_masses_close(w_g[0, 0], w_o, nc)
    pool_o = O.pool_scores(psi, W, pool_k, avg).astype(np.float32)
    pool_g = eng.psi_pool[0, 0].cpu().numpy()
    if avg:
        np.testing.assert_allclose(pool_g, pool_o, rtol=1e-6)
    else:
        np.testing.assert_array_equal(pool_g, pool_o)
    for h in range(H):
        for m in range(M):
            vals = psi[h, :nc][mh[:nc] == m]
            # (a mass of a few units of the 2^-44 fixed point says nothing about theta)
            if k_g[0, 0, h, m] != k_o[h, m] and vals.sum() > 1e4 * max(1, vals.size) * 2.0 ** -44:
                assert PU.k_count_ok(int(k_g[0, 0, h, m]), vals, 0.9), (h, m, k_g[0, 0, h, m], k_o[h, m])
    eng.close()


@pytest.mark.parametrize("L,W,M", [(12, 8, 2), (15, 8, 2), (200, 5, 2), (4096 + 8, 8, 2), (4097 + 8, 8, 3), (16383 + 8, 8, 2), (16384 + 8, 8, 4),
                                   (16385 + 8, 8, 2), (20483 + 1, 1, 4), (70001, 8, 2), (70001, 8, 3)])
def test_selection_at_edges(L, W, M):
    """Kept positions, bit for bit, at and around the groups, workgroups and chunks of the selection kernel, with scores
    inside and outside the range the descent's first level is made for, plateaus of ties across its passes, and
    negative scores."""
    H, d, nc = 6, 64, L - W
    r = np.random.default_rng(L * 7 + M)
    mh = r.integers(0, M, size=L).astype(np.uint8)
    pool = np.exp(r.normal(size=(H, nc)) * 2 - 8).astype(np.float32)
    pool[1] *= 1e-12                                             # all below the first level's range
    pool[2] *= 1e9                                               # all above it
    pool[3] = np.repeat(pool[3][::53], 53)[:nc]                  # plateaus
    pool[4] = -pool[4]
    pool[5] = np.where(r.random(nc) < 0.5, 0.0, pool[5])         # many zeros
    n_m = np.array([(mh[:nc] == m).sum() for m in range(M)])
    bud = np.stack([(n_m * f).astype(np.int32) for f in (0.3, 0.9, 0.01, 0.5, 0.2, 0.8)])
    eng = MB.MadaKV(n_layers=1, batch=1, n_q_heads=H, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=L - 1, dtype="bf16",
                    pool_k=1, n_modalities=M, device=DEV)
    k = torch.zeros(1, 1, H, L, d, dtype=torch.bfloat16, device=DEV)
    say(f"selection L={L} W={W} M={M}")
    eng.select_gather(0, 1, k, k, torch.from_numpy(mh)[None].to(DEV), psi_pool=torch.from_numpy(pool)[None, None].to(DEV),
                      budgets=torch.from_numpy(bud)[None, None].to(DEV))
    torch.cuda.synchronize()
    kept, off, ln = eng.kept_idx.cpu().numpy(), eng.kv_off.cpu().numpy()[0, 0], eng.kv_len.cpu().numpy()[0, 0]
    for h in range(H):
        ref = O.select_n(pool[h].astype(np.float64), mh, [int(x) for x in bud[h]], L, W)
        np.testing.assert_array_equal(kept[off[h]:off[h] + ln[h]], ref)
    eng.close()


@pytest.mark.parametrize("Hq,H,W,d,L", [(8, 1, 9, 64, 65), (8, 1, 9, 128, 63), (12, 2, 16, 128, 700), (12, 2, 16, 64, 1025), (28, 4, 32, 128, 2049),
                                        (16, 2, 32, 64, 4097), (7, 1, 10, 128, 1088), (8, 1, 32, 128, 9000), (6, 2, 40, 64, 20011)])
@pytest.mark.parametrize("out_fp32", [1, 0])
def test_window_attention_many_rows(Hq, H, W, d, L, out_fp32):
    """The last-window attention with 65 to 256 proxy rows per KV head (four and eight waves, ragged last blocks, tiles and
    chunks, fewer keys than a tile) against 64-bit arithmetic on the same bf16 inputs.  Logits of <= 128 exact products summed
    in fp32 are within 1e-5, P as two or three bf16 parts within 2^-17: 2e-5 of the result in the 2-norm, 4e-5 on a log-sum-exp;
    a bf16 output adds half a unit of its last place."""
    G, B = Hq // H, 2
    g = torch.Generator().manual_seed(L)
    q, k, v = (torch.randn(1, B, h, n, d, generator=g).to(DEV, torch.bfloat16) for h, n in ((Hq, W), (H, L), (H, L)))
    mask = torch.randint(0, 2, (B, L), generator=g).to(torch.uint8).to(DEV)
    eng = MB.MadaKV(n_layers=1, batch=B, n_q_heads=Hq, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=W + max(1, (L - W) // 2), dtype="bf16",
                    pool_k=7, out_fp32=out_fp32, device=DEV)
    out = torch.full((1, B, Hq, W, d), float("nan"), dtype=torch.float32 if out_fp32 else torch.bfloat16, device=DEV)
    lse = torch.full((1, B, Hq, W), float("nan"), dtype=torch.float32, device=DEV)
    say(f"window {Hq}/{H} W={W} d={d} L={L} out_fp32={out_fp32}")
    for _ in range(2):
        eng.window_attn_score(0, 1, q, k, v, mask, out, lse)
    torch.cuda.synchronize()
    for b in range(B):
        for h in range(H):
            qq = q[0, b, h * G:(h + 1) * G].cpu().double().reshape(G * W, d)
            x = qq @ k[0, b, h].cpu().double().T / d ** 0.5
            pos = (L - W + torch.arange(W)).repeat(G)
            x = x.masked_fill(torch.arange(L)[None] > pos[:, None], float("-inf"))
            p = torch.softmax(x, -1)
            ref = p @ v[0, b, h].cpu().double()
            got = out[0, b, h * G:(h + 1) * G].cpu().double().reshape(G * W, d)
            err = float((got - ref).norm() / ref.norm())
            assert err < (2e-5 if out_fp32 else 2.0 ** -9), err
            assert float((lse[0, b, h * G:(h + 1) * G].cpu().double().reshape(-1) - torch.logsumexp(x, -1)).abs().max()) < 4e-5
            nbad, worst = PU.psi_close(eng.psi[0, b, h].cpu().numpy()[None], p.sum(0).numpy()[None], G, W, L)
            assert nbad == 0, (nbad, worst)
    eng.close()


def minus_inf_case(dtype, Hq, H, W, d, L, where, NL=1):
    """Queries whose first element is negative, keys of which those at `where` hold +Inf there: every row's logit on such
    a key is -Inf, its softmax entry and its psi are 0, everything else is as if the key were not there."""
    g = torch.Generator().manual_seed(L + Hq)
    q, k, v = (torch.randn(NL, 1, h, n, d, generator=g) for h, n in ((Hq, W), (H, L), (H, L)))
    q[..., 0] = -q[..., 0].abs() - 0.25
    k[..., list(where), 0] = float("inf")
    mask = torch.randint(0, 2, (1, L), generator=g).to(torch.uint8).to(DEV)
    q, k, v = (t.to(DEV, torch.bfloat16 if dtype == "bf16" else torch.float32) for t in (q, k, v))
    eng = MB.MadaKV(n_layers=NL, batch=1, n_q_heads=Hq, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=W + (L - W) // 2, dtype=dtype,
                    pool_k=1, out_fp32=1, device=DEV)
    return eng, q, k, v, mask


def softmax_rows(q, k, W, kv_head):
    """64-bit softmax entries [G * W, L] of one KV head's proxy rows, and their log-sum-exp"""
    G, L, d = q.shape[0] // k.shape[0], k.shape[1], k.shape[2]
    x = q[kv_head * G:(kv_head + 1) * G].cpu().double().reshape(G * W, d) @ k[kv_head].cpu().double().T / d ** 0.5
    pos = (L - W + torch.arange(W)).repeat(G)
    x = x.masked_fill(torch.arange(L)[None] > pos[:, None], float("-inf"))
    return torch.softmax(x, -1), torch.logsumexp(x, -1)


@pytest.mark.parametrize("G,W,d,L", [(3, 43, 128, 700), (4, 40, 128, 4100), (7, 23, 64, 2100), (6, 32, 128, 64), (3, 64, 64, 1500),
                                      (7, 32, 128, 3000), (5, 45, 128, 1030)], ids=lambda x: str(x))
def test_scores_where_waves_own_one_or_two_row_blocks(G, W, d, L):
    """Five to eight blocks of 32 proxy rows for four waves (129, 160, 161, 192, 224 and 225 rows), whose second block is left out where
    it is empty, in chunks that start the round of the waves anywhere.  The tolerance of every psi check (1e-3)."""
    wl = workload("row_blocks", n_q_heads=3 * G, n_kv_heads=3, head_dim=d, window=W, ctx_len=max(L, W + 24), budget=W + 16)
    q, k, v, mask, masks = PU.make_inputs(wl, DEV)
    eng = engine(wl)
    say(f"row blocks {G * W} rows d={d} L={wl.ctx_len}")
    eng.score(0, 1, q, k, mask)
    torch.cuda.synchronize()
    assert check_psi(eng, wl, q, k) < 1e-4
    eng.close()


@pytest.mark.parametrize("top,base", [(-105, 0), (0, 0), (-105, -300)], ids=["far_below", "above", "all_low"])
@pytest.mark.parametrize("dtype,H,W,d,L", [("bf16", 2, 32, 128, 4100), ("bf16", 2, 64, 128, 3900), ("bf16", 2, 17, 64, 3000),
                                            ("bf16", 2, 64, 64, 2500), ("fp32", 2, 16, 64, 2048), ("fp32", 2, 40, 128, 1500)])
def test_scores_far_from_a_waves_first_keys(dtype, H, W, d, L, top, base):
    """Keys whose logits are up to 2^95, or 2^200, times those of the first keys that their wave sees, while the row's normaliser is
    2^200 times those: the terms' factor alone would flush to zero, or the terms pass what they are kept for.  Or
    all that 2^300 lower, where a row that sees none of a wave's keys has nothing to be scaled up.  Logits are at most 500 (log2),
    rounded to 2^-24 of that a few times: 1e-4 relative; 1e-3 is allowed, down to the smallest normal numbers."""
    g = torch.Generator().manual_seed(L + W)
    want = torch.empty(H, L).uniform_(-195, top, generator=g)                # a key's logit, log2
    want[:, :1024] = 0.
    want[:, (torch.arange(L) >= 1024) & (torch.arange(L) % 1024 < 128)] = -200.
    if W > 32:                                   # (768 keys per chunk)
        want[:, (torch.arange(L) >= 768) & (torch.arange(L) % 768 < 128)] = -200.
    q, k = 0.25 * torch.randn(1, 1, H, W, d, generator=g), 0.5 * torch.randn(1, 1, H, L, d, generator=g)
    q[..., 0] = 4.
    k[0, 0, :, :, 0] = (want + base) * (d ** 0.5 / (4. * 1.4427))
    q, k = (t.to(DEV, torch.bfloat16 if dtype == "bf16" else torch.float32) for t in (q, k))
    mask = torch.randint(0, 2, (1, L), generator=g).to(torch.uint8).to(DEV)
    eng = MB.MadaKV(n_layers=1, batch=1, n_q_heads=H, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=W + L // 4, dtype=dtype,
                    pool_k=1, out_fp32=1, device=DEV)
    say(f"scores far from a wave's first keys {dtype} H={H} W={W} d={d} L={L} top={top} base={base}")
    eng.score(0, 1, q, k, mask)
    torch.cuda.synchronize()
    for h in range(H):
        ref = softmax_rows(q[0, 0], k[0, 0], W, h)[0].sum(0)
        err = (eng.psi[0, 0, h].cpu().double() - ref).abs()
        assert (err <= 1e-3 * ref + 2.0 ** -125 * W).all(), float((err / ref).max())
    eng.close()


def logits_by_chunk(shape, L, chunk, top, base, g):
    """Logits (log2) for keys in chunks of `chunk`: 0 in the first chunk, then by turns a chunk whose waves' first keys (its first 128) are
    at -200 and whose others are anywhere up to `top`, and one of ordinary keys.  All of them `base` lower.  top = "steps": chunks whose first
    keys are at -130, the next up to -35 and the others up to 0, and where those that follow are another 130 higher."""
    i = torch.arange(L)
    if top == "steps":
        most = torch.tensor([0., 95., 130., 130., 260., 260., 260., 260.])[i % chunk // 128]
        want = torch.rand(*shape, L, generator=g) * most - (260. if chunk > 512 else 130.)
    else:
        want = torch.empty(*shape, L).uniform_(-195, top, generator=g)
        want[..., i % chunk < 128] = -200.
    ordinary = i // chunk % 2 == 0
    want[..., ordinary] = torch.empty(*shape, int(ordinary.sum())).uniform_(-20, 0, generator=g)
    want[..., :chunk] = 0.
    return want + base


@pytest.mark.parametrize("top,base", [(-105, 0), (0, 0), (-105, -300), ("steps", 0)], ids=["far_below", "above", "all_low", "steps"])
@pytest.mark.parametrize("dtype,H,W,d,L,chunk", [("fp32", 2, 16, 64, 9000, 256), ("fp32", 2, 40, 128, 9000, 256), ("fp32", 1, 40, 64, 17000, 512),
                                                  ("fp32", 1, 16, 128, 17000, 512), ("bf16", 1, 64, 64, 131072, 768), ("bf16", 1, 20, 128, 70000, 1024),
                                                  ("bf16", 2, 40, 128, 5000, 768), ("bf16", 3, 32, 64, 6000, 1024)])
def test_scores_far_from_a_waves_first_keys_by_chunk(dtype, H, W, d, L, chunk, top, base):
    """As above, for fp32 in the longer chunks (2 and 4 subtiles per wave), where some keys of a wave are not among its first, and for heads
    of more than 64 chunks, in whose exchange of two levels workgroups of both kinds meet (and, with 171 chunks, the one that
    only leaves its logits)."""
    g = torch.Generator().manual_seed(L + W)
    q, k = 0.25 * torch.randn(1, 1, H, W, d, generator=g), 0.5 * torch.randn(1, 1, H, L, d, generator=g)
    q[..., 0] = 4.
    k[0, 0, :, :, 0] = logits_by_chunk((H,), L, chunk, top, base, g) * (d ** 0.5 / (4. * 1.4427))
    q, k = (t.to(DEV, torch.bfloat16 if dtype == "bf16" else torch.float32) for t in (q, k))
    mask = torch.randint(0, 2, (1, L), generator=g).to(torch.uint8).to(DEV)
    eng = MB.MadaKV(n_layers=1, batch=1, n_q_heads=H, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=W + L // 4, dtype=dtype,
                    pool_k=1, out_fp32=1, device=DEV)
    say(f"scores by chunk {dtype} H={H} W={W} d={d} L={L} top={top} base={base}")
    eng.score(0, 1, q, k, mask)
    torch.cuda.synchronize()
    for h in range(H):
        ref = softmax_rows(q[0, 0], k[0, 0], W, h)[0].sum(0)
        err = (eng.psi[0, 0, h].cpu().double() - ref).abs()
        assert (err <= 1e-3 * ref + 2.0 ** -125 * W).all(), float((err / ref).max())
    eng.close()


@pytest.mark.parametrize("W,L,chunk", [(32, 16384, 1024), (64, 65536, 768)])
def test_time_of_scores_does_not_depend_on_where_the_large_ones_are(W, L, chunk):
    """Keys far above those that their wave sees first: 1.05 times the time of ordinary ones (1.6 and 1.5 with a second pass over them)."""
    H, us = 32, {}
    q, mask = torch.randn(1, 1, H, W, 128, device=DEV, dtype=torch.bfloat16), torch.zeros(1, L, dtype=torch.uint8, device=DEV)
    q[..., 0] = 16.
    k = torch.randn(1, 1, H, L, 128, device=DEV, dtype=torch.bfloat16)
    eng = MB.MadaKV(n_layers=1, batch=1, n_q_heads=H, n_kv_heads=H, head_dim=128, ctx_len=L, window=W, budget=2048, device=DEV)
    for far in (0, 1):
        k[..., 0] = torch.where(torch.arange(L, device=DEV) % chunk < 128, -200. * far * 128 ** 0.5 / (16. * 1.4427), 0.)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(22)]
        for e in ev:
            eng.score(0, 1, q, k, mask)
            e.record()
        torch.cuda.synchronize()
        us[far] = sorted(a.elapsed_time(b) for a, b in zip(ev[1:], ev[2:]))[10] * 1e3
    eng.close()
    say(f"scores of {H} heads of {L} keys, {W} rows: {us[0]:.0f} us, large ones far from the first {us[1]:.0f} us")
    assert us[1] < 1.3 * us[0]


@pytest.mark.parametrize("Hq,H,W,d,L,dtype", [(2, 2, 16, 64, 700, "bf16"), (2, 2, 40, 128, 3000, "bf16"), (2, 2, 16, 128, 2100, "bf16"),
                                              (3, 1, 16, 64, 500, "fp32"), (2, 2, 16, 128, 9000, "fp32"), (1, 1, 16, 64, 17000, "fp32")], ids=lambda x: str(x))
@pytest.mark.parametrize("log2", [11, 20, 23, 24, 26, 30, 40])
def test_scores_of_large_logits(Hq, H, W, d, L, dtype, log2):
    """Logits of +-2^11 to 2^40, of which fp32 holds a short fraction or none: a quarter of the keys have the one, the others the
    other, so every proxy row pays the same to each of the visible keys that have the larger one and nothing to the rest.  A logit and a
    row's max + log2(sum) are rounded by half a unit of their last place, 2^(log2 - 24), a score by that many times ln 2 in all.  Beyond 2^23 the sum of a row
    is lost in that; the keys with the larger logit still score above the others."""
    g = torch.Generator().manual_seed(L)
    sign = torch.where(torch.rand(H, L, generator=g) < 0.25, 1., -1.)
    sign[:, 512:640] = sign[:, L - W:] = -1.                                          # (waves whose first keys have the smaller one alone)
    a = (2.0 ** log2 / (2.1 * d ** 0.5)) ** 0.5
    q, k = torch.full((1, 1, Hq, W, d), a), 1.3 * a * sign[None, None, :, :, None].expand(1, 1, H, L, d)
    q, k = (t.contiguous().to(DEV, torch.bfloat16 if dtype == "bf16" else torch.float32) for t in (q, k))
    q[:, :, 0] *= -1.                                                                 # (a head whose large logits are the others')
    mask = torch.randint(0, 2, (1, L), generator=g).to(torch.uint8).to(DEV)
    eng = MB.MadaKV(n_layers=1, batch=1, n_q_heads=Hq, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=W + L // 4, dtype=dtype,
                    pool_k=1, out_fp32=1, device=DEV)
    say(f"logits of 2^{log2} {dtype} {Hq}/{H} W={W} d={d} L={L}")
    eng.score(0, 1, q, k, mask)
    torch.cuda.synchronize()
    for h in range(H):
        psi, ref = eng.psi[0, 0, h].cpu().double(), softmax_rows(q[0, 0], k[0, 0], W, h)[0].sum(0)
        assert torch.isfinite(psi).all() and (psi[ref > 1e-9] > 0).all() and (psi[ref <= 1e-9] == 0).all()
        if log2 <= 23:
            err = (psi - ref).abs()
            assert (err <= (1e-5 + 0.7 * 2.0 ** (log2 - 24)) * ref).all(), float((err / ref.clamp_min(1e-30)).max())
    eng.close()


@pytest.mark.parametrize("dtype,H,W,d,L", [("bf16", 4, 32, 128, 4100), ("bf16", 4, 64, 64, 3900), ("fp32", 4, 16, 64, 2048)])
@pytest.mark.parametrize("spin", [None, "1"])
def test_scores_of_a_head_with_a_key_that_is_no_number(dtype, H, W, d, L, spin, monkeypatch):
    """Every proxy row sees the key, so no score of its head is a number, in whichever chunk and also where a workgroup stopped
    waiting and went its own way; the other heads' scores are as ever."""
    g = torch.Generator().manual_seed(L)
    q, k = torch.randn(1, 1, H, W, d, generator=g), torch.randn(1, 1, H, L, d, generator=g)
    k[0, 0, 0, L - W - 3, 5], k[0, 0, 2, 7, 0] = float("nan"), float("nan")
    mask = torch.randint(0, 2, (1, L), generator=g).to(torch.uint8).to(DEV)
    q, k = (t.to(DEV, torch.bfloat16 if dtype == "bf16" else torch.float32) for t in (q, k))
    eng = MB.MadaKV(n_layers=1, batch=1, n_q_heads=H, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=W + L // 4, dtype=dtype,
                    pool_k=1, out_fp32=1, device=DEV)
    if spin:
        monkeypatch.setenv("MADAKV_SCORE_SPIN_LIMIT", spin)          # workgroups that find a word missing go their own way
    eng.score_ws.zero_()
    say(f"a key that is no number {dtype} H={H} W={W} d={d} L={L} spin={spin}")
    eng.score(0, 1, q, k, mask)
    torch.cuda.synchronize()
    say(f"{int(eng.score_ws[:4].view(torch.int32)[0])} workgroups went their own way")
    assert torch.isnan(eng.psi[0, 0, 0::2]).all()
    for h in range(1, H, 2):
        nbad, worst = PU.psi_close(eng.psi[0, 0, h].cpu().numpy()[None], softmax_rows(q[0, 0], k[0, 0], W, h)[0].sum(0).numpy()[None], 1, W, L)
        assert nbad == 0, (nbad, worst)
    eng.close()


@pytest.mark.parametrize("Hq,H,W,d,L,where", [
    (3, 3, 17, 64, 600, [5]), (3, 3, 32, 64, 1100, range(0, 512)), (5, 1, 9, 128, 1100, [31, 32, 700]), (5, 1, 9, 128, 1100, range(512, 1024)),
    (7, 1, 10, 64, 900, [0, 600]), (2, 2, 16, 64, 400, range(0, 128))],
    ids=lambda x: str(len(x)) if isinstance(x, (list, range)) else str(x))
def test_fp32_scores_of_keys_with_infinite_elements(Hq, H, W, d, L, where):
    """Padding rows (row counts that are no multiple of 32) and waves or chunks that see nothing but -Inf leave no NaN."""
    eng, q, k, v, mask = minus_inf_case("fp32", Hq, H, W, d, L, where)
    say(f"fp32 scores with infinite key elements {Hq}/{H} W={W} d={d} L={L}")
    eng.score(0, 1, q, k, mask)
    torch.cuda.synchronize()
    psi = eng.psi[0, 0].cpu()
    for h in range(H):
        p, _ = softmax_rows(q[0, 0], k[0, 0], W, h)
        assert (psi[h, list(where)] == 0).all()
        nbad, worst = PU.psi_close(psi[h].numpy()[None], p.sum(0).numpy()[None], Hq // H, W, L)
        assert nbad == 0, (nbad, worst)
    eng.close()


@pytest.mark.parametrize("NL,Hq,H,W,d,L,where", [
    (1, 7, 1, 10, 128, 1088, [40]), (1, 7, 1, 10, 64, 1088, range(0, 128)), (8, 48, 16, 23, 64, 4200, [40, 3000]), (8, 56, 8, 21, 128, 4200, [0, 900])],
    ids=lambda x: str(len(x)) if isinstance(x, (list, range)) else str(x))
def test_window_attention_of_keys_with_infinite_elements(NL, Hq, H, W, d, L, where):
    """As above, more than 64 proxy rows that are no multiple of 32, in calls of few and of many heads."""
    eng, q, k, v, mask = minus_inf_case("bf16", Hq, H, W, d, L, where, NL)
    out = torch.empty(NL, 1, Hq, W, d, dtype=torch.float32, device=DEV)
    say(f"window with infinite key elements {NL} x {Hq}/{H} W={W} d={d} L={L}")
    eng.window_attn_score(0, NL, q, k, v, mask, out)
    torch.cuda.synchronize()
    assert (eng.psi[..., list(where)] == 0).all()
    G = Hq // H
    for l in (0, NL - 1):
        for h in (0, H - 1):
            p, _ = softmax_rows(q[l, 0], k[l, 0], W, h)
            nbad, worst = PU.psi_close(eng.psi[l, 0, h].cpu().numpy()[None], p.sum(0).numpy()[None], G, W, L)
            assert nbad == 0, (nbad, worst)
            ref = p @ v[l, 0, h].cpu().double()
            assert float((out[l, 0, h * G:(h + 1) * G].cpu().double().reshape(G * W, d) - ref).norm() / ref.norm()) < 2e-5
    eng.close()


@pytest.mark.parametrize("NL,Hq,H,W,d,L", [
    (18, 36, 12, 22, 64, 64), (18, 36, 12, 22, 128, 65), (18, 36, 12, 22, 128, 63),                    # fewest keys of a tile, and one less: the blocks
    (6, 128, 32, 24, 64, 1025), (14, 32, 8, 32, 128, 1024), (7, 96, 16, 16, 128, 1600), (5, 84, 28, 32, 128, 1537),   # 3 and 4 blocks of rows
    (10, 40, 8, 31, 128, 2100), (26, 64, 8, 29, 64, 700), (26, 64, 8, 32, 128, 129),                   # 5 and 8 blocks
    (1, 8, 1, 32, 128, 65536 + 700), (2, 3, 1, 32, 64, 131072), (1, 7, 1, 30, 128, 100003),            # few long heads: many chunks each
    (8, 4, 1, 32, 64, 32768 - 31), (20, 32, 8, 32, 64, 768), (20, 32, 8, 32, 64, 769)],                # either side of the dispatch
    ids=lambda x: str(x))
@pytest.mark.parametrize("out_fp32", [1, 0])
def test_window_attention_many_rows_many_workgroups(NL, Hq, H, W, d, L, out_fp32):
    """As test_window_attention_many_rows, in calls large enough for the kernel that takes all rows in one pass, and at the
    edges of its dispatch and of its chunks; the first, last and some other heads against 64-bit arithmetic (same bounds)."""
    G = Hq // H
    g = torch.Generator(device=DEV).manual_seed(L + Hq)
    q, k, v = (torch.randn(NL, 1, h, n, d, generator=g, device=DEV).to(torch.bfloat16) for h, n in ((Hq, W), (H, L), (H, L)))
    mask = torch.randint(0, 2, (1, L), generator=g, device=DEV).to(torch.uint8)
    eng = MB.MadaKV(n_layers=NL, batch=1, n_q_heads=Hq, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=W + max(1, (L - W) // 4), dtype="bf16",
                    pool_k=7, out_fp32=out_fp32, device=DEV)
    out = torch.full((NL, 1, Hq, W, d), float("nan"), dtype=torch.float32 if out_fp32 else torch.bfloat16, device=DEV)
    lse = torch.full((NL, 1, Hq, W), float("nan"), dtype=torch.float32, device=DEV)
    eng.psi.fill_(float("nan"))
    say(f"window {NL} x {Hq}/{H} W={W} d={d} L={L} out_fp32={out_fp32}")
    for _ in range(2):
        eng.window_attn_score(0, NL, q, k, v, mask, out, lse)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all() and torch.isfinite(lse).all() and torch.isfinite(eng.psi).all()
    for l, h in {(0, 0), (NL - 1, H - 1), (NL // 2, H // 2), (NL // 3, H // 3)}:
        p, ls = softmax_rows(q[l, 0], k[l, 0], W, h)
        ref = p @ v[l, 0, h].cpu().double()
        err = float((out[l, 0, h * G:(h + 1) * G].cpu().double().reshape(G * W, d) - ref).norm() / ref.norm())
        assert err < (2e-5 if out_fp32 else 2.0 ** -9), err
        assert float((lse[l, 0, h * G:(h + 1) * G].cpu().double().reshape(-1) - ls).abs().max()) < 4e-5
        nbad, worst = PU.psi_close(eng.psi[l, 0, h].cpu().numpy()[None], p.sum(0).numpy()[None], G, W, L)
        assert nbad == 0, (nbad, worst)
    eng.close()


def test_window_attention_of_one_long_head_fills_the_chip():
    """One layer of one KV head (256 rows, 128K keys) has a quarter of the work of four heads and must not take longer:
    a fixed number of chunks per head left it to a sixteenth of the compute units (690 us against 560; 174 and 266 with
    chunks by the launch)."""
    us = {}
    for H in (1, 4):
        q, k, v = (torch.randn(1, 1, h, n, 128, device=DEV, dtype=torch.bfloat16) for h, n in ((8 * H, 32), (H, 131072), (H, 131072)))
        mask = torch.zeros(1, 131072, dtype=torch.uint8, device=DEV)
        eng = MB.MadaKV(n_layers=1, batch=1, n_q_heads=8 * H, n_kv_heads=H, head_dim=128, ctx_len=131072, window=32, budget=2048, out_fp32=0, device=DEV)
        out = torch.empty(1, 1, 8 * H, 32, 128, dtype=torch.bfloat16, device=DEV)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(12)]
        for e in ev:
            eng.window_attn_score(0, 1, q, k, v, mask, out)
            e.record()
        torch.cuda.synchronize()
        us[H] = min(a.elapsed_time(b) for a, b in zip(ev[1:], ev[2:])) * 1e3
        eng.close()
    say(f"one long head {us[1]:.0f} us, four {us[4]:.0f} us")
    assert us[1] < us[4]


def evicted_engine(lens, **kw):
    """An engine whose heads (one layer, one batch item) hold `lens` rows after a selection with hand-made budgets."""
    args = dict(n_layers=1, batch=1, window=8, dtype="bf16", pool_k=1, max_new_tokens=16, out_fp32=1)
    args.update(kw)
    eng = MB.MadaKV(device=DEV, **args)
    H, L, W, d = args["n_kv_heads"], args["ctx_len"], args["window"], args["head_dim"]
    g = torch.Generator().manual_seed(11)
    k, v = (torch.randn(1, 1, H, L, d, generator=g).to(DEV, eng.tdtype) for _ in range(2))
    mask = torch.zeros(1, L, dtype=torch.uint8, device=DEV)
    bud = torch.zeros(1, 1, H, 2, dtype=torch.int32)
    bud[0, 0, :, 0] = torch.tensor(lens) - W
    eng.select_gather(0, 1, k, v, mask, psi_pool=torch.rand(1, 1, H, L - W, generator=g).to(DEV), budgets=bud.to(DEV))
    torch.cuda.synchronize()
    assert eng.kv_len.view(-1).tolist() == list(lens)
    return eng, args


def like_without_known_lengths(eng, args):
    """The same reduced cache in a handle that has made no eviction and so knows nothing of the heads' lengths."""
    other = MB.MadaKV(device=DEV, **args)
    for name in ("k_c", "v_c", "kv_off", "kv_len"):
        getattr(other, name).copy_(getattr(eng, name))
    return other


@pytest.mark.parametrize("kw,lens", [
    (dict(n_q_heads=4, n_kv_heads=4, head_dim=128, ctx_len=1500, budget=250), [249, 120, 9, 31]),           # one piece each, grows to two
    (dict(n_q_heads=4, n_kv_heads=1, head_dim=64, ctx_len=1500, budget=130), [121]),                        # grouped queries: pieces of 128 rows
    (dict(n_q_heads=14, n_kv_heads=2, head_dim=128, ctx_len=1500, budget=130, cache_fp8=1), [127, 126]),
    (dict(n_q_heads=2, n_kv_heads=2, head_dim=64, ctx_len=1500, budget=256, dtype="fp32"), [254, 200]),
    (dict(n_q_heads=6, n_kv_heads=3, head_dim=128, ctx_len=9000, budget=700, hcc_rho=1), [1400, 128, 300]), # more rows than the average head's
    (dict(n_q_heads=32, n_kv_heads=32, head_dim=64, ctx_len=9000, budget=400, hcc_rho=64), [5100, 2550, 2560, 100] + [40] * 28),   # many times the average
    (dict(n_q_heads=64, n_kv_heads=16, head_dim=128, ctx_len=9000, budget=600, hcc_rho=1024), [7000, 1270, 511] + [30] * 13),
], ids=lambda x: f"q{x['n_q_heads']}_kv{x['n_kv_heads']}_d{x['head_dim']}_{x.get('dtype', 'bf16')}" if isinstance(x, dict) else "")
def test_decode_known_lengths(kw, lens):
    """The launch is sized by the heads' lengths once the host knows them (nobody meets anybody while every head is one piece): the same
    bits as without, at every step of a growth across a piece's end, and the lengths of the heads grow by one."""
    eng, args = evicted_engine(lens, **kw)
    other = like_without_known_lengths(eng, args)
    H, Hq, d = args["n_kv_heads"], args["n_q_heads"], args["head_dim"]
    g = torch.Generator().manual_seed(5)
    for step in range(16):
        q, kn, vn = (torch.randn(1, 1, h, d, generator=g).to(DEV, eng.tdtype) for h in (Hq, H, H))
        outs = []
        for e in (eng, other):
            out = torch.full((1, 1, Hq, d), float("nan"), device=DEV)
            say(f"known lengths {kw} step {step}")
            e.decode_attn(0, 1, q, kn, vn, out)
            torch.cuda.synchronize()
            outs.append(out)
            assert e.kv_len.view(-1).tolist() == [n + step + 1 for n in lens]
        assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])
    eng.close(); other.close()


def test_decode_of_short_heads_merges_nothing():
    """Heads of one piece each have nobody to meet once that is known, and no workgroups that only arrive: 3.8 against 4.5 us
    per call."""
    eng, args = evicted_engine([120] * 32, n_q_heads=32, n_kv_heads=32, head_dim=128, ctx_len=4096, budget=120)
    us = []
    for e in (eng, like_without_known_lengths(eng, args)):
        q, out = torch.randn(1, 1, 32, 128, device=DEV).to(e.tdtype), torch.empty(1, 1, 32, 128, device=DEV)
        for _ in range(2):
            e.decode_attn(0, 1, q, None, None, out)
            torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(50):
                e.decode_attn(0, 1, q, None, None, out)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(12)]
        for x in ev:
            graph.replay()
            x.record()
        torch.cuda.synchronize()
        us.append(min(x.elapsed_time(y) for x, y in zip(ev[1:], ev[2:])) * 20)
        e.close()
    say(f"short heads: {us[0]:.2f} us per call, lengths unknown {us[1]:.2f}")
    assert us[0] < 0.95 * us[1]


@pytest.mark.parametrize("kw,lens", [
    (dict(n_layers=16, n_q_heads=512, n_kv_heads=64, head_dim=128, ctx_len=600, budget=56), [200, 130, 255]),     # 1024 heads x 8 queries
    (dict(n_layers=8, n_q_heads=512, n_kv_heads=64, head_dim=128, ctx_len=900, budget=100), [600, 385, 384]),     # 512: short pieces, three at most
    (dict(n_layers=2, n_q_heads=56, n_kv_heads=14, head_dim=128, ctx_len=24000, budget=2000, hcc_rho=16), [20000, 9100, 3000]),
], ids=lambda x: f"heads{x['n_layers'] * x['n_kv_heads']}" if isinstance(x, dict) else "")
def test_decode_static_cuts_heads_like_the_workspace_call(kw, lens):
    """The call without a workspace, whose scratch is small, gives the same bits wherever it is accepted."""
    args = dict(batch=1, window=8, dtype="bf16", pool_k=1, max_new_tokens=8, out_fp32=1)
    args.update(kw)
    NL, H, Hq, L, W, d = (args[x] for x in ("n_layers", "n_kv_heads", "n_q_heads", "ctx_len", "window", "head_dim"))
    g = torch.Generator(device=DEV).manual_seed(11)
    k, v = (torch.randn(NL, 1, H, L, d, generator=g, device=DEV).to(torch.bfloat16) for _ in range(2))
    ln = torch.full((NL * H,), 24, dtype=torch.int32)
    ln[7::7][:len(lens)] = torch.tensor(lens, dtype=torch.int32)
    assert int(ln.sum()) <= NL * H * args["budget"]
    bud = torch.stack([ln - W, torch.zeros_like(ln)], -1).view(NL, 1, H, 2).to(DEV)
    eng = MB.MadaKV(device=DEV, **args)
    eng.select_gather(0, NL, k, v, torch.zeros(1, L, dtype=torch.uint8, device=DEV), budgets=bud, psi_pool=torch.rand(NL, 1, H, L - W, generator=g, device=DEV))
    torch.cuda.synchronize()
    assert torch.equal(eng.kv_len.view(-1).cpu(), ln)
    q = torch.randn(NL, 1, Hq, d, generator=g, device=DEV).to(torch.bfloat16)
    out, out_static = torch.empty(NL, 1, Hq, d, device=DEV), torch.empty(NL, 1, Hq, d, device=DEV)
    say(f"static {kw}")
    eng.decode_attn(0, NL, q, None, None, out)
    torch.cuda.synchronize()
    eng.decode_attn_static(0, NL, q, None, None, out_static)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all() and torch.equal(out, out_static)
    eng.close()


@pytest.mark.parametrize("kw,lens", [
    (dict(n_q_heads=64, n_kv_heads=64, head_dim=64, ctx_len=30000, budget=25000, page_rows=64), [24990, 769, 768, 767, 64, 63] + [40] * 58),   # pieces of 768 rows
    (dict(n_q_heads=14, n_kv_heads=2, head_dim=128, ctx_len=2000, budget=400, page_rows=64), [128, 640]),       # grouped queries: pieces of 128 rows
    (dict(n_q_heads=8, n_kv_heads=1, head_dim=64, ctx_len=2000, budget=400, page_rows=16, cache_fp8=1), [255]),
    (dict(n_q_heads=8, n_kv_heads=4, head_dim=128, ctx_len=9000, budget=6000, page_rows=256, hcc_rho=16), [8000, 512, 1, 256 + 128]),
    (dict(n_q_heads=64, n_kv_heads=16, head_dim=64, ctx_len=9000, budget=4300, page_rows=64), [8000, 512, 511, 256, 240, 32, 16] + [40] * 9),     # 64 dims: tiles of 32 rows
    (dict(n_q_heads=32, n_kv_heads=16, head_dim=64, ctx_len=9000, budget=4300, page_rows=16, cache_fp8=1), [8000, 512, 511, 256, 240, 32, 16] + [40] * 9),
    (dict(n_q_heads=4, n_kv_heads=4, head_dim=128, ctx_len=2000, budget=400, page_rows=32, cache_fp8=1), [256, 255, 512, 33]),
    (dict(n_q_heads=6, n_kv_heads=2, head_dim=128, ctx_len=1500, budget=600, page_rows=16, dtype="fp32"), [512, 271]),
    # single queries, little to read: pieces of 128 rows in one trip, the last head longer than all of them
    (dict(n_q_heads=4, n_kv_heads=4, head_dim=128, ctx_len=2000, budget=400, page_rows=16), [128, 127, 256, 1060]),
    (dict(n_q_heads=4, n_kv_heads=4, head_dim=64, ctx_len=2000, budget=400, page_rows=64, dtype="fp32"), [128, 127, 256, 1060]),
    (dict(n_q_heads=4, n_kv_heads=4, head_dim=128, ctx_len=2000, budget=400, page_rows=16, dtype="fp32"), [128, 127, 256, 1060]),
], ids=lambda x: f"q{x['n_q_heads']}_kv{x['n_kv_heads']}_d{x['head_dim']}_P{x['page_rows']}_{x.get('dtype', 'bf16')}" if isinstance(x, dict) else "")
def test_decode_pieces_paged(kw, lens):
    """The kernels' paged forms at the edges of pieces, tiles and pages, the appended row being the first of a piece and of a
    page among them: bit for bit what contiguous segments give, which 64-bit attention confirms at the last step."""
    flat, args = evicted_engine([max(n, 9) for n in lens], max_new_tokens=40, **{k: v for k, v in kw.items() if k != "page_rows"})
    paged, _ = evicted_engine([max(n, 9) for n in lens], max_new_tokens=40, **kw)
    H, Hq, d, n0 = args["n_kv_heads"], args["n_q_heads"], args["head_dim"], flat.kv_len.view(-1).tolist()
    g = torch.Generator().manual_seed(2)
    for step in range(34):
        q, kn, vn = (torch.randn(1, 1, h, d, generator=g).to(DEV, flat.tdtype) for h in (Hq, H, H))
        outs = [torch.full((1, 1, Hq, d), float("nan"), device=DEV) for _ in range(2)]
        say(f"paged pieces {kw} step {step}")
        for e, out in zip((flat, paged), outs):
            e.decode_attn(0, 1, q, kn, vn, out)
        torch.cuda.synchronize()
        assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])
        assert flat.kv_len.view(-1).tolist() == paged.kv_len.view(-1).tolist() == [n + step + 1 for n in n0]
    f64 = lambda t: (t.view(torch.float8_e4m3fn) if args.get("cache_fp8") else t).cpu().double()
    off = flat.kv_off.view(-1).tolist()
    for h in range(H):
        k, v = (f64(x[off[h]:off[h] + n0[h] + 34]) for x in (flat.k_c, flat.v_c))
        ref = torch.softmax(q.view(H, Hq // H, d)[h].cpu().double() @ k.T / d ** 0.5, -1) @ v
        assert float((outs[0].view(H, Hq // H, d)[h].cpu().double() - ref).abs().max()) < 1e-4          # (the bound of test_decode_pieces)
    flat.close(); paged.close()


@pytest.mark.parametrize("top,base", [(-105, 0), (0, 0), (-105, -300), ("steps", 0)], ids=["far_below", "above", "all_low", "steps"])
@pytest.mark.parametrize("G,W,d,fp8", [(2, 16, 128, 1), (8, 8, 64, 1), (4, 16, 128, 1), (4, 24, 64, 1), (8, 16, 128, 1), (3, 7, 64, 0), (4, 24, 128, 0)])
def test_reeviction_scores_far_from_a_waves_first_keys(G, W, d, fp8, top, base):
    """test_scores_far_from_a_waves_first_keys_by_chunk on the ragged rows of a reduced cache, of 8 bits and of 16, with up to 64 proxy rows and with
    more (blocks of 64).  The reference reads what the cache holds."""
    lens = [3000, 1100, 200, 40]
    eng, args = evicted_engine(lens, n_q_heads=4 * G, n_kv_heads=4, head_dim=d, ctx_len=3200, budget=1200, window=W, cache_fp8=fp8)
    g = torch.Generator().manual_seed(G * W + d)
    q = 0.25 * torch.randn(1, 1, 4 * G, W, d, generator=g)
    q[..., 0] = 16.                                    # (so that a key's element is one of 8 bits)
    q = q.to(torch.bfloat16)
    off, keys = eng.kv_off.view(-1).tolist(), []
    for h, n in enumerate(lens):
        k = 0.5 * torch.randn(n, d, generator=g)
        k[:, 0] = logits_by_chunk((), n, 1024 if G * W <= 32 else 768, top, base, g) * (d ** 0.5 / (16. * 1.4427))
        k = k.to(torch.float8_e4m3fn if fp8 else torch.bfloat16)
        eng.k_c[off[h]:off[h] + n] = (k.view(torch.uint8) if fp8 else k).to(DEV)
        keys.append(k.double())
    say(f"re-eviction scores G={G} W={W} d={d} fp8={fp8} top={top} base={base}")
    eng.reevict(0, 1, q.to(DEV), torch.zeros(1, args["ctx_len"], dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    psi = eng.reevict_ws[:eng.capacity * 4].view(torch.float32).cpu().double()
    for h, n in enumerate(lens):
        ref = softmax_rows(q[0, 0, h * G:(h + 1) * G], keys[h][None], W, 0)[0].sum(0)
        err = (psi[off[h]:off[h] + n] - ref).abs()
        assert (err <= 1e-3 * ref + 2.0 ** -125 * G * W).all(), (h, float((err / ref).max()))
    eng.close()


@pytest.mark.parametrize("kw", [dict(head_dim=128), dict(head_dim=64, n_q_heads=8), dict(head_dim=128, cache_fp8=1), dict(head_dim=64, page_rows=16)],
                         ids=lambda kw: "_".join(f"{k}{v}" for k, v in kw.items()))
@pytest.mark.parametrize("steps,goes", [(0, "none"), (1, "first"), (1, "last"), (5, "first"), (5, "spread"), (12, "late"), (12, "first")])
def test_compaction_at_edges(kw, steps, goes):
    """Re-eviction where the first row that goes is the first of the head, the last candidate, as late as it can be (all the
    last proxy rows and appended candidates) or none: known rows go by construction, the others stay bit for bit and in
    order, with their positions.  Heads around the number of rows the kernel moves at a time."""
    W, lens = 8, [40, 255, 256, 257]
    eng, args = evicted_engine(lens, n_kv_heads=4, ctx_len=1200, budget=300, **dict(dict(n_q_heads=4), **kw))
    d, Hq = args["head_dim"], args["n_q_heads"]
    g = torch.Generator().manual_seed(steps + 1)
    drop = []
    for n in lens:
        cand = n + steps - W
        drop.append({"none": [], "first": [0] + list(range(cand - steps + 1, cand)), "last": [cand - 1], "late": list(range(n - W, n - W + steps)),
                     "spread": [0, 7, 20, cand - 2, cand - 1]}[goes])
        assert len(set(drop[-1])) == steps and all(0 <= r < cand for r in drop[-1])
    def row(head, i):                    # a row's K: against the queries (q = 4) if it goes, with them if it stays
        return (-0.5 if i in drop[head] else 0.5) + 0.05 * torch.randn(d, generator=g)
    off = eng.kv_off.view(-1).tolist()
    store = lambda t: t.to(torch.float8_e4m3fn).view(torch.uint8) if args.get("cache_fp8") else t.to(eng.tdtype)
    for h, n in enumerate(lens):
        eng.k_c[off[h]:off[h] + n] = store(torch.stack([row(h, i) for i in range(n)])).to(DEV)
    q = torch.full((1, 1, Hq, d), 4.0, device=DEV, dtype=eng.tdtype)
    out = torch.empty(1, 1, Hq, d, device=DEV)
    for t in range(steps):
        kn = torch.stack([row(h, n + t) for h, n in enumerate(lens)]).view(1, 1, 4, d).to(DEV, eng.tdtype)
        eng.decode_attn(0, 1, q, kn, torch.randn(1, 1, 4, d, generator=g).to(DEV, eng.tdtype), out)
    torch.cuda.synchronize()

    def rows_of(h, n):                   # where the rows of a head are
        if not args.get("page_rows"):
            return list(range(off[h], off[h] + n))
        P, tbl = args["page_rows"], eng.page_table_host()[0, 0, h]
        return [off[h] + r if r < tbl[0] * P else int(tbl[1 + (r - tbl[0] * P) // P]) * P + (r - tbl[0] * P) % P for r in range(n)]
    at = [rows_of(h, n + steps) for h, n in enumerate(lens)]
    k0, v0, idx0 = [[x[a].clone() for a in at] for x in (eng.k_c, eng.v_c, eng.kept_idx)]
    say(f"compaction {kw} steps={steps} {goes}")
    eng.reevict(0, 1, q[:, :, :, None].expand(1, 1, Hq, W, d).contiguous(), torch.zeros(1, args["ctx_len"], dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    assert eng.kv_len.view(-1).tolist() == lens
    for h, n in enumerate(lens):
        stay = [r for r in range(n + steps) if r not in drop[h]]
        now = rows_of(h, n)
        assert torch.equal(eng.k_c[now], k0[h][stay]) and torch.equal(eng.v_c[now], v0[h][stay])
        want = [int(idx0[h][r]) if r < n else args["ctx_len"] + r - n for r in stay]
        assert eng.kept_idx[now].tolist() == want
    eng.close()


@pytest.mark.parametrize("dtype,Hq,d,rows", [("fp32", 1, 128, 2 ** 23 + 4000), ("bf16", 4, 128, 2 ** 24 + 4000)])
def test_decode_beyond_4_gib_of_rows(dtype, Hq, d, rows):
    """A head whose K rows take more than 4 GiB: all its weight is on four rows beyond that, the output is their mean
    (the other rows' logits are 0 against 60: 2^24 e^-60 of the weight)."""
    slack = 64
    eng = MB.MadaKV(n_layers=1, batch=1, n_q_heads=Hq, n_kv_heads=1, head_dim=d, ctx_len=64, window=8, budget=16, dtype=dtype, pool_k=1,
                    max_new_tokens=rows + slack, out_fp32=1, device=DEV)
    g = torch.Generator().manual_seed(3)
    eng.k_c.zero_(); eng.v_c.zero_()
    eng.kv_off.zero_(); eng.kv_len.fill_(rows)
    q = torch.ones(1, 1, Hq, d, device=DEV, dtype=eng.tdtype)
    at = torch.tensor([rows - 3900, rows - 2049, rows - 1000])
    vals = torch.randn(4, d, generator=g).to(eng.tdtype)
    eng.k_c[at.to(DEV)] = 60 / d ** 0.5
    eng.v_c[at.to(DEV)] = vals[:3].to(DEV)
    kn = torch.full((1, 1, 1, d), 60 / d ** 0.5, device=DEV, dtype=eng.tdtype)
    out = torch.empty(1, 1, Hq, d, device=DEV)
    say(f"decode over {rows} rows of {d} {dtype}")
    eng.decode_attn(0, 1, q, kn, vals[3:].view(1, 1, 1, d).to(DEV), out)
    torch.cuda.synchronize()
    assert int(eng.kv_len) == rows + 1
    ref = vals.double().mean(0)
    assert float((out[0, 0].cpu().double() - ref).abs().max()) < 1e-5
    eng.close()


def test_calls_use_the_current_stream(monkeypatch):
    """The handle the binding hands to the library is that of torch's current stream, with and without torch's shortcut."""
    side = torch.cuda.Stream()
    shortcut = MB._raw_stream
    for raw in (shortcut, lambda device: torch.cuda.current_stream(device).cuda_stream):
        monkeypatch.setattr(MB, "_raw_stream", raw)
        assert MB._stream() == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(side):
            assert MB._stream() == side.cuda_stream


@pytest.mark.parametrize("kw", [dict(n_q_heads=5, n_kv_heads=5, head_dim=128), dict(n_q_heads=5, n_kv_heads=5, head_dim=64, dtype="fp32"),
                                dict(n_q_heads=35, n_kv_heads=5, head_dim=128), dict(n_q_heads=10, n_kv_heads=5, head_dim=64),
                                dict(n_q_heads=15, n_kv_heads=5, head_dim=128, dtype="fp32"), dict(n_q_heads=5, n_kv_heads=5, head_dim=64, cache_fp8=1)],
                         ids=lambda kw: "_".join(f"{k}{v}" for k, v in kw.items()))
def test_decode_pieces_that_come_into_being(kw):
    """Heads that grow into pieces which held nothing before, with many workgroups that only arrive (room for 700 appended
    rows): two layers in turn, two steps on two streams one behind the other, calls that append nothing in between; lengths after every call and the
    last output against a 64-bit attention (bound: that of test_decode_pieces)."""
    lens = [255, 256, 511, 127, 384]
    args = dict(dict(n_layers=2, batch=1, window=8, dtype="bf16", pool_k=1, ctx_len=1200, budget=400, max_new_tokens=700, out_fp32=1), **kw)
    eng = MB.MadaKV(device=DEV, **args)
    H, Hq, d, L = args["n_kv_heads"], args["n_q_heads"], args["head_dim"], args["ctx_len"]
    g = torch.Generator().manual_seed(4)
    k, v = (torch.randn(2, 1, H, L, d, generator=g).to(DEV, eng.tdtype) for _ in range(2))
    bud = torch.stack([torch.tensor(lens + lens) - 8, torch.zeros(2 * H, dtype=torch.int64)], -1).view(2, 1, H, 2).to(DEV, torch.int32)
    eng.select_gather(0, 2, k, v, torch.zeros(1, L, dtype=torch.uint8, device=DEV), psi_pool=torch.rand(2, 1, H, L - 8, generator=g).to(DEV), budgets=bud)
    side = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [torch.full((1, 1, Hq, d), float("nan"), device=DEV) for _ in range(2)]
    for step in range(4):
        rows = [[torch.randn(1, 1, h, d, generator=g).to(DEV, eng.tdtype) for h in (Hq, H, H)] for _ in range(2)]
        torch.cuda.synchronize()
        say(f"growing pieces {kw} step {step}")
        for l in (0, 1):
            with torch.cuda.stream(side[l] if step >= 2 else torch.cuda.current_stream()):
                torch.cuda.current_stream().wait_stream(side[1 - l])          # calls on one handle do not overlap
                eng.decode_attn(l, 1, *rows[l], outs[l])
        torch.cuda.synchronize()
        assert eng.kv_len.view(-1).tolist() == [n + step + 1 for n in lens + lens]
        again = [torch.empty_like(outs[l]) for l in (0, 1)]
        for l in (0, 1):
            eng.decode_attn(l, 1, rows[l][0], None, None, again[l])
        torch.cuda.synchronize()
        assert eng.kv_len.view(-1).tolist() == [n + step + 1 for n in lens + lens]
        assert all(torch.isfinite(outs[l]).all() and torch.equal(outs[l], again[l]) for l in (0, 1))
    f64 = lambda t: (t.view(torch.float8_e4m3fn) if args.get("cache_fp8") else t).cpu().double()
    off = eng.kv_off.view(-1).tolist()
    for l in (0, 1):
        for h in range(H):
            lo, hi = off[l * H + h], off[l * H + h] + lens[h] + 4
            k, v = f64(eng.k_c[lo:hi]), f64(eng.v_c[lo:hi])
            ref = torch.softmax(rows[l][0].view(H, Hq // H, d)[h].cpu().double() @ k.T / d ** 0.5, -1) @ v
            assert float((outs[l].view(H, Hq // H, d)[h].cpu().double() - ref).abs().max()) < 1e-4
    eng.close()


@pytest.mark.parametrize("L,W,M", [(3000, 8, 2), (9001, 8, 3), (20000, 8, 2), (40001, 8, 2), (70001, 8, 2), (70001, 8, 3), (200001, 16, 2)])
def test_statistics_of_crowded_bins(L, W, M, monkeypatch):
    """Scores so close together that the bin where the running mass crosses theta holds a few, hundreds (ranked, or walked once
    more), thousands (more than a workgroup's list, or than the chunk's share of the head's) or all of the candidates, equal ones
    among them; two layers in one call, one after the other and in two groups.  The rules of test_statistics_at_edges."""
    scale = [0.0, 0.001, 0.01, 0.03, 0.1, 0.4]
    H, d, nc = len(scale), 64, L - W
    g = torch.Generator().manual_seed(L + M)
    mask_h = torch.randint(0, M, (1, L), generator=g).to(torch.uint8)
    q = torch.randn(2, 1, H, W, d, generator=g).to(DEV, torch.bfloat16)
    k = (torch.randn(2, 1, H, L, d, generator=g) * torch.tensor(scale)[None, None, :, None, None]).to(DEV, torch.bfloat16)
    eng = MB.MadaKV(n_layers=2, batch=1, n_q_heads=H, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=W + nc // 3, dtype="bf16", pool_k=7,
                    n_modalities=M, device=DEV)
    mask, mh = mask_h.to(DEV), mask_h[0].numpy()
    say(f"crowded bins L={L} M={M}")
    eng.score(0, 2, q, k, mask)
    torch.cuda.synchronize()
    w_g, k_g = eng.stats_host()
    pool = eng.psi_pool.clone()
    for l in range(2):
        eng.score(l, 1, q[l:l + 1], k[l:l + 1], mask)
        torch.cuda.synchronize()
    w_1, k_1 = eng.stats_host()
    assert np.array_equal(w_g, w_1) and np.array_equal(k_g, k_1) and torch.equal(pool, eng.psi_pool)
    monkeypatch.setenv("MADAKV_LAYER_GROUPS", "2")              # the kernels that fit beside a gather
    eng.evict(0, 2, q, k, k, mask)
    torch.cuda.synchronize()
    w_1, k_1 = eng.stats_host()
    assert np.array_equal(w_g, w_1) and np.array_equal(k_g, k_1) and torch.equal(pool, eng.psi_pool)
    for l in range(2):
        psi = eng.psi[l, 0].cpu().numpy().astype(np.float64)
        w_o, k_o, _ = O.modality_stats(psi, mh, W, 0.9, 0, M)
        PU.assert_masses_close(w_g[l, 0], w_o, nc)
        for h in range(H):
            for m in range(M):
                if k_g[l, 0, h, m] != k_o[h, m]:
                    assert PU.k_count_ok(int(k_g[l, 0, h, m]), psi[h, :nc][mh[:nc] == m], 0.9), (l, h, m, k_g[l, 0, h, m], k_o[h, m])
    eng.close()


@pytest.mark.parametrize("L,M", [(9000, 2), (9000, 3), (20001, 2), (40001, 2), (70001, 2), (70001, 4), (200001, 2)])
def test_selection_of_crowded_bins(L, M, monkeypatch):
    """Kept positions, bit for bit, where the threshold is among 2 to 5000 scores of one bin (or all of them), at and around
    what is ranked at once and what a list holds, in bins of either width and next to their boundary, with ties; two layers in
    one call, one after the other and in two groups."""
    W, d, nc = 8, 64, L - 8
    sizes = [2, 63, 65, 255, 257, 1023, 1025, 2047, 2049, 5000, nc]
    H = len(sizes)
    r = np.random.default_rng(L + M)
    mh = r.integers(0, M, size=L).astype(np.uint8)
    pool = np.empty((2, H, nc), dtype=np.float32)
    bud = np.zeros((2, H, M), dtype=np.int32)
    for l in range(2):
        for h, n in enumerate(sizes):
            at = (2.0 ** -3, 2.0 ** -16, 2.0 ** -20 * 1.01)[(h + l) % 3]           # the crowd: 1 / 128 wide, from `at` on
            row = np.where(r.random(nc) < 0.3, at * 8 * (1 + r.random(nc)), at / 8 * r.random(nc))
            for m in range(M):
                who = r.permutation(np.flatnonzero(mh[:nc] == m))[:n]
                row[who] = at * (1 + r.integers(0, max(2, n // 2), size=len(who)) / max(2, n // 2) / 128)
                above = int(((row > at * 2) & (mh[:nc] == m)).sum())
                bud[l, h, m] = above + max(1, int(len(who) * (0.1, 0.5, 0.97)[m % 3]))
            pool[l, h] = row
    eng = MB.MadaKV(n_layers=2, batch=1, n_q_heads=H, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=L - 1, dtype="bf16", pool_k=1,
                    n_modalities=M, device=DEV)
    k = torch.zeros(2, 1, H, L, d, dtype=torch.bfloat16, device=DEV)
    args = dict(psi_pool=torch.from_numpy(pool)[:, None].to(DEV), budgets=torch.from_numpy(bud)[:, None].to(DEV))
    mask = torch.from_numpy(mh)[None].to(DEV)
    say(f"crowded selection L={L} M={M}")
    eng.select_gather(0, 2, k, k, mask, **args)
    torch.cuda.synchronize()
    kept, off, ln = eng.kept_idx.clone(), eng.kv_off.cpu().numpy()[:, 0], eng.kv_len.cpu().numpy()[:, 0]
    for l in range(2):
        eng.select_gather(l, 1, k[l:l + 1], k[l:l + 1], mask, **{x: t[l:l + 1] for x, t in args.items()})
    torch.cuda.synchronize()
    used = int(off[-1, -1] + ln[-1, -1])
    assert torch.equal(kept[:used], eng.kept_idx[:used])
    monkeypatch.setenv("MADAKV_LAYER_GROUPS", "2")              # the kernel that fits beside a gather
    eng.kept_idx.fill_(-1)
    eng.select_gather(0, 2, k, k, mask, **args)
    torch.cuda.synchronize()
    assert torch.equal(kept[:used], eng.kept_idx[:used])
    kept = kept.cpu().numpy()
    for l in range(2):
        for h in range(H):
            ref = O.select_n(pool[l, h].astype(np.float64), mh, [int(x) for x in bud[l, h]], L, W)
            np.testing.assert_array_equal(kept[off[l, h]:off[l, h] + ln[l, h]], ref)
    eng.close()


@pytest.mark.parametrize("kw", [
    dict(head_dim=64, n_q_heads=2, n_kv_heads=2, window=16, ctx_len=129, budget=40),         # one key in the second chunk of 128
    dict(head_dim=64, n_q_heads=3, n_kv_heads=3, window=16, ctx_len=9000, budget=200),       # chunks of 256 keys
    dict(head_dim=128, n_q_heads=20, n_kv_heads=20, window=32, ctx_len=1025, budget=100),    # chunks of 256 keys, 128 dims
    dict(head_dim=128, n_q_heads=32, n_kv_heads=32, window=33, ctx_len=1100, budget=100),    # of 512, two row blocks
], ids=lambda kw: f"d{kw['head_dim']}_q{kw['n_q_heads']}_w{kw['window']}_L{kw['ctx_len']}")
def test_fp32_scores_by_size(kw):
    """The chunks of the fp32 kernel by the size of the model (tolerance: test_fp32_scores); the layers of a model one by one
    give the bits of one call."""
    wl = workload("fp32_sizes", dtype="fp32", n_layers=2, **kw)
    q, k, v, mask, masks = PU.make_inputs(wl, DEV)
    eng = engine(wl)
    eng.score(0, 2, q, k, mask)
    torch.cuda.synchronize()
    worst = check_psi(eng, wl, q, k)
    say(f"{kw}: psi worst scaled error {worst:.2e}")
    assert worst < 1e-4
    one = eng.psi.clone()
    eng.psi.zero_()
    for l in range(2):
        eng.score(l, 1, q[l:l + 1], k[l:l + 1], mask)
    torch.cuda.synchronize()
    assert torch.equal(one, eng.psi)
    eng.close()


@pytest.mark.parametrize("kw", [dict(ctx_len=5000, budget=600), dict(ctx_len=66000, budget=1500, n_layers=1), dict(ctx_len=3000, budget=300, page_rows=16)],
                         ids=lambda kw: f"L{kw['ctx_len']}")
def test_first_call_is_captured(kw):
    """A handle's first work is captured on a stream that waits for nobody and replayed while the null stream still has in front
    of it what it had when the handle was made: eviction (chunks that meet in the handle's words and records) and decode over
    several pieces (the handle's counters).  Every replay against the same calls made eagerly, bit for bit."""
    paged = kw.get("page_rows", 0)
    kw = {x: y for x, y in kw.items() if x != "page_rows"}
    wl = workload("captured", **dict(dict(n_layers=2, head_dim=128, n_q_heads=4, n_kv_heads=2, window=16), **kw))
    NL = wl.n_layers
    q, k, v, mask, masks = PU.make_inputs(wl, DEV)
    dq, dk, dv = (torch.randn(NL, 1, h, wl.head_dim, device=DEV).to(torch.bfloat16) for h in (wl.n_q_heads, wl.n_kv_heads, wl.n_kv_heads))
    outs = [torch.full((NL, 1, wl.n_q_heads, wl.head_dim), float("nan"), device=DEV) for _ in range(2)]

    def calls(eng, out):
        eng.evict(0, NL, q, k, v, mask)
        for l in range(NL):
            eng.decode_attn(l, 1, dq[l:l + 1], dk[l:l + 1], dv[l:l + 1], out[l:l + 1])

    eager = engine(wl, page_rows=paged)
    calls(eager, outs[0])
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    say(f"captured first call {kw}")
    torch.cuda._sleep(20_000_000)
    eng = engine(wl, page_rows=paged)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        graph.capture_begin()
        calls(eng, outs[1])
        graph.capture_end()
    for replay in range(3):
        with torch.cuda.stream(side):
            graph.replay()
        side.synchronize()
        for name in ("psi", "psi_pool", "stats", "budgets", "kv_len", "kv_off"):
            assert torch.equal(getattr(eng, name), getattr(eager, name)), (replay, name)
        assert torch.equal(outs[0], outs[1]), replay
        outs[1].fill_(float("nan"))
        torch.cuda.synchronize()
    del graph
    eng.close(); eager.close()
