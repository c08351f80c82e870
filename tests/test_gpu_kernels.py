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
