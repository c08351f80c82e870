"""What the library's calls do on the host (allocations, clears, launches, waits), on a runtime that only keeps a log
(fake_hip.cpp).  No GPU: every scenario is a program of its own, in which that runtime stands in front of the real one."""
import os
import subprocess
import sys
import textwrap

import pytest

from paper_2506_15724_amd import binding as MB
from paper_2506_15724_amd import build as B
from tests.test_abi import good

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
fake.fake_log.restype = C.c_char_p
class Line:
    def __init__(self, s): self.kind, *self.rest = s.split(" ")
    def __repr__(self): return " ".join([self.kind, *self.rest[:5]])
def log():
    lines = [Line(s) for s in fake.fake_log().decode().splitlines()]
    fake.fake_clear()
    return lines
def num(s): return 0 if s == "(nil)" else int(s, 16)
P, I, Z = C.c_void_p, C.c_int32, C.c_size_t
def create(hexed):
    h = P()
    assert lib.madakv_create(bytes.fromhex(hexed), C.byref(h)) == 0
    return h
class Room:                                     # stands for a device tensor: an address with so many bytes behind it
    at = 1 << 44
    def __init__(self, size):
        self.size, self.p = size, Room.at
        Room.at += (size + 4095) // 4096 * 4096
    def has(self, x): return self.p <= x < self.p + self.size
    def __bool__(self): return True
def T(size=1 << 30): return Room(size)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host") / "fake_hip.so")
    subprocess.check_call(["g++", "-shared", "-fPIC", "-O1", "-std=c++17", os.path.join(HERE, "fake_hip.cpp"), "-o", so])
    return so


def scenario(runtime, body, *configs):
    """Runs `body` with the configurations (bytes in hex) as sys.argv[3:]; its assertions are the test's."""
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), runtime, B.LIB, *[bytes(c).hex() for c in configs]],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_creation_leaves_no_clear_behind(runtime):
    """The memory that calls rely on (carry state, arrival counters, exchange words, records of split heads) is clear when
    madakv_create returns: a first call may be on any stream, and may be one that is captured and replayed later, so nothing
    can make it wait.  A captured first call launches its kernels and nothing else."""
    out = scenario(runtime, """
        for hexed in sys.argv[3:]:
            h = create(hexed)
            lines = log()
            open_streams = set()
            cleared = 0
            for x in lines:
                if x.kind == "memset":
                    open_streams.add(x.rest[3]); cleared += 1
                    assert x.rest[3] != "(nil)", "the null stream holds whatever the caller has put there"
                if x.kind == "stream_wait": open_streams.discard(x.rest[0])
            assert cleared and not open_streams, lines
            s = 0x77000
            fake.fake_capture(P(s))
            rc = lib.madakv_allocate(h, I(0), I(1), P(T().p), P(T().p), P(T().p), P(s))
            assert rc == 0 and [x.kind for x in log()] == ["launch"]
            fake.fake_capture(P(0))
            rc = lib.madakv_allocate(h, I(0), I(1), P(T().p), P(T().p), P(T().p), P(s))
            assert rc == 0 and [x.kind for x in log()] == ["launch"]
            lib.madakv_destroy(h)
        print("ok")
        """, good(), good(ctx_len=131072, window=64, budget=4096), good(page_rows=16), good(n_layers=28, n_q_heads=28, n_kv_heads=4))
    assert out.strip() == "ok"


def test_exchange_words_after_a_failed_launch(runtime):
    """The words in which the workgroups of a head exchange row statistics are empty when a call begins, also after one whose
    statistics (which empty them) could not be launched: they are emptied at once, so that a graph that was captured before
    finds them so; if that fails too, in front of the next scores, which are not launched without it.  A clear that is only
    captured has not happened yet."""
    body = """
        h = create(sys.argv[3])
        NL = 8
        s, s2 = 0x77000, 0x88000
        def score(st):
            return lib.madakv_score(h, I(0), I(NL), P(T().p), P(T().p), P(T().p), P(T().p), P(T().p), P(T().p), P(T().p), P(T().p), Z(1 << 30), P(st))
        def evict(st):
            t = [P(T().p) for _ in range(14)]
            return lib.madakv_evict(h, I(0), I(NL), *t, P(T().p), Z(1 << 30), P(T().p), Z(1 << 30), P(st))
        def kinds():
            what = dict(clear="xchg_init", score="score_fused")
            return [(x.kind, next((w for w in what if what[w] in str(x)), ""), x.rest[0]) for x in log() if x.kind in ("launch", "failed")]
        launched = lambda k, what: [x for x in k if x[0] == "launch" and x[1] == what]
        log()
        for call in (score, evict):
            assert call(s) == 0
            assert not launched(kinds(), "clear")                       # nothing was left behind
            fake.fake_fail(b"stats_kernel")
            assert call(s) == -6
            k = kinds()
            last = max(i for i, x in enumerate(k) if x[:2] == ("launch", "score"))
            clears = [i for i, x in enumerate(k) if x[:2] == ("launch", "clear")]
            assert clears and clears[-1] > last and k[clears[-1]][2] == hex(s), k
            fake.fake_fail(b"")
            assert call(s2) == 0 and not launched(kinds(), "clear")
        # neither the statistics nor the clear behind them
        fake.fake_fail(b"stats_kernel|xchg_init")
        assert score(s) == -6; kinds()
        assert score(s) == -6
        assert not launched(kinds(), "score")
        fake.fake_fail(b"")
        fake.fake_capture(P(s))
        assert score(s) == 0
        assert kinds()[0][1] == "clear"
        fake.fake_capture(P(0))
        assert score(s) == 0
        assert kinds()[0][1] == "clear"
        assert score(s) == 0 and not launched(kinds(), "clear")
        print("ok")
        """
    cfg = good(n_layers=8, ctx_len=5000, budget=600)
    assert scenario(runtime, body, cfg).strip() == "ok"


def configs_of_size():
    from perf import cases
    names = [f[0] for f in MB.Config._fields_]
    for c in cases.listed():
        kw = {k: v for k, v in c.items() if k in names}
        yield c["name"], good(**dict(kw, dtype=MB.BF16 if c["dtype"] == "bf16" else MB.FP32, max_new_tokens=c["steps"] + 1))
    yield "few heads, little kept", good(n_layers=8, n_q_heads=8, n_kv_heads=1, ctx_len=65536, window=32, budget=256, hcc_rho=1024)
    yield "many heads", good(n_layers=64, batch=2, n_q_heads=64, n_kv_heads=32, ctx_len=8192, budget=512, hcc_rho=64)
    yield "paged", good(n_layers=4, ctx_len=9000, budget=700, page_rows=32, cache_fp8=1)


@pytest.mark.parametrize("cfg", [pytest.param(c, id=n.replace(" ", "_")) for n, c in configs_of_size()])
def test_where_partial_results_of_decode_go(runtime, cfg):
    """A launch of madakv_decode_attn leaves the pieces' partial results in the caller's workspace, within what
    madakv_workspace_bytes reports; one of madakv_decode_attn_static in the handle's scratch, or it is refused.  The handle
    holds what the header says."""
    heads = cfg.n_layers * cfg.batch * cfg.n_kv_heads
    G = cfg.n_q_heads // cfg.n_kv_heads
    per_key = 1.1 if G * cfg.window <= 64 else 4.4
    most = (8 << 20) + 4096 + heads * (128 * G + 4) + max(1 << 20, int(heads * per_key * cfg.ctx_len))
    if cfg.page_rows:
        most += heads * 4 * (2 + (cfg.ctx_len + cfg.max_new_tokens) // cfg.page_rows)
    scenario(runtime, f"""
        h = create(sys.argv[3])
        mallocs = [(num(x.rest[0]), int(x.rest[1])) for x in log() if x.kind == "malloc"]
        assert mallocs[0][1] <= {most}, (mallocs, {most})
        assert len(mallocs) == 1 or mallocs[1][1] <= 128 * {72 * 1024} * {(cfg.ctx_len + 16383) // 16384}
        heads1, G, d = {cfg.batch * cfg.n_kv_heads}, {G}, {cfg.head_dim}
        def launch(static, n):
            b = Z()
            assert lib.madakv_workspace_bytes(h, I(n), None, None, C.byref(b)) == 0
            ws = T(b.value)
            t = [P(T().p), None, None, *(P(T().p) for _ in range(5))]
            if static: rc = lib.madakv_decode_attn_static(h, I(0), I(n), *t, P(0))
            else: rc = lib.madakv_decode_attn(h, I(0), I(n), *t, P(ws.p), b, P(0))
            if rc == -4 and static: return
            assert rc == 0
            (x,) = [x for x in log() if x.kind == "launch" and "decode" in str(x)]
            grid = [int(g) for g in x.rest[1].split(",")]
            if grid[1] == 1: return                                  # nothing to leave
            size = heads1 * n * grid[1] * G * (d + 2) * 4            # as many pieces per head as the grid has
            lo, hi = (mallocs[0][0], mallocs[0][0] + mallocs[0][1]) if static else (ws.p, ws.p + ws.size)
            words = [int(w, 16) for w in x.rest[4:]]
            # the array of partial results and, behind it, that of their (max, sum) pairs
            found = [w for w in words if lo <= w < hi and w + heads1 * n * grid[1] * G * d * 4 in words]
            assert len(found) == 1 and found[0] + size <= hi, (found, lo, hi, size)
        for n in sorted({{1, {min(2, cfg.n_layers)}, {cfg.n_layers}}}):
            launch(False, n)
            launch(True, n)
        """, cfg)


@pytest.mark.parametrize("cfg", [good(n_layers=4, ctx_len=16384, budget=2048), good(n_layers=2, n_q_heads=28, n_kv_heads=4, ctx_len=8192, budget=600),
                                 good(n_layers=3, n_q_heads=12, n_kv_heads=2, window=40, ctx_len=3001, budget=600, head_dim=64)],
                         ids=lambda c: f"q{c.n_q_heads}_kv{c.n_kv_heads}_w{c.window}")
def test_window_workspace_holds_no_exchange_words(runtime, cfg):
    """The words that workgroups exchange are the handle's; a caller's workspace of the window attention is the counter and the
    row blocks' shares of O and of psi."""
    heads, rows, L, d = cfg.n_layers * cfg.batch * cfg.n_kv_heads, cfg.n_q_heads // cfg.n_kv_heads * cfg.window, cfg.ctx_len, cfg.head_dim
    up = lambda x, n: (x + n - 1) // n * n
    blocks, chunks = up(rows, 32) // 32, up(L, 512 if d == 128 else 768) // (512 if d == 128 else 768)
    window = 256 + up(heads * blocks * chunks * 32 * d * 4, 256) + (blocks * heads * L * 4 if blocks > 1 else 0)
    scenario(runtime, f"""
        h = create(sys.argv[3])
        b = Z()
        assert lib.madakv_window_attn_workspace_bytes(h, I({cfg.n_layers}), C.byref(b)) == 0
        assert b.value == {window}, (b.value, {window})
        """, cfg)


@pytest.mark.parametrize("cfg", [good(n_layers=32, batch=4, n_q_heads=32, n_kv_heads=32, ctx_len=16384, budget=2048), good(n_layers=64, ctx_len=4096, cache_fp8=1),
                                 good(n_layers=48, batch=4, n_q_heads=28, n_kv_heads=4, ctx_len=12000, budget=1000)], ids=lambda c: f"layers{c.n_layers}")
def test_per_head_kernels_fit_beside_a_gather(runtime, cfg):
    """In a call over several layer groups statistics and selection run beside a gather, whose workgroups claim LDS to leave them
    room: what the claims leave of a compute unit's 160 KB takes a selection workgroup over up to 16K candidates at once, and one
    of the statistics when a single gather workgroup has left (2 KB for what the kernels declare themselves)."""
    scenario(runtime, f"""
        h = create(sys.argv[3])
        log()
        t = [P(T().p) for _ in range(14)]
        assert lib.madakv_evict(h, I(0), I({cfg.n_layers}), *t, P(T().p), Z(1 << 34), P(T().p), Z(1 << 34), P(0)) == 0
        lds = {{}}
        for x in log():
            if x.kind == "launch":
                for name in ("gather", "select", "stats"):
                    if name + "_kernel" in str(x): lds.setdefault(name, set()).add(int(x.rest[2]))
        unit = 160 * 1024
        (claim,) = lds["gather"]
        left = unit - unit // claim * claim
        assert max(lds["select"]) + 2048 <= left and max(lds["stats"]) + 2048 <= left + claim, (lds, left)
        """, cfg)


SHORT, USUAL = "decode_attn_kernelIttLi16ELi1ELi4ELi8E", "decode_attn_kernelIttLi16ELi1ELi4ELi4E"          # eight waves, pieces of 128 rows; four
TILES16, TILES32 = "Li8ELi1EE", "Li4ELi2EE"


@pytest.mark.parametrize("heads,rows,want", [(32, 160, USUAL), (32, 161, SHORT), (64, 1024, SHORT), (64, 1025, USUAL), (28, 2048, SHORT), (29, 2048, USUAL),
                                             (15, 2049, SHORT), (16, 2049, USUAL), (8, 4096, SHORT), (8, 4097, USUAL), (128, 200, SHORT), (129, 200, USUAL),
                                             (512, 200, USUAL)])
def test_single_queries_take_short_pieces_up_to(runtime, heads, rows, want):
    """Where pieces of 128 rows are the faster ones for heads of one query: by the heads of a launch, their rows and the rows of all."""
    scenario(runtime, f"""
        h = create(sys.argv[3])
        b = Z()
        assert lib.madakv_workspace_bytes(h, I(1), None, None, C.byref(b)) == 0
        log()
        assert lib.madakv_decode_attn(h, I(0), I(1), *[P(T().p) for _ in range(8)], P(T(b.value).p), b, P(0)) == 0
        (x,) = [x for x in log() if x.kind == "launch"]
        assert {want!r} in str(x), x
        """, good(n_layers=1, batch=heads, n_q_heads=1, n_kv_heads=1, ctx_len=9000, budget=rows - 2, max_new_tokens=2, hcc_rho=2))


@pytest.mark.parametrize("d,heads,rows,want", [(64, 32, 2048, TILES16), (64, 32, 2049, TILES32), (64, 128, 400, TILES16), (64, 129, 400, TILES32), (64, 512, 128, TILES32),
                                               (128, 512, 128, TILES16), (128, 64, 8192, TILES16)])
@pytest.mark.parametrize("fp8", [0, 1])
def test_grouped_queries_take_tiles_of(runtime, d, heads, rows, want, fp8):
    """Tiles of 32 rows for heads of 64 dims in longer pieces than 128 rows or on more than 128 heads, of 16 rows otherwise."""
    scenario(runtime, f"""
        h = create(sys.argv[3])
        b = Z()
        assert lib.madakv_workspace_bytes(h, I(1), None, None, C.byref(b)) == 0
        log()
        assert lib.madakv_decode_attn(h, I(0), I(1), *[P(T().p) for _ in range(8)], P(T(b.value).p), b, P(0)) == 0
        (x,) = [x for x in log() if x.kind == "launch"]
        assert "decode_gqa_kernel" in str(x) and {want!r} in str(x), x
        """, good(n_layers=1, batch=heads, n_q_heads=4, n_kv_heads=1, head_dim=d, ctx_len=9000, budget=rows - 2, max_new_tokens=2, hcc_rho=2, cache_fp8=fp8))
