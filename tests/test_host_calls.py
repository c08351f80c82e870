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
