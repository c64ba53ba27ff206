"""The host side of the library (slh_api.cpp) against a stand-in for the HIP runtime
and the kernels (host_stub.cpp): what is launched, on which stream, in which order,
what is allocated and when the host waits.  No GPU."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

from paper_2607_19368_amd import slh as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_19368_amd", "csrc")
X = ctypes.c_void_p(1 << 20)          # never read by the stand-in


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    assert shutil.which("g++")
    out = str(tmp_path_factory.mktemp("host") / "libhost.so")
    cmd = ["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__", "-w",
           "-isystem", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(CSRC, "slh_api.cpp"), os.path.join(ROOT, "tests", "host_stub.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


@pytest.fixture
def lib(built, tmp_path):
    """A copy of its own for each test: the library's state per device starts afresh."""
    L = ctypes.CDLL(shutil.copy(built, tmp_path))
    L.stub_log.restype = ctypes.c_char_p
    L.slh_last_error.restype = ctypes.c_char_p
    L.slh_last_error.argtypes = [ctypes.c_void_p]
    return L


class Ctx:
    """A context of the stand-in library; calls raise with its error text."""

    def __init__(self, lib, N, D=64, m=1024, r=4, bits=8, **options):
        self.lib, self.N = lib, N
        self.h = ctypes.c_void_p()
        assert lib.slh_create(ctypes.byref(self.h), ctypes.c_int64(N), ctypes.c_int64(D), ctypes.c_int64(m),
                              r, bits, ctypes.c_uint64(0)) == 0
        self.r, self.bits, self.D = r, bits, D
        for k, v in options.items():
            self.option(k, v)

    def call(self, name, *args):
        rc = getattr(self.lib, name)(self.h, *args)
        if rc != 0:
            raise B.SLHError(f"{name} {rc}: {self.lib.slh_last_error(self.h).decode()}")

    def option(self, name, v):
        self.call("slh_set_option", getattr(B, "SLH_OPT_" + name), ctypes.c_double(v))

    def feature_map(self, dtype=B.SLH_BF16):
        self.call("slh_feature_map", X, dtype, ctypes.c_int64(self.D))

    def lanczos(self, n_it=16):
        self.call("slh_lanczos", n_it, None, None)

    def stream(self, s):
        self.call("slh_set_stream", ctypes.c_void_p(s))

    def destroy(self):
        self.lib.slh_destroy(self.h)
        self.h = None


@pytest.fixture
def stub(lib):
    """The stand-in with its switches at rest; stub.log() gives and clears the log."""
    lib.stub_groups(-1)
    lib.stub_resident(0)
    lib.stub_fail_resident(0)
    lib.stub_fail_events(0)
    lib.stub_capture(None, 0)
    made = []

    class S:
        def ctx(self, *a, **k):
            made.append(Ctx(lib, *a, **k))
            return made[-1]

        def log(self, memory=False):
            out = [tuple(int(x) if i else x for i, x in enumerate(t.split()))
                   for t in lib.stub_log().decode().splitlines()]
            lib.stub_clear()
            return [t for t in out if memory or t[0] not in ("malloc", "free")]

        def names(self):
            return [t[0] for t in self.log()]

    s = S()
    s.lib = lib
    s.log()
    yield s
    lib.stub_capture(None, 0)
    for c in made:
        if c.h:
            c.destroy()


def test_streaming_run_is_one_graph(stub):
    """Off the resident path a run on every row is captured once per configuration and
    replayed as one graph; grouped rows, whose number is the prompt's own, are launched
    directly."""
    c = stub.ctx(20000)
    c.feature_map(B.SLH_F32)
    c.lanczos()
    stub.log()
    for _ in range(2):
        c.feature_map(B.SLH_F32)
        c.lanczos()
        names = stub.names()
        assert names.count("graph_launch") == 1 and "begin_capture" not in names
        assert "lanczos" not in names and "eigh_ritz" not in names
    stub.lib.stub_groups(5000)
    c.feature_map()
    c.lanczos()
    names = stub.names()
    assert "graph_launch" not in names and names.count("lanczos") == 1 and names.count("eigh_ritz") == 1


@pytest.mark.parametrize("resident", [0, 128])
@pytest.mark.parametrize("normalise", [0, 1])
def test_first_call_of_a_shape_sizes_every_prompt(stub, resident, normalise):
    """The workspaces follow the window length, not the prompt's distinct rows: prompts
    with more of them than all before, or with none repeated, allocate nothing, and
    neither does a call under the caller's capture, which takes every row."""
    c = stub.ctx(8192, NORMALIZE=normalise)
    c.stream(16)
    stub.lib.stub_resident(resident)

    def prompt(groups):
        stub.lib.stub_groups(groups)
        c.feature_map()
        c.lanczos()
        c.call("slh_simhash", None)
        return stub.log(memory=True)

    assert any(t[0] == "malloc" for t in prompt(500))
    for groups, rows in ((600, 601), (1500, 1501), (7000, 7001), (-1, 8192), (501, 502)):
        log = prompt(groups)
        assert not [t for t in log if t[0] in ("malloc", "free")], groups
        assert ("featmap", 16, rows) in log
    stub.lib.stub_capture(ctypes.c_void_p(16), 1)
    log = prompt(500)
    assert ("featmap", 16, 8192) in log and not [t for t in log if t[0] in ("malloc", "free", "group", "query")]


def test_norms_run_while_the_host_waits_for_the_groups(stub):
    """The row search goes out first, the row norms behind the event that the host
    waits for: the GPU is not idle until the host has sized the feature map."""
    c = stub.ctx(8192)
    stub.lib.stub_groups(500)
    c.feature_map()
    stub.log()
    c.feature_map()
    assert stub.names() == ["group", "record", "rownorm", "query", "featmap"]
    c.option("DISTINCT", 0)
    c.feature_map()
    assert stub.names() == ["rownorm", "featmap"]      # asynchronous


@pytest.mark.parametrize("run", [False, True])
def test_row_sums_keep_to_their_own_groups(stub, run):
    """Row sums of grouped rows are expanded by the groups they were formed on: after
    another prompt's search into the same set they are refused; where that search took
    the other set (the first stays behind Q) they are still there."""
    c = stub.ctx(8192, NORMALIZE=1)
    stub.lib.stub_groups(500)
    c.feature_map()
    out = (ctypes.c_double * 8192)()
    sums = (B.SLH_OUT_ROWSUM, out, ctypes.c_int64(8 * 8192))
    c.call("slh_copy_out", *sums)
    if run:
        c.lanczos()
    c.option("NORMALIZE", 0)
    stub.lib.stub_groups(400)
    c.feature_map()
    stub.log()
    if run:
        c.call("slh_copy_out", *sums)
        assert stub.names().count("group_copy") == 1
    else:
        with pytest.raises(B.SLHError, match="not computed"):
            c.call("slh_copy_out", *sums)


def test_groups_of_other_windows_are_refused(stub):
    """Loaded codes let a caller go on after the windows changed: what is still there
    of grouped rows, with fewer rows per window than the windows now have, is refused
    rather than read past its end."""
    c = stub.ctx(8192)
    stub.lib.stub_groups(500)
    c.feature_map()
    c.lanczos()
    c.option("WINDOW_LEN", 1024)
    codes = (ctypes.c_uint32 * 8192)()
    c.call("slh_load", B.SLH_OUT_CODES, codes, ctypes.c_int64(4 * 8192))
    stub.log()
    energy = (ctypes.c_double * 8)()
    for call in (("slh_simhash", None), ("slh_eigh_ritz", 16, None, None), ("slh_spectral_energy", energy),
                 ("slh_lanczos", 16, None, None)):
        with pytest.raises(B.SLHError):
            c.call(*call)
    assert not set(stub.names()) & {"simhash", "eigh_ritz", "energy", "lanczos", "graph_launch"}


def _all_in_turn(log):
    """Every resident launch of the log is ordered behind all earlier ones: by its
    stream, or by an event recorded behind them that its stream waits for."""
    before, snap, made, host = {}, {}, 0, set()
    for name, stream, arg in log:
        done = before.setdefault(stream, set())
        done |= host
        if name == "record":
            snap[arg] = set(done)
        elif name == "wait":
            done |= snap[arg]
        elif name == "event_sync":         # the host waited: everything after it is behind
            host |= snap[arg]
        elif name == "stream_sync":
            host |= done
        elif name == "device_sync":
            host |= set(range(made))
        elif name == "resident":
            assert done == set(range(made)), (made, stream)
            done.add(made)
            made += 1
    return made


@pytest.mark.parametrize("seed", range(6))
def test_resident_launches_take_turns(stub, seed):
    """Contexts that are made, destroyed and moved between streams, some of whose
    launches fail: no resident kernel can meet another."""
    rng = random.Random(seed)
    stub.lib.stub_resident(64)
    live = []
    for _ in range(150):
        if not live or rng.random() < 0.15:
            live.append(stub.ctx(64, m=256))
            live[-1].stream(rng.randint(11, 14))
            live[-1].feature_map(B.SLH_F32)
        c = rng.choice(live)
        what = rng.random()
        if what < 0.1:
            live.remove(c)
            c.destroy()
        elif what < 0.3:
            c.stream(rng.randint(11, 14))
        elif what < 0.4:
            stub.lib.stub_fail_resident(1)
            with pytest.raises(B.SLHError):
                c.lanczos()
        else:
            stub.lib.stub_fail_events(1 if what > 0.95 else 0)
            c.lanczos()
    stub.lib.stub_fail_events(0)
    assert _all_in_turn(stub.log()) > 50


def test_one_stream_needs_no_event(stub):
    """While every resident launch comes from one stream nothing is recorded; the first
    launch on a second one goes behind all that the first holds, then each has its
    event."""
    stub.lib.stub_resident(64)
    a, b = stub.ctx(64, m=256), stub.ctx(64, m=256)
    for c in (a, b):
        c.stream(11)
        c.feature_map(B.SLH_F32)
    stub.log()
    for c in (a, b, a):
        c.lanczos()
    assert stub.names() == ["resident", "eigh_ritz"] * 3
    b.stream(12)
    for c in (b, b, a):
        c.lanczos()
    log = stub.log()
    ev = log[0][2]
    assert log[:4] == [("record", 11, ev), ("wait", 12, ev), ("resident", 12, 0), ("record", 12, ev)]
    assert [t[:2] for t in log[5:7]] == [("resident", 12), ("record", 12)]
    assert log[8:] == [("wait", 11, ev), ("resident", 11, 0), ("record", 11, ev), ("eigh_ritz", 11, 0)]


@pytest.mark.parametrize("why", ["destroyed", "captured"])
def test_a_first_stream_that_cannot_be_asked(stub, why):
    """Where no event can go behind the first stream's launches, the host waits once."""
    stub.lib.stub_resident(64)
    a, b = stub.ctx(64, m=256), stub.ctx(64, m=256)
    for c, s in ((a, 11), (b, 12)):
        c.stream(s)
        c.feature_map(B.SLH_F32)
    stub.lib.stub_resident(0)
    b.lanczos()                        # its workspaces (none can be made during a capture)
    stub.lib.stub_resident(64)
    a.lanczos()
    stub.log()
    if why == "destroyed":
        stub.lib.stub_fail_events(1)
    else:
        stub.lib.stub_capture(ctypes.c_void_p(11), 1)
    b.lanczos()
    stub.lib.stub_capture(None, 0)
    assert [t[0] for t in stub.log()] == ["device_sync", "resident", "record", "eigh_ritz"]
    a.lanczos()
    assert stub.names() == ["wait", "resident", "record", "eigh_ritz"]


def test_streams_of_each_thread_always_wait(stub):
    """hipStreamPerThread is one value for a stream of each thread."""
    stub.lib.stub_resident(64)
    c = stub.ctx(64, m=256)
    c.stream(2)
    c.feature_map(B.SLH_F32)
    c.lanczos()
    stub.log()
    c.lanczos()
    assert stub.names() == ["device_sync", "resident", "record", "eigh_ritz"]
    c.lanczos()
    assert stub.names() == ["wait", "resident", "record", "eigh_ritz"]


def test_captured_resident_launch_joins_the_capture_alone(stub):
    """Under the caller's capture a resident launch neither waits for nor records an
    event of another stream (either would tie the capture to work outside it)."""
    stub.lib.stub_resident(64)
    a, b = stub.ctx(64, m=256), stub.ctx(64, m=256)
    for c, s in ((a, 11), (b, 12)):
        c.stream(s)
        c.feature_map(B.SLH_F32)
        c.lanczos()
    stub.log()
    stub.lib.stub_capture(ctypes.c_void_p(11), 1)
    a.lanczos()
    assert stub.names() == ["resident", "eigh_ritz"]
    stub.lib.stub_capture(None, 0)
    b.lanczos()
    a.lanczos()
    assert stub.names().count("wait") == 1
