"""The worker replay's host side without a GPU: a stand-in for the HIP runtime counts launches, captures and graphs, and fails on
request.  Every scenario runs in a process of its own, where the stand-in's symbols come before the runtime's."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
extern "C" {
struct dim3_ { unsigned x, y, z; };
typedef struct Stream { int nodes = -1; } *stream_t;          // nodes: of the graph under capture, -1 outside one
int fake_launches, fake_captures, fake_graph_launches, fake_graphs_alive, fake_fail_graph_launch, fake_waits;
static int token;
static std::set<void*> caller_captures;                        // streams that the caller has under capture
void fake_caller_capture(void* s, int on) { if (on) caller_captures.insert(s); else caller_captures.erase(s); }
static dim3_ cfg_grid, cfg_block; static size_t cfg_lds; static void* cfg_stream;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t l, void* s) { cfg_grid = g; cfg_block = b; cfg_lds = l; cfg_stream = s; return 0; }
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* l, void** s) { *g = cfg_grid; *b = cfg_block; *l = cfg_lds; *s = cfg_stream; return 0; }
static std::map<void*, int> own;                               // streams made here
int hipLaunchKernel(const void*, dim3_ g, dim3_ b, void** args, size_t, void* s) {
    if (g.x == 1 && b.x == 1) { token = *(int*)args[0]; return 0; }       // the search for streams
    if (own.count(s) && ((stream_t)s)->nodes >= 0) ++((stream_t)s)->nodes; else ++fake_launches;
    return 0;
}
int hipMemcpyFromSymbolAsync(void* dst, const void*, size_t n, size_t, int, void*) { memcpy(dst, &token, n); return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = new Stream; own[*s] = 1; return 0; }
int hipStreamDestroy(void* s) { own.erase(s); delete (stream_t)s; return 0; }
int hipStreamSynchronize(void* s) { if (caller_captures.count(s)) return 900; ++fake_waits; return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamIsCapturing(void* s, int* status) { *status = caller_captures.count(s) ? 1 : 0; return 0; }
int hipEventCreate(void** e) { *e = malloc(8); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = malloc(8); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.f; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "stand-in error"; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)4096; return 0; }
int hipThreadExchangeStreamCaptureMode(int*) { return 0; }
int hipStreamBeginCapture(void* s, int) { ((stream_t)s)->nodes = 0; ++fake_captures; return 0; }
int hipStreamEndCapture(void* s, void** g) { *g = new int(((stream_t)s)->nodes); ((stream_t)s)->nodes = -1; return 0; }
int hipGraphDestroy(void* g) { delete (int*)g; return 0; }
int hipGraphInstantiate(void** e, void* g, void**, char*, size_t) { *e = new int(*(int*)g); ++fake_graphs_alive; return 0; }
int hipGraphExecDestroy(void* e) { delete (int*)e; --fake_graphs_alive; return 0; }
int hipGraphLaunch(void*, void*) {
    if (fake_fail_graph_launch > 0 && --fake_fail_graph_launch == 0) return 999;
    ++fake_graph_launches;
    return 0;
}
}
"""

SETUP = r"""
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_2107_06925_amd import binding as b
L = b.lib()
count = lambda name: C.c_int.in_dll(fake, "fake_" + name).value
space = iter(range(1 << 32, 1 << 40, 1 << 28))                # addresses that nothing follows
class Made:
    pass
def stage(mb=2, keep=True, slots=4, weights=None, stream=None, seq=64):
    st = Made()
    st.handle = L.chimera_stage_create(2, 128, 4, seq, mb, b.F32)
    b.check(L.chimera_stage_set_option(st.handle, b.OPT_KEEP, int(keep)))
    st.buffers = [weights or next(space), next(space), next(space), slots, next(space), stream]
    b.check(L.chimera_stage_bind(st.handle, *st.buffers))
    return st
def io(st, mb):
    b.check(L.chimera_stage_set_io(st.handle, mb, *[next(space) for _ in range(4)]))
def worker(D=4, N=4, **kw):
    stages = [stage(**kw) for _ in range(2)]
    for st in stages:
        st.io = {}
        for mb in range(2 * N):
            st.io[mb] = [next(space) for _ in range(4)]
            b.check(L.chimera_stage_set_io(st.handle, mb, *st.io[mb]))
    b.chimera_worker_bind_pipes(stages)
    return stages
def zero(stages):
    for st in stages:
        b.check(L.chimera_stage_zero_grads(st.handle))
def replay(stages, N=4, z=True):
    if z:
        zero(stages)
    b.chimera_run_worker_pipes(b.DIRECT, 1, 4, N, 1)
    assert b.chimera_worker_last_lanes() == 2
    return b.chimera_worker_last_replay()
def fills(st):
    # whether reading the gradients fills them with zeros first
    before, buf = count("launches"), (C.c_char * L.chimera_stage_grad_bytes(st.handle))()
    b.check(L.chimera_stage_read_grads(st.handle, buf, len(buf)))
    return count("launches") - before
"""

SCENARIOS = {
    "third replay on": r"""
s = worker()
assert [replay(s) for _ in range(4)] == [0, 1, 2, 2]
one_by_one = count("launches")
assert replay(s) == 2 and count("launches") == one_by_one and count("captures") == 2 and count("graphs_alive") == 2
assert [fills(st) for st in s] == [0, 0]
for st in s:
    L.chimera_stage_destroy(st.handle)
assert count("graphs_alive") == 0
""",
    "same io set again": r"""
s = worker()
def set_again():
    for st in s:
        for mb, p in st.io.items():
            b.check(L.chimera_stage_set_io(st.handle, mb, *p))
how = []
for _ in range(4):
    set_again()
    how.append(replay(s))
assert how == [0, 1, 2, 2], how
io(s[0], 0)
assert replay(s) == 0
""",
    "gradients accumulated": r"""
s = worker()
assert [replay(s, z=z) for z in [1, 0, 0] * 4] == [0, 0, 1] + [1, 2, 2] + [2, 2, 2] * 2
assert count("captures") == 4 and count("graphs_alive") == 4
s = worker()
assert [replay(s, z=z) for z in [1, 0] * 4] == [0, 0] + [1, 1] + [2, 2] * 2
""",
    "schedules in turn": r"""
s = worker(N=16)
assert [replay(s, N=n) for n in [4, 8, 12] * 3] == [0] * 3 + [1] * 3 + [2] * 3
assert count("graphs_alive") == 6
# more than are kept: never recorded, the graphs of what is not used any more given back
assert [replay(s, N=n, z=z) for n, z in [(4, 0), (8, 0), (12, 0), (16, 0), (16, 1)] * 3] == [0] * 15
assert count("graphs_alive") == 0
assert [replay(s, N=16) for _ in range(3)] == [1, 2, 2]
""",
    "failed launches": r"""
fail = C.c_int.in_dll(fake, "fake_fail_graph_launch")
def refused(s, nth, z=True):
    fail.value = nth
    try:
        replay(s, z=z)
    except b.ChimeraError as e:
        assert e.code == b.EDEVICE
        return True
s = worker()
for before in (1, 2, 3):                                       # while recording, and from graphs
    # the first lane's graph is refused: neither stage's zeroing has been done; the second's: that stage's has not
    for nth, left in ((1, (True, True)), (2, (False, True))):
        assert [replay(s) for _ in range(before)] == [0, 1, 2][:before]
        assert refused(s, nth)
        assert tuple(fills(st) > 0 for st in s) == left, (before, nth)
        assert count("graphs_alive") == 0                      # recorded again, from the start
# nothing to zero: nothing is left to zero
assert [replay(s, z=False) for _ in range(2)] == [0, 1] and refused(s, 1, z=False)
assert [fills(st) for st in s] == [0, 0]
""",
    "caller's capture": r"""
home = 0x5000
s = worker(stream=home)
assert [replay(s) for _ in range(2)] == [0, 1]
def refused(z):
    before = [count(n) for n in ("launches", "captures", "graph_launches", "waits")]
    fake.fake_caller_capture(C.c_void_p(home), 1)
    try:
        replay(s, z=z)
        return False
    except b.ChimeraError as e:
        assert e.code == b.EDEVICE
    finally:
        fake.fake_caller_capture(C.c_void_p(home), 0)
    return [count(n) for n in ("launches", "captures", "graph_launches", "waits")] == before
assert refused(True) and [replay(s) for _ in range(2)] == [2, 2]
assert refused(False) and [replay(s, z=False) for _ in range(3)] == [0, 1, 2]
zero(s)
assert refused(False) and [fills(st) > 0 for st in s] == [True, True]
""",
    "outlived plans": r"""
s = worker(N=8)
assert [replay(s, N=n) for n in [4, 4, 8, 8]] == [0, 1, 0, 1] and count("graphs_alive") == 4
io(s[1], 0)                                                    # every recording of this stage is void
assert replay(s) == 0 and count("graphs_alive") == 0
assert [replay(s) for _ in range(2)] == [1, 2] and count("graphs_alive") == 2
b.check(L.chimera_op_gemm_tuning(0, 0, 0, 0))
assert [replay(s) for _ in range(3)] == [0, 1, 2] and count("graphs_alive") == 2
b.check(L.chimera_stage_bind(s[0].handle, *s[0].buffers))
assert count("graphs_alive") == 0 and [replay(s) for _ in range(3)] == [0, 1, 2]
""",
}


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("runtime")
    src, lib = d / "runtime.cpp", d / "libruntime.so"
    src.write_text(RUNTIME)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-O1", str(src), "-o", str(lib)], check=True)
    return str(lib)


@pytest.mark.parametrize("name", SCENARIOS)
def test_replay(runtime, name):
    r = subprocess.run([sys.executable, "-c", SETUP + SCENARIOS[name], runtime, ROOT], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-3000:]
