"""GPU parity at the edges of dispatch rules: sizes where a kernel variant begins or ends, and the
replay with its stages beside each other against the replay in turn."""
import numpy as np
import pytest

from oracle import edges_oracle as eo
from paper_2107_06925_amd import binding as b
from paper_2107_06925_amd import synth
from gpu_util import assert_close, make_stage, to_dev, to_np

pytestmark = pytest.mark.gpu


def _worker(overlap, shared_dx, D=4, N=8, L=2, H=128, heads=2, S=72, B=1):
    import torch
    rank = 1
    need = b.stash_slots_needed(b.DIRECT, D, N, rank)
    stages = []
    for pipe, sid in ((0, rank), (1, D - 1 - rank)):
        p = synth.make_stage_params(H, L, sid, 0, "bf16", qk_gain=synth.qk_gain_for(H))
        st = b.Stage(L, H, heads, S, B, b.BF16, stash_slots=need[pipe], overlap=overlap)
        st.set_weights(synth.flatten_params(p))
        stages.append(st)
    outs, io = [], {}
    for o in b.chimera_schedule(b.DIRECT, D, N, rank):
        if o.kind == b.OP_F:
            x, dy = synth.make_microbatch(S * B, H, o.mb, 0, "bf16")
            io[o.mb] = (to_dev(x, b.BF16), to_dev(dy, b.BF16))
            y, dx = stages[o.pipe].set_io(o.mb, *io[o.mb])
            if shared_dx is not None:          # one buffer for every gradient: only the last one in list order survives
                b.check(b.lib().chimera_stage_set_io(stages[o.pipe].handle, o.mb, *[b._ptr(t) for t in (io[o.mb][0], y, io[o.mb][1], shared_dx)]))
                dx = shared_dx
            outs += [y, dx]
    b.chimera_worker_bind(*stages)
    for st in stages:
        st.zero_grads()
    b.chimera_run_worker(rank, D, N)
    assert b.chimera_worker_last_lanes() == (2 if overlap and shared_dx is None else 1)
    torch.cuda.synchronize()
    return [t.clone() for t in outs] + [st.grads.clone() for st in stages]


@pytest.mark.parametrize("shared", [False, True])
def test_replay_beside_equals_replay_in_turn(shared):
    import torch
    print("replay lanes, shared dx", shared, flush=True)
    dx = torch.zeros((72, 128), device="cuda", dtype=torch.bfloat16) if shared else None
    for a, c in zip(_worker(True, dx), _worker(False, dx)):
        assert torch.equal(a, c)


# In a process of its own, so that the replay is the first to look for streams: binding stays legal under stream capture; the
# search may meet a busy GPU or another thread's capture; with a single hardware queue the stages take turns.
_FIRST_REPLAY = """
import threading
import torch
from paper_2107_06925_amd import binding as b
what = %r
stages, io = [], []
for pipe in (0, 1):
    st = b.Stage(1, 128, 2, 64, 1, b.BF16, stash_slots=2)
    st.weights.normal_(0, 0.02)
    stages.append(st)
for o in b.chimera_schedule(b.DIRECT, 2, 2, 0):
    if o.kind == b.OP_F:
        x = torch.randn(64, 128, device="cuda").bfloat16()
        io += [x, stages[o.pipe].set_io(o.mb, x, x)]
x, graph = torch.zeros(1024, device="cuda"), torch.cuda.CUDAGraph()
begun, end = threading.Event(), threading.Event()
torch.cuda.synchronize()

def capture():
    with torch.cuda.stream(torch.cuda.Stream()), torch.cuda.graph(graph):
        x.add_(1)
        if what == "bind":
            b.chimera_worker_bind(*stages)
        begun.set()
        end.wait(30)
        x.add_(1)

if what == "bind":
    end.set()
    capture()
else:
    b.chimera_worker_bind(*stages)
    if what == "thread":
        other = threading.Thread(target=capture)
        other.start()
        begun.wait(30)
    elif what == "busy":
        a = torch.randn(4096, 4096, device="cuda").bfloat16()
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(100):
                a @ a
b.chimera_run_worker(0, 2, 2)
lanes = [b.chimera_worker_last_lanes()]
if what == "thread":
    end.set()
    other.join()
if what in ("bind", "thread"):
    graph.replay()
    torch.cuda.synchronize()
    assert float(x[0]) == 2.0
for _ in range(3):
    b.chimera_run_worker(0, 2, 2)
    lanes.append(b.chimera_worker_last_lanes())
b.chimera_worker_set_timing(True)
b.chimera_run_worker(0, 2, 2)
lanes.append(b.chimera_worker_last_lanes())
print("lanes", *lanes)
"""


@pytest.mark.parametrize("what", ["idle", "bind", "busy", "thread", "one queue"])
def test_first_replay_finds_its_streams(what):
    import os
    import subprocess
    import sys
    print("first replay", what, flush=True)
    env = dict(os.environ, **({"GPU_MAX_HW_QUEUES": "1"} if what == "one queue" else {}))
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", _FIRST_REPLAY % what], cwd=root, env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split() == ["lanes"] + ["1" if what == "one queue" else "2"] * 4 + ["1"]


# Products of 256x128 tiles, which only a replay of two stages beside each other takes: up to 256 of 128x128 in
# turn (the same order of summation), beyond them with ragged rows, columns and k, and in place of 64x64.  Two
# orders of summing a few thousand products in float differ by less than a bf16 rounding; each of a block's
# results is rounded a few times: well within the bf16 bar.
@pytest.mark.parametrize("H,heads,S,B,same", [(1024, 16, 1000, 4, True), (1032, 43, 1300, 3, False), (2048, 16, 512, 2, False)])
def test_replay_beside_wide_tiles(H, heads, S, B, same):
    import torch
    print("replay lanes, wide tiles", H, S, B, flush=True)
    shape = dict(D=2, N=2, L=1, H=H, heads=heads, S=S, B=B)
    for i, (a, c) in enumerate(zip(_worker(True, None, **shape), _worker(False, None, **shape))):
        if same:
            assert torch.equal(a, c)
        else:
            assert_close(to_np(a), to_np(c), b.BF16, "output %d" % i)


# tokens: all the same, few distinct, more than one window of the list; widths of one to eight pieces per lane
@pytest.mark.parametrize("tokens,seq,hidden,vocab,dtype", [
    (300, 100, 72, 1, b.F32), (4097, 17 * 241, 520, 3, b.BF16), (9000, 9, 1032, 1500, b.BF16), (64, 8, 4096, 40, b.BF16),
    (4095, 1365, 2048, 70000, b.F32), (130, 13, 640, 1024, b.F32)])
def test_embedding_backward(tokens, seq, hidden, vocab, dtype):
    import torch
    tokens -= tokens % seq
    print("embedding backward", tokens, seq, hidden, vocab, dtype, flush=True)
    rng = np.random.default_rng(0)
    ids = (vocab ** rng.random(tokens)).astype(np.int32) - 1
    dx = rng.standard_normal((tokens, hidden)).astype(np.float32)
    dx = synth.round_to_bf16(dx) if dtype == b.BF16 else dx
    flat = torch.zeros((vocab + seq) * hidden + 1, device="cuda")          # tables at an odd offset: not 16-byte aligned
    dwte, dwpe = flat[1:1 + vocab * hidden].view(vocab, hidden), flat[1 + vocab * hidden:].view(seq, hidden)
    b.chimera_op_embedding_bwd(torch.from_numpy(ids).cuda(), seq, to_dev(dx, dtype), dwte, dwpe)
    want_te, want_pe = eo.embedding_bwd(dx, ids, seq, vocab)
    assert_close(to_np(dwte), want_te, b.F32, "dwte")
    assert_close(to_np(dwpe), want_pe, b.F32, "dwpe")


# Several windows of the list with at most a few entries of a token in each: no workgroup meets a frequent token, so
# between its windows only the windows' own barriers order the wavefronts.  Small whole numbers: float sums are exact.
@pytest.mark.parametrize("tokens,hidden,vocab,dtype", [(8193, 64, 1024, b.BF16), (30000, 512, 5000, b.BF16), (40960, 264, 40000, b.F32)])
def test_embedding_backward_windows(tokens, hidden, vocab, dtype):
    import torch
    print("embedding backward windows", tokens, hidden, vocab, dtype, flush=True)
    rng = np.random.default_rng(3)
    ids = rng.permutation(np.arange(tokens) % vocab).astype(np.int32)
    dx = rng.integers(-8, 9, size=(tokens, hidden)).astype(np.float32)
    want = np.zeros((vocab, hidden), dtype=np.float32)
    np.add.at(want, ids, dx)
    dwte, dwpe = torch.zeros((vocab, hidden), device="cuda"), torch.zeros((1, hidden), device="cuda")
    for n in range(1, 4):
        b.chimera_op_embedding_bwd(torch.from_numpy(ids).cuda(), 1, to_dev(dx, dtype), dwte, dwpe)
        assert np.array_equal(to_np(dwte), n * want)
        assert np.array_equal(to_np(dwpe)[0], n * dx.sum(0))


def _rand(shape, seed, dtype, scale=1.0):
    a = np.random.default_rng(seed).standard_normal(shape).astype(np.float32) * scale
    return synth.round_to_bf16(a) if dtype == b.BF16 else a


# float products: 128 and 136 tiles of 64x64 (where the 32x32 form ends), one tile, ragged tiles, k with a remainder
# in both forms and for four and eight wavefronts
@pytest.mark.parametrize("m,n,k", [(512, 1024, 40), (520, 1024, 168), (8, 8, 8), (40, 104, 264), (200, 72, 1000), (1032, 520, 72)])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
def test_float_gemm(m, n, k, layout):
    import torch
    print("float gemm", m, n, k, layout, flush=True)
    a_kc, b_kc = {"fwd": (1, 0), "dgrad": (1, 1), "wgrad": (0, 0)}[layout]
    A, B = _rand((m, k), 1, b.F32), _rand((k, n), 2, b.F32)
    want = A.astype(np.float64) @ B.astype(np.float64)
    c = torch.full((m, n), 0.5, device="cuda")
    b.chimera_op_gemm(to_dev(A if a_kc else A.T, b.F32), to_dev(B.T if b_kc else B, b.F32), c, m, n, k, a_kc, b_kc,
                      b.EPI_NONE if a_kc else b.EPI_ACCUM_F32)
    assert_close(to_np(c) - (0.0 if a_kc else 0.5), want, b.F32)


# float attention: head dimensions inside and at the end of each compiled size, rows around the 32-row tiles
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("batch,seq,heads,d", [(1, 33, 2, 4), (2, 31, 3, 36), (1, 129, 2, 64), (2, 160, 1, 100), (1, 97, 2, 128)])
def test_float_attention(batch, seq, heads, d, causal):
    _attention(b.F32, batch, seq, heads, d, causal)


# The float kernels lose no more than the plain ones do: root mean square error against float64, over thousands of
# rounding errors of the same size on either side (their own spread is below 2 %), 10 % allowed.
@pytest.mark.parametrize("batch,seq,heads,d,causal,score", [(2, 512, 4, 64, False, 1.7), (2, 200, 5, 36, False, 1.5), (1, 640, 4, 32, True, 2.0),
                                                            (1, 300, 4, 128, True, 1.0)])
def test_float_attention_precision(batch, seq, heads, d, causal, score):
    import ctypes as C
    import torch
    from oracle import block_oracle as bo
    print("float attention precision", batch, seq, heads, d, causal, flush=True)
    H, M = heads * d, batch * seq
    qkv, dctx = _rand((M, 3 * H), 1, b.F32), _rand((M, H), 2, b.F32)
    qkv[:, :2 * H] *= np.float32(score ** 0.5)
    _, probs = bo.attention_fwd(qkv.astype(np.float64), batch, seq, heads, causal)
    grad = bo.attention_bwd(dctx.astype(np.float64), qkv.astype(np.float64), probs, batch, seq, heads)
    q = qkv.astype(np.float64).reshape(batch, seq, 3, heads, d).transpose(2, 0, 3, 1, 4)
    z = q[0] @ q[1].transpose(0, 1, 3, 2) / np.sqrt(d)
    z = np.where(np.tril(np.ones((seq, seq))) > 0, z, -np.inf) if causal else z
    top = z.max(-1)
    want_lse = top + np.log(np.exp(z - top[..., None]).sum(-1))
    t, do = to_dev(qkv, b.F32), to_dev(dctx, b.F32)
    err = []
    for impl in (0, 1):
        ctx, dqkv = torch.empty((M, H), device="cuda"), torch.empty_like(t)
        lse, delta = torch.empty((batch, heads, seq), device="cuda"), torch.empty((batch, heads, seq), device="cuda")
        p = [C.c_void_p(v.data_ptr()) for v in (t, ctx, lse, do, dqkv, delta)]
        b.check(b.lib().chimera_op_attention_fwd(b.F32, impl, batch, seq, heads, d, int(causal), *p[:3], None))
        b.check(b.lib().chimera_op_attention_bwd(b.F32, impl, batch, seq, heads, d, int(causal), *p, None))
        torch.cuda.synchronize()
        rms = lambda got, want: float(np.sqrt(np.mean((to_np(got) - want) ** 2)))
        err.append([rms(lse, want_lse)] + [rms(dqkv[:, i * H:(i + 1) * H], grad[:, i * H:(i + 1) * H]) for i in range(3)])
    for name, mine, plain in zip(("lse", "dq", "dk", "dv"), *err):
        assert mine <= 1.1 * plain, (name, mine, plain)


def _attention(dtype, batch, seq, heads, d, causal):
    import torch
    from oracle import block_oracle as bo
    print("attention", dtype, batch, seq, heads, d, causal, flush=True)
    H, M = heads * d, batch * seq
    qkv, dctx = _rand((M, 3 * H), 1, dtype, 1.5), _rand((M, H), 2, dtype)
    ctx64, probs = bo.attention_fwd(qkv.astype(np.float64), batch, seq, heads, causal)
    want = bo.attention_bwd(dctx.astype(np.float64), qkv.astype(np.float64), probs, batch, seq, heads)
    q = to_dev(qkv, dtype)
    ctx, dqkv = torch.full((M, H), float("nan"), dtype=q.dtype, device="cuda"), torch.full_like(q, float("nan"))
    lse, delta = torch.empty((batch, heads, seq), device="cuda"), torch.empty((batch, heads, seq), device="cuda")
    b.chimera_op_attention_fwd(q, ctx, lse, batch, seq, heads, d, causal)
    assert_close(to_np(ctx), ctx64, dtype, "ctx")
    b.chimera_op_attention_bwd(q, ctx, lse, to_dev(dctx, dtype), dqkv, delta, batch, seq, heads, d, causal)
    for name, lo in (("dq", 0), ("dk", H), ("dv", 2 * H)):
        assert_close(to_np(dqkv)[:, lo:lo + H], want[:, lo:lo + H], dtype, name)


# bf16 head dimensions other than the compiled 64 and 128, and rows around the 128- and 64-row tiles
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("batch,seq,heads,d", [(1, 65, 3, 8), (2, 129, 2, 40), (1, 200, 2, 80), (9, 130, 32, 96), (1, 127, 2, 120)])
def test_bf16_attention_head_dims(batch, seq, heads, d, causal):
    _attention(b.BF16, batch, seq, heads, d, causal)


# bf16 backward at both sides of the lines where the dK/dV role forms the row sums of dO * O itself: sequence lengths around its
# 64-row tiles and the last served one, workgroups per role of 256 and the next, partly filled quarters of a row
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("batch,seq,heads,d", [(1, 1, 1, 64), (2, 63, 3, 24), (1, 129, 2, 64), (2, 191, 2, 56), (1, 1024, 2, 64), (1, 1025, 2, 64),
                                               (8, 129, 16, 64), (8, 129, 17, 64), (1, 256, 3, 128), (1, 257, 3, 128), (2, 65, 3, 104)])
def test_bf16_attention_row_sums(batch, seq, heads, d, causal):
    _attention(b.BF16, batch, seq, heads, d, causal)


# results and gradients at addresses that wide accesses cannot take: served at head dimensions other than 64 and 128, refused there
@pytest.mark.parametrize("d,served", [(40, True), (96, True), (64, False), (128, False)])
@pytest.mark.parametrize("shifted", ["ctx", "dctx", "dqkv"])
def test_bf16_attention_alignment(d, served, shifted):
    import torch
    from oracle import block_oracle as bo
    print("attention alignment", d, shifted, flush=True)
    batch, seq, heads = 1, 70, 2
    H = heads * d
    qkv, dctx = _rand((seq, 3 * H), 1, b.BF16, 1.5), _rand((seq, H), 2, b.BF16)
    ctx64, probs = bo.attention_fwd(qkv.astype(np.float64), batch, seq, heads, True)
    want = bo.attention_bwd(dctx.astype(np.float64), qkv.astype(np.float64), probs, batch, seq, heads)

    def place(name, shape):
        at = 2 if name == shifted else 0                     # 4 bytes past a boundary
        n = shape[0] * shape[1]
        return torch.zeros(n + at, device="cuda", dtype=torch.bfloat16)[at:].view(shape)

    q, ctx, do, dqkv = to_dev(qkv, b.BF16), place("ctx", (seq, H)), place("dctx", (seq, H)), place("dqkv", (seq, 3 * H))
    do.copy_(to_dev(dctx, b.BF16))
    lse, delta = torch.empty((batch, heads, seq), device="cuda"), torch.empty((batch, heads, seq), device="cuda")
    if not served and shifted == "ctx":
        with pytest.raises(b.ChimeraError) as e:
            b.chimera_op_attention_fwd(q, ctx, lse, batch, seq, heads, d, True)
        assert e.value.code == b.EINVAL
        return
    b.chimera_op_attention_fwd(q, ctx, lse, batch, seq, heads, d, True)
    assert_close(to_np(ctx), ctx64, b.BF16, "ctx")
    if not served:
        with pytest.raises(b.ChimeraError) as e:
            b.chimera_op_attention_bwd(q, ctx, lse, do, dqkv, delta, batch, seq, heads, d, True)
        assert e.value.code == b.EINVAL
        return
    b.chimera_op_attention_bwd(q, ctx, lse, do, dqkv, delta, batch, seq, heads, d, True)
    assert_close(to_np(dqkv), want, b.BF16, "dqkv")


# bf16 products on 64x64 tiles: the two forms meet at 256 tiles, the form ends at 512; k below one step, with a
# remainder, and around the lengths of the rings; a single row
@pytest.mark.parametrize("m,n,k", [(1, 8, 8), (1000, 1024, 72), (1024, 1032, 136), (64, 64, 448), (40, 72, 520), (200, 136, 1032),
                                   (2048, 1024, 200), (2056, 1024, 192)])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
def test_bf16_small_gemm(m, n, k, layout):
    import torch
    print("bf16 gemm", m, n, k, layout, flush=True)
    a_kc, b_kc = {"fwd": (1, 0), "dgrad": (1, 1), "wgrad": (0, 0)}[layout]
    m = m if a_kc else max(m, 8)
    A, B = _rand((m, k), 1, b.BF16), _rand((k, n), 2, b.BF16)
    want = A.astype(np.float64) @ B.astype(np.float64)
    c = torch.full((m, n), 0.5, device="cuda", dtype=torch.bfloat16 if a_kc else torch.float32)
    b.chimera_op_gemm(to_dev(A if a_kc else A.T, b.BF16), to_dev(B.T if b_kc else B, b.BF16), c, m, n, k, a_kc, b_kc,
                      b.EPI_NONE if a_kc else b.EPI_ACCUM_F32)
    assert_close(to_np(c) - (0.0 if a_kc else 0.5), want, b.BF16)


# bf16 products on 256x256 tiles: one to six steps of 64 with and without a remainder, ragged rows and columns
@pytest.mark.parametrize("m,n,k", [(3080, 2824, 8), (3080, 2824, 64), (3080, 2824, 72), (3080, 2824, 128), (3080, 3064, 200),
                                   (2817, 3072, 320), (3072, 3080, 384)])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
def test_bf16_large_tiles(m, n, k, layout):
    test_bf16_small_gemm(m if layout != "wgrad" else m // 8 * 8 + 8, n, k, layout)


# rows so far apart that 255 of them exceed 32-bit byte offsets: each operand in turn, sizes of every tile
@pytest.mark.parametrize("m,n,k", [(264, 72, 72), (264, 4616, 64)])
def test_bf16_far_rows(m, n, k):
    import torch
    print("bf16 gemm far rows", m, n, k, flush=True)
    ld = (1 << 23) + 8
    A, B = _rand((m, k), 1, b.BF16), _rand((n, k), 2, b.BF16)
    far = torch.empty((m, ld), device="cuda", dtype=torch.bfloat16)
    far[:, :k] = to_dev(A, b.BF16)
    want = A.astype(np.float64) @ B.astype(np.float64).T
    c = torch.empty((m, n), device="cuda", dtype=torch.bfloat16)
    b.chimera_op_gemm(far, to_dev(B, b.BF16), c, m, n, k, 1, 1, lda=ld)
    assert_close(to_np(c), want, b.BF16)
    c = torch.empty((n, m), device="cuda", dtype=torch.bfloat16)
    b.chimera_op_gemm(to_dev(B, b.BF16), far, c, n, m, k, 1, 1, ldb=ld)
    assert_close(to_np(c), want.T, b.BF16)


# few rows of k, so far apart that 31 (or 15) of them exceed 32-bit byte offsets, and the widest that do not: index-contiguous
# operands on 128x128 and 256x256 tiles
@pytest.mark.parametrize("m,n,k,ld", [(2048, 2048, 32, 70000000), (2048, 2048, 32, 69273648), (2048, 2056, 32, 69273648), (2048, 2048, 56, 70000000),
                                      (3080, 2824, 16, 143165584), (3080, 2824, 16, 143165552), (264, 72, 32, 70000000)])
def test_bf16_far_k_rows(m, n, k, ld):
    import torch
    print("bf16 gemm far k rows", m, n, k, ld, flush=True)
    A, B = _rand((m, k), 1, b.BF16), _rand((k, n), 2, b.BF16)
    want = A.astype(np.float64) @ B.astype(np.float64)
    far = torch.empty((k, ld), device="cuda", dtype=torch.bfloat16)
    far[:, :n] = to_dev(B, b.BF16)
    c = torch.empty((m, n), device="cuda", dtype=torch.bfloat16)
    b.chimera_op_gemm(to_dev(A, b.BF16), far, c, m, n, k, 1, 0, ldb=ld)
    assert_close(to_np(c), want, b.BF16)
    c = torch.zeros((m, n), device="cuda")
    b.chimera_op_gemm(to_dev(A.T, b.BF16), far, c, m, n, k, 0, 0, b.EPI_ACCUM_F32, ldb=ld)
    assert_close(to_np(c), want, b.BF16)
    far[:, :m] = to_dev(A.T, b.BF16)
    c = torch.zeros((m, n), device="cuda")
    b.chimera_op_gemm(far, to_dev(B, b.BF16), c, m, n, k, 0, 0, b.EPI_ACCUM_F32, lda=ld)
    assert_close(to_np(c), want, b.BF16)


# 260 tiles of 256x256 in four tile rows: the last columns go to 128x128 tiles
@pytest.mark.parametrize("m,n,k", [(1000, 16424, 72), (1024, 16640, 200), (776, 16392, 128)])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
def test_bf16_peeled_columns(m, n, k, layout):
    test_bf16_small_gemm(m, n, k, layout)


# bf16 products on 128x128 tiles: up to one per CU (a ring of four steps) and beyond (two buffers)
@pytest.mark.parametrize("k", [8, 72, 128, 192, 264, 320, 456, 520, 584])
@pytest.mark.parametrize("m,n", [(2056, 1032), (3080, 2056)])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
def test_bf16_middle_tiles(m, n, k, layout):
    test_bf16_small_gemm(m, n, k, layout)


# launches of several rounds: 256x256 tiles with a partly filled last round (561, 873 and 792 tiles), 128x128 tiles two per CU (572)
@pytest.mark.parametrize("m,n,k", [(4104, 8200, 72), (2056, 24584, 64), (5640, 9216, 72), (2816, 3328, 72)])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
def test_bf16_products_of_several_rounds(m, n, k, layout):
    import torch
    print("bf16 rounds", m, n, k, layout, flush=True)
    a_kc, b_kc = {"fwd": (1, 0), "dgrad": (1, 1), "wgrad": (0, 0)}[layout]
    gen = torch.Generator().manual_seed(m)
    A, B = torch.randn((m, k), generator=gen).to(torch.bfloat16), torch.randn((k, n), generator=gen).to(torch.bfloat16)
    want = A.double() @ B.double()
    da, db = (A if a_kc else A.T.contiguous()).cuda(), (B.T.contiguous() if b_kc else B).cuda()
    dc = torch.full((m, n), 0.0 if layout == "wgrad" else float("nan"), dtype=torch.float32 if layout == "wgrad" else torch.bfloat16, device="cuda")
    b.chimera_op_gemm(da, db, dc, m, n, k, a_kc, b_kc, b.EPI_ACCUM_F32 if layout == "wgrad" else b.EPI_NONE)
    # float sums of k exact products, and one rounding to bf16
    tol = 2.0 ** -24 * k * 8 + (0 if layout == "wgrad" else 2.0 ** -8)
    assert float((dc.cpu().double() - want).abs().max()) <= tol * float(want.abs().max())


# launches of several rounds whose B exceeds half of the memory-side cache (128 MB): tile columns in bands, several groups of tile rows in each.  9x66 tiles of
# 256x256 in bands of 28, 28 and 10 (as a weight gradient 8x64 of them in bands of 32, and halves); 6x86, the last column on smaller
# tiles and the others in bands of 42, 42 and 1; 22x26 tiles of 128x128, two per CU, in bands of 23 and 3
@pytest.mark.parametrize("m,n,k", [(2056, 16648, 4040), (1512, 21960, 3064), (2816, 3328, 20168)])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
def test_bf16_products_in_bands_of_columns(m, n, k, layout):
    import torch
    print("bf16 bands", m, n, k, layout, flush=True)
    assert n * k * 2 > 128 << 20
    a_kc, b_kc = {"fwd": (1, 0), "dgrad": (1, 1), "wgrad": (0, 0)}[layout]
    gen = torch.Generator(device="cuda").manual_seed(m)
    A, B = (torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16) for shape in ((m, k), (k, n)))
    want = A.double() @ B.double()
    da, db = A if a_kc else A.T.contiguous(), B.T.contiguous() if b_kc else B
    dc = torch.full((m, n), 0.0 if layout == "wgrad" else float("nan"), dtype=torch.float32 if layout == "wgrad" else torch.bfloat16, device="cuda")
    b.chimera_op_gemm(da, db, dc, m, n, k, a_kc, b_kc, b.EPI_ACCUM_F32 if layout == "wgrad" else b.EPI_NONE)
    # float sums of k exact products of the order of sqrt(k), a rounding for 16 or 32 of them; and one rounding to bf16
    tol = 2.0 ** -24 * k / 16 * 8 + (0 if layout == "wgrad" else 2.0 ** -8)
    assert float((dc.double() - want).abs().max()) <= tol * float(want.abs().max())


# grouped weight gradients with column sums on 256x256 tiles and on both forms of 128x128 tiles
@pytest.mark.parametrize("k", [64, 128, 192, 320, 576])
@pytest.mark.parametrize("shapes", [[(1032, 1544), (2056, 1032), (1032, 2312), (1032, 1288)], [(1032, 1544), (1032, 520)],
                                    [(1032, 1544), (2056, 1032), (1032, 1032)]])
def test_bf16_groups(k, shapes):
    import torch
    print("bf16 group", k, shapes, flush=True)
    probs, sums, want = [], [], []
    for i, (m, n) in enumerate(shapes):
        X, Y = _rand((k, m), i, b.BF16), _rand((k, n), 10 + i, b.BF16)
        probs.append((to_dev(X, b.BF16), to_dev(Y, b.BF16), torch.full((m, n), 0.5, device="cuda")))
        sums.append(torch.full((n,), 0.25, device="cuda"))
        want.append((X.astype(np.float64).T @ Y.astype(np.float64), Y.astype(np.float64).sum(0)))
    b.chimera_op_gemm_group_accumulate(probs, k, sums)
    for (_, _, c), bs, (wc, wb) in zip(probs, sums, want):
        assert_close(to_np(c) - 0.5, wc, b.BF16)
        assert_close(to_np(bs) - 0.25, wb, b.BF16)


# groups on tiles of several sizes: remainders of 64 and 8 rows and columns on half tiles, what a full round leaves over on quarters
# (44 and 20 tiles; bands of rows, and of columns where a row is wider than that; 62 tiles: a row of 53 and two columns of 5) or halves (128), a product that is one half tile high; accumulating (column sums too) and overwriting
@pytest.mark.parametrize("k", [64, 192, 320])
@pytest.mark.parametrize("shapes", [[(5120, 1280), (1280, 5120), (1280, 1280), (1280, 3840)], [(6400, 1600), (1600, 6400), (1600, 1600), (1600, 4800)],
                                    [(5376, 1344), (1344, 5376), (1344, 1344), (1344, 4032)], [(4104, 4104), (72, 2056), (2056, 72)],
                                    [(1032, 17416)], [(17416, 1032)], [(1496, 13464)]])
def test_bf16_groups_of_mixed_tiles(k, shapes):
    import torch
    print("bf16 mixed group", k, shapes, flush=True)
    gen = torch.Generator().manual_seed(k)
    probs, sums, want = [], [], []
    for m, n in shapes:
        X, Y = (torch.randn((k, c), generator=gen).to(torch.bfloat16) for c in (m, n))
        probs.append((X.cuda(), Y.cuda(), torch.full((m, n), float("nan"), device="cuda")))
        sums.append(torch.full((n,), float("nan"), device="cuda"))
        want.append((X.double().T @ Y.double(), Y.double().sum(0)))
    for passes, overwrite in ((1, True), (2, False)):
        b.chimera_op_gemm_group_accumulate(probs, k, sums, overwrite=overwrite)
        for (_, _, c), bs, (wc, wb) in zip(probs, sums, want):
            # exact products of bf16 numbers, summed in float: k roundings of sums of the order of sqrt(k), once more when added
            tol = 2.0 ** -24 * k * passes * 8
            assert float((c.cpu().double() / passes - wc).abs().max()) <= tol * float(wc.abs().max())
            assert float((bs.cpu().double() / passes - wb).abs().max()) <= tol * float(wb.abs().max())


# a single weight gradient, on the same kernel as large groups, is none: the name for reports stays the last group's
def test_last_group_kernel_is_of_a_group():
    import torch
    print("last group kernel", flush=True)
    name = lambda: b.lib().chimera_op_gemm_group_last_kernel().decode()
    X, c = torch.zeros((64, 4096), dtype=torch.bfloat16, device="cuda"), torch.zeros((4096, 4096), device="cuda")
    b.chimera_op_gemm_group_accumulate([(X[:, :128], X[:, :256], c.view(-1)[:128 * 256].view(128, 256))], 64)
    small = name()
    assert "mixed" not in small and small
    b.chimera_op_gemm(X, X, c, 4096, 4096, 64, 0, 0, b.EPI_ACCUM_F32)
    assert name() == small
    b.chimera_op_gemm_group_accumulate([(X, X, c)], 64)
    assert name() == "gemm_bf16_mixed_group_kernel"
    torch.cuda.synchronize()


# token counts that are no multiple of the contraction steps, and gradients that start from anything
@pytest.mark.parametrize("dtype,hidden,heads,seq,microbatch", [(b.F32, 64, 2, 75, 1), (b.F32, 136, 2, 37, 3), (b.F32, 256, 4, 130, 2),
                                                                 (b.BF16, 128, 2, 75, 1), (b.BF16, 136, 1, 37, 3), (b.BF16, 560, 7, 99, 1),
                                                                 (b.BF16, 1024, 16, 75, 2)])
def test_stage_ragged_tokens(dtype, hidden, heads, seq, microbatch):
    _stage(dtype, hidden, heads, seq, microbatch)


def _stage(dtype, hidden, heads, seq, microbatch, causal=True):
    from oracle import block_oracle as bo
    from gpu_util import compare_grads, dtype_name
    print("stage", dtype, hidden, heads, seq, microbatch, flush=True)
    gain = synth.qk_gain_for(hidden) if dtype == b.BF16 else 1.0
    st, params = make_stage(2, hidden, heads, seq, microbatch, dtype, 0, causal=causal, qk_gain=gain)
    x, dy = synth.make_microbatch(seq * microbatch, hidden, 0, 0, dtype_name(dtype))
    y, dx = st.set_io(0, to_dev(x, dtype), to_dev(dy, dtype))
    st.grads.fill_(float("nan"))
    st.zero_grads()
    st.fwd(0)
    st.bwd(0)
    wy, wdx, gr = bo.stage_pass(x, dy, params, microbatch, seq, heads, causal)
    compare_grads(st.read_grads(), gr, 2, hidden, dtype)
    assert_close(to_np(y), wy, dtype, "y")
    assert_close(to_np(dx), wdx, dtype, "dx")


# A worker of small launches replays from graphs from its third replay on: new contents of the same buffers, gradients overwritten or
# accumulated, io set anew and another schedule in between give what a worker gives whose launches always go out one by one.  Bit for
# bit, so the sizes are those whose products take the same tiles beside another stage as in turn: at most 128 of 32x32 (here 64).
@pytest.mark.parametrize("dtype, hidden, heads, seq, mb", [(b.F32, 128, 4, 64, 2), (b.BF16, 128, 4, 64, 2)])
def test_worker_replays_from_graphs(dtype, hidden, heads, seq, mb):
    import torch
    tdt, M, D = (torch.float32 if dtype == b.F32 else torch.bfloat16), seq * mb, 4
    gen = torch.Generator(device="cuda").manual_seed(3)
    rn = lambda *s, std=1.0: torch.empty(s, dtype=tdt, device="cuda").normal_(0.0, std, generator=gen)
    workers = []
    for overlap in (True, False):
        stages = [b.Stage(2, hidden, heads, seq, mb, dtype, stash_slots=4, overlap=overlap) for _ in range(2)]
        workers.append((stages, {}))
    for i in range(2):
        workers[0][0][i].weights.copy_(rn(workers[0][0][i].weights.numel(), std=0.05))
        workers[1][0][i].weights.copy_(workers[0][0][i].weights)
        for st in (workers[0][0][i], workers[1][0][i]):
            st.grads.zero_()

    def set_io():
        for stages, io in workers:
            for g in range(2 * D):
                x, dy = torch.zeros(M, hidden, dtype=tdt, device="cuda"), torch.zeros(M, hidden, dtype=tdt, device="cuda")
                io[g] = (x, dy) + tuple(stages[0 if g % D < D // 2 else 1].set_io(g, x, dy))

    set_io()
    one_by_one, recorded, graphs = b.REPLAY_LAUNCHES, b.REPLAY_RECORDED, b.REPLAY_GRAPHS
    #           N, gradients zeroed first, io set anew, how it goes out
    for step, (N, zero, anew, how) in enumerate([
            (4, 1, 0, one_by_one), (4, 1, 0, recorded), (4, 1, 0, graphs), (4, 1, 0, graphs), (4, 0, 0, one_by_one), (4, 0, 0, recorded),
            (4, 0, 0, graphs), (8, 1, 0, one_by_one), (8, 1, 0, recorded), (8, 1, 1, one_by_one), (8, 1, 0, recorded), (8, 1, 0, graphs),
            (4, 1, 0, one_by_one), (8, 1, 0, graphs), (4, 1, 0, recorded), (8, 0, 0, one_by_one), (4, 1, 0, graphs), (8, 0, 0, recorded),
            (4, 0, 0, one_by_one), (8, 0, 0, graphs), (8, 1, 0, graphs), (4, 0, 0, recorded), (4, 0, 0, graphs), (4, 1, 0, graphs)]):
        print("replay", dtype, step, flush=True)
        if anew:
            set_io()
        for g in range(2 * D):
            x, dy = rn(M, hidden), rn(M, hidden)
            for _, io in workers:
                io[g][0].copy_(x), io[g][1].copy_(dy), io[g][2].zero_(), io[g][3].zero_()
        torch.cuda.synchronize()
        for stages, _ in workers:
            if zero:
                for st in stages:
                    st.zero_grads()
            b.chimera_worker_bind_pipes(stages)
            b.chimera_run_worker_pipes(b.DIRECT, 1, D, N)
            beside = stages is workers[0][0]
            assert (b.chimera_worker_last_lanes(), b.chimera_worker_last_replay()) == ((2, how) if beside else (1, one_by_one)), step
        for g in range(N):
            assert torch.equal(workers[0][1][g][2], workers[1][1][g][2]) and torch.equal(workers[0][1][g][3], workers[1][1][g][3]), (step, g)
            assert workers[0][1][g][2].abs().sum() > 0
        for i in range(2):
            assert torch.equal(workers[0][0][i].grads, workers[1][0][i].grads), (step, i)
    for stages, _ in workers:
        for st in stages:
            st.close()


# Replays from graphs against replays of the same worker launch by launch, bit for bit, up to the largest launches that are recorded: doubled forwards and
# the backwards that recompute them, halved backwards, four pipelines, weight gradients one by one (their zero fill is recorded).  A change of the
# products' tuning (to what it is) makes a replay go out launch by launch again.
@pytest.mark.parametrize("algo,f,rank,dtype,hidden,heads,seq,mb,reference", [
    (b.DIRECT, 1, 1, b.BF16, 1024, 16, 256, 4, False), (b.DOUBLING, 1, 1, b.BF16, 320, 5, 200, 2, False), (b.DOUBLING, 1, 0, b.F32, 128, 4, 64, 2, False),
    (b.HALVING, 1, 2, b.BF16, 640, 10, 128, 2, False), (b.DIRECT, 2, 3, b.BF16, 256, 4, 128, 2, False), (b.DIRECT, 2, 1, b.F32, 128, 4, 40, 1, False),
    (b.DIRECT, 1, 0, b.BF16, 128, 4, 40, 1, True)])
def test_graphs_of_every_schedule(algo, f, rank, dtype, hidden, heads, seq, mb, reference):
    import torch
    print("graphs", algo, f, rank, dtype, hidden, seq, mb, reference, flush=True)
    tdt, M, D, N = (torch.float32 if dtype == b.F32 else torch.bfloat16), seq * mb, 4, 8
    gen = torch.Generator(device="cuda").manual_seed(5)
    rn = lambda *s, std=1.0: torch.empty(s, dtype=tdt, device="cuda").normal_(0.0, std, generator=gen)
    need = b.stash_slots_needed_pipes(algo, D, N, f, rank)
    kw = dict(reference_kernels=reference)
    stages = [b.Stage(2, hidden, heads, seq, mb, dtype, stash_slots=max(n, 1), **kw) for n in need]
    for st in stages:
        st.weights.copy_(rn(st.weights.numel(), std=0.05))
    x, dy, y, dx = rn(N, M, hidden), rn(N, M, hidden), torch.zeros(N, M, hidden, dtype=tdt, device="cuda"), torch.zeros(N, M, hidden, dtype=tdt, device="cuda")
    y2 = torch.zeros_like(y)
    doubled = [b.Stage(2, hidden, heads, seq, 2 * mb, dtype, keep=False, share_weights_of=st, **kw) for st in stages] if algo == b.DOUBLING else []
    io = lambda st, mb_, *t: b.check(b.lib().chimera_stage_set_io(st.handle, mb_, *[b._ptr(v) for v in t]))
    for o in b.chimera_schedule_pipes(algo, D, N, f, rank):
        if o.kind == b.OP_F2:
            io(doubled[o.pipe], o.mb, x[o.mb:o.mb + 2], y2[o.mb:o.mb + 2], x[o.mb:o.mb + 2], y2[o.mb:o.mb + 2])
        else:
            io(stages[o.pipe], o.mb, x[o.mb], y[o.mb], dy[o.mb], dx[o.mb])

    def replay(how, zero):
        for t in (y, dx, y2):
            t.zero_()
        if zero:
            for st in stages:
                st.zero_grads()
        b.chimera_worker_bind_pipes(stages)
        if doubled:
            b.chimera_worker_bind_doubling(*doubled)
        torch.cuda.synchronize()
        b.chimera_run_worker_pipes(algo, rank, D, N, f)
        assert b.chimera_worker_last_lanes() >= 2 and b.chimera_worker_last_replay() == how
        assert all(float(t.float().abs().sum()) > 0 for t in (y2 if doubled else y, dx))
        return [t.clone() for t in [y, dx, y2] + [st.grads for st in stages]]

    for zero in (True, False):
        b.check(b.lib().chimera_op_gemm_tuning(0, 0, 0, 0))
        got = {}
        for i, how in enumerate((b.REPLAY_LAUNCHES, b.REPLAY_RECORDED, b.REPLAY_GRAPHS, b.REPLAY_GRAPHS)):
            if i == 3:
                x.copy_(rn(N, M, hidden)), dy.copy_(rn(N, M, hidden))
            if not zero:
                for st in stages:
                    st.grads.fill_(0.25)
            got[i] = replay(how, zero)
        b.check(b.lib().chimera_op_gemm_tuning(0, 0, 0, 0))
        if not zero:
            for st in stages:
                st.grads.fill_(0.25)
        got[4] = replay(b.REPLAY_LAUNCHES, zero)
        for i, j in ((1, 0), (2, 0), (3, 4)):
            assert all(torch.equal(p, q) for p, q in zip(got[i], got[j])), (zero, i)
    for st in doubled + stages:
        st.close()


# A replay while its stages' stream is under capture is refused; the capture goes on, and so do the graphs of the worker.
def test_replay_under_capture():
    import torch
    home, graph, x = torch.cuda.Stream(), torch.cuda.CUDAGraph(), torch.zeros(64, device="cuda")
    stages = [b.Stage(1, 128, 2, 64, 1, b.BF16, stash_slots=2, stream=home) for _ in range(2)]
    for st in stages:
        st.weights.normal_(0, 0.02)
        for mb in range(2):
            t = torch.randn(64, 128, device="cuda").bfloat16()
            st.set_io(mb, t, t)
    torch.cuda.synchronize()
    b.chimera_worker_bind_pipes(stages)

    def replay():
        for st in stages:
            st.zero_grads()
        b.chimera_run_worker(0, 2, 2)
        return b.chimera_worker_last_replay()

    assert [replay() for _ in range(2)] == [b.REPLAY_LAUNCHES, b.REPLAY_RECORDED]
    want = [st.grads.clone() for st in stages]
    with torch.cuda.graph(graph, stream=home):
        x.add_(1)
        with pytest.raises(b.ChimeraError) as e:
            replay()
        x.add_(1)
    assert e.value.code == b.EDEVICE
    assert replay() == b.REPLAY_GRAPHS and all(torch.equal(st.grads, w) for st, w in zip(stages, want))
    for i in range(1, 4):
        graph.replay()
        torch.cuda.synchronize()
        assert float(x.min()) == float(x.max()) == 2.0 * i
    for st in stages:
        st.close()


# bf16 products on 32x32, 32x64 and 128x64 tiles: a single row or tile, the last and first sizes of each form (256 tiles), k below one step,
# with a remainder, and around the lengths of the rings
@pytest.mark.parametrize("m,n,k", [(1, 8, 8), (32, 32, 64), (33, 40, 520), (512, 512, 72), (512, 520, 584), (100, 1600, 1032),
                                   (1024, 512, 448), (1000, 520, 200), (1264, 1600, 136), (2048, 1024, 456), (2040, 1032, 328), (1100, 1800, 392)])
@pytest.mark.parametrize("layout", ["fwd", "dgrad"])
def test_bf16_small_output_tiles(m, n, k, layout):
    test_bf16_small_gemm(m, n, k, layout)


# ... with every epilogue, ragged rows and columns
@pytest.mark.parametrize("m,n,k", [(45, 72, 200), (333, 776, 136), (1100, 1448, 120), (1100, 1448, 192),
                                   (1100, 1448, 328), (1100, 1448, 640)])
def test_bf16_small_output_epilogues(m, n, k):
    import torch
    print("bf16 gemm epilogues", m, n, k, flush=True)
    A, B, bias, R = _rand((m, k), 1, b.BF16), _rand((k, n), 2, b.BF16, 0.05), _rand((n,), 3, b.BF16), _rand((m, n), 4, b.BF16)
    z = A.astype(np.float64) @ B.astype(np.float64)
    gelu = lambda u: 0.5 * u * (1 + np.tanh(np.sqrt(2 / np.pi) * (u + 0.044715 * u ** 3)))
    dgelu = lambda u: (gelu(u + 1e-5) - gelu(u - 1e-5)) / 2e-5
    dA, dB, dBT, dbias, dR = (to_dev(t, b.BF16) for t in (A, B, B.T, bias, R))
    c, c2 = torch.empty((m, n), device="cuda", dtype=torch.bfloat16), torch.empty((m, n), device="cuda", dtype=torch.bfloat16)
    for epi, b_kc, want in ((b.EPI_BIAS, 0, z + bias), (b.EPI_BIAS_GELU, 0, z + bias), (b.EPI_BIAS_RESIDUAL, 0, z + bias + R),
                            (b.EPI_DGELU, 1, z * dgelu(R.astype(np.float64)))):
        b.chimera_op_gemm(dA, dBT if b_kc else dB, c, m, n, k, 1, b_kc, epi, dbias, dR, c2)
        assert_close(to_np(c), want, b.BF16, "epilogue %d" % epi)
        if epi == b.EPI_BIAS_GELU:
            assert_close(to_np(c2), gelu(z + bias), b.BF16, "gelu")


# float products on 16x16 tiles: one row, edges of tiles, the last size of the form (512 tiles) and the first beyond it, k below a slice, with a
# remainder, and around the turns of 4 and 8 wavefronts; every epilogue, results and residual at an odd offset
@pytest.mark.parametrize("m,n,k", [(1, 8, 8), (16, 16, 32), (17, 24, 40), (250, 128, 128), (33, 40, 136), (256, 256, 264),
                                   (512, 256, 520), (513, 256, 104), (72, 1816, 296)])
def test_float_smallest_outputs(m, n, k):
    import torch
    print("float gemm smallest", m, n, k, flush=True)
    A, B, bias, R = _rand((m, k), 1, b.F32), _rand((k, n), 2, b.F32, 0.05), _rand((n,), 3, b.F32), _rand((m, n), 4, b.F32)
    z = A.astype(np.float64) @ B.astype(np.float64)
    gelu = lambda u: 0.5 * u * (1 + np.tanh(np.sqrt(2 / np.pi) * (u + 0.044715 * u ** 3)))
    dgelu = lambda u: (gelu(u + 1e-5) - gelu(u - 1e-5)) / 2e-5
    odd = lambda a: torch.from_numpy(np.concatenate([[0.0], a.ravel()]).astype(np.float32)).cuda()[1:].view(a.shape)
    dA, dB, dBT, dbias, dR = to_dev(A, b.F32), to_dev(B, b.F32), to_dev(np.ascontiguousarray(B.T), b.F32), odd(bias), odd(R)
    for epi, b_kc, want in ((b.EPI_NONE, 1, z), (b.EPI_NONE, 0, z), (b.EPI_BIAS, 0, z + bias), (b.EPI_BIAS_GELU, 0, z + bias),
                            (b.EPI_BIAS_RESIDUAL, 0, z + bias + R), (b.EPI_DGELU, 1, z * dgelu(R.astype(np.float64)))):
        c, c2 = odd(np.zeros((m, n))), odd(np.zeros((m, n)))
        b.chimera_op_gemm(dA, dBT if b_kc else dB, c, m, n, k, 1, b_kc, epi, dbias, dR, c2)
        # sums of k float products of size 0.05: well below 1e-5 of the largest
        assert np.max(np.abs(to_np(c) - want)) <= 1e-5 * np.max(np.abs(want)), "epilogue %d" % epi
        if epi == b.EPI_BIAS_GELU:
            assert_close(to_np(c2), gelu(z + bias), b.F32, "gelu")


# float products on split operands, 64x64 tiles (the first three) and 128x128 tiles: ragged edges, fewer steps than are loaded ahead, k with a
# remainder; every epilogue, results and residual at an odd offset; weight gradients
@pytest.mark.parametrize("m,n,k", [(1032, 584, 8), (1001, 776, 72), (584, 1480, 200), (2600, 2600, 24), (2601, 2600, 232), (2040, 2040, 776)])
def test_float_split_products(m, n, k):
    import torch
    print("float split", m, n, k, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(m)
    odd = lambda *shape: torch.randn(1 + int(np.prod(shape)), generator=gen, device="cuda")[1:].view(shape)
    A, B, bias, R = torch.randn((m, k), generator=gen, device="cuda"), torch.randn((k, n), generator=gen, device="cuda") * 0.05, odd(n), odd(m, n)
    z, size = A.double() @ B.double(), A.double().abs() @ B.double().abs()
    # of the sum of a product's absolute terms: 2^-24 for parts left out, a rounding for every 16 products and for the few sums at the end (and of the epilogue)
    tol = size * (1 + k / 16 + 8) * 2.0 ** -24 + 2.0 ** -21
    gelu = lambda u: 0.5 * u * (1 + torch.tanh(np.sqrt(2 / np.pi) * (u + 0.044715 * u ** 3)))
    u = R.double().requires_grad_()
    slope, = torch.autograd.grad(gelu(u).sum(), u)
    for epi, b_kc, want in ((b.EPI_NONE, 1, z), (b.EPI_BIAS, 0, z + bias), (b.EPI_BIAS_GELU, 0, z + bias), (b.EPI_BIAS_RESIDUAL, 0, z + bias + R),
                            (b.EPI_DGELU, 1, z * slope)):
        c, c2 = odd(m, n), odd(m, n)
        b.chimera_op_gemm(A, B.T.contiguous() if b_kc else B, c, m, n, k, 1, b_kc, epi, bias, R, c2)
        # of the values added and of GeLU's derivative (up to 1.13, hardware exp2 and reciprocal) some roundings
        assert bool(((c.double() - want).abs() <= 1.2 * tol + want.abs() * 2.0 ** -20).all()), "epilogue %d" % epi
        if epi == b.EPI_BIAS_GELU:
            assert_close(to_np(c2), to_np(gelu(want)), b.F32, "gelu")
    m = m // 8 * 8
    c = torch.full((m, n), 0.5, device="cuda")
    b.chimera_op_gemm(A[:m].T.contiguous(), B, c, m, n, k, 0, 0, b.EPI_ACCUM_F32)
    assert bool(((c.double() - 0.5 - z[:m]).abs() <= tol[:m]).all())


# what the products leave out does not add up: operands whose parts beyond the first all have one sign and nearly their largest size, sums of
# the first parts that take no rounding; 64x64 and 128x128 tiles
@pytest.mark.parametrize("m,n,k", [(1024, 1024, 8), (1024, 1024, 64), (1032, 1032, 256), (2600, 2600, 256)])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
def test_float_split_of_one_sign(m, n, k, layout):
    import torch
    print("float split one sign", m, n, k, layout, flush=True)
    a_kc, b_kc = {"fwd": (1, 0), "dgrad": (1, 1), "wgrad": (0, 0)}[layout]
    for value in (1.0077362, 1.0038910):                         # 1 + 2^-7 or 1 + 2^-8, and most of a bit of the first part less or more
        A, B = (torch.full((m, k) if a_kc else (k, m), value, device="cuda"), torch.full((n, k) if b_kc else (k, n), -value, device="cuda"))
        c = torch.zeros((m, n), device="cuda")
        b.chimera_op_gemm(A, B, c, m, n, k, a_kc, b_kc, b.EPI_NONE if a_kc else b.EPI_ACCUM_F32)
        want = -k * float(A[0, 0]) ** 2
        # left out: two products of a second part (2^-8 of the value) and a third (2^-17), 2^-24; then the sum of large and small products and that of two halves
        # of k, a rounding each, and the small products' own (at most 80, of 2^-8 of the sum)
        assert float((c.double() / want - 1).abs().max()) <= (1 + 2 + 80 * 2.0 ** -8) * 2.0 ** -24


# what a split has to keep: every bit of a float (times one, in all ranges of exponents), infinities, NaN, sums near the largest float; 64x64 and 128x128 tiles
@pytest.mark.parametrize("n", [1024, 2048])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
def test_float_split_ranges(n, layout):
    import torch
    print("float split ranges", n, layout, flush=True)
    a_kc, b_kc = {"fwd": (1, 0), "dgrad": (1, 1), "wgrad": (0, 0)}[layout]

    def product(A, B):
        c = torch.zeros((n, n), device="cuda")
        b.chimera_op_gemm(A if a_kc else A.T.contiguous(), B.T.contiguous() if b_kc else B, c, n, n, n, a_kc, b_kc,
                          b.EPI_NONE if a_kc else b.EPI_ACCUM_F32)
        return c

    gen = torch.Generator(device="cuda").manual_seed(n)
    X, Y, one = torch.randn((n, n), generator=gen, device="cuda"), torch.randn((n, n), generator=gen, device="cuda"), torch.eye(n, device="cuda")
    for scale in (1.0, torch.exp2(torch.randint(-70, 120, (n, n), generator=gen, device="cuda").float()), 2.0 ** -97, 2.0 ** -120, 5e37):       # the largest of n^2 normal numbers: below 6.8
        assert torch.equal(product(X * scale, one), X * scale) and torch.equal(product(one, X * scale), X * scale)
    tiny = product(X * 2.0 ** -118, Y * 2.0 ** 100).double() * 2.0 ** 18
    assert float((tiny - X.double() @ Y.double()).norm() / (X.double() @ Y.double()).norm()) <= n * 2.0 ** -24
    X[5, 7], X[900, 3], X[70, 1], X[70, 2] = float("inf"), float("nan"), 3.4e38, 3.4e38
    Y[1, 40] = Y[2, 40] = 1.0
    got, want = product(X, Y), X.double() @ Y.double()
    assert torch.equal(got[5].double(), want[5]) and bool(got[900].isnan().all()) and float(got[70, 40]) == float("inf")
    rest = [i for i in range(n) if i not in (5, 70, 900)]
    assert float((got[rest].double() - want[rest]).abs().max()) <= n * 2.0 ** -24 * float(want[rest].abs().max())


# numbers too small for three parts beside ordinary ones: each is seen, whatever a thread or a row has besides; 64x64 and 128x128 tiles
@pytest.mark.parametrize("n", [1024, 2048])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
@pytest.mark.parametrize("small", ["a", "b"])
def test_float_split_of_mixed_magnitudes(n, layout, small):
    import torch
    print("float split mixed magnitudes", n, layout, small, flush=True)
    a_kc, b_kc = {"fwd": (1, 0), "dgrad": (1, 1), "wgrad": (0, 0)}[layout]
    gen = torch.Generator(device="cuda").manual_seed(n)
    X, Y = torch.randn((n, n), generator=gen, device="cuda"), torch.randn((n, n), generator=gen, device="cuda")
    for least, ones, left in ((-118, slice(0, None, 4), n - n // 4), (-125, slice(0, n - 1), 1)):         # ones in every chunk of k; in all places but one
        A, B = X * 2.0 ** least, Y * 2.0 ** 100
        A[:, ones], B[ones] = 1.0, 0.0
        if small == "b":
            A, B = B.T.contiguous(), A.T.contiguous()
        c = torch.zeros((n, n), device="cuda")
        b.chimera_op_gemm(A if a_kc else A.T.contiguous(), B.T.contiguous() if b_kc else B, c, n, n, n, a_kc, b_kc, b.EPI_NONE if a_kc else b.EPI_ACCUM_F32)
        want, size = A.double() @ B.double(), A.double().abs() @ B.double().abs()
        # the float instructions, which take every number here with all its bits, round once for every second product that is not zero; few sums at the end
        assert bool(((c.double() - want).abs() <= size * (left / 2 + 3) * 2.0 ** -24).all())


# single numbers too small for three parts in every tile of ordinary ones, which loses nothing that a result holds; beside them rows of zeros, and a row
# and a column of such numbers only, whose results would lose half of their bits; 64x64 and 128x128 tiles, ragged
@pytest.mark.parametrize("m,n,k", [(1032, 1016, 392), (2120, 2056, 200)])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
def test_float_split_of_few_small_numbers(m, n, k, layout):
    import torch
    print("float split few small", m, n, k, layout, flush=True)
    a_kc, b_kc = {"fwd": (1, 0), "dgrad": (1, 1), "wgrad": (0, 0)}[layout]
    gen = torch.Generator(device="cuda").manual_seed(m)
    A, B = torch.randn((m, k), generator=gen, device="cuda"), torch.randn((k, n), generator=gen, device="cuda")
    A[::7, ::11] *= 2.0 ** -121
    A[5::64], B[:, 9::64], B[3] = 0.0, 0.0, 0.0
    A[m - 1] *= 2.0 ** -125
    B[:, 200] *= 2.0 ** -125
    c = torch.zeros((m, n), device="cuda")
    b.chimera_op_gemm(A if a_kc else A.T.contiguous(), B.T.contiguous() if b_kc else B, c, m, n, k, a_kc, b_kc, b.EPI_NONE if a_kc else b.EPI_ACCUM_F32)
    want, size = A.double() @ B.double(), A.double().abs() @ B.double().abs()
    # a rounding for every second product on the float instructions, fewer on the others, and few sums at the end; what two such numbers make is below the
    # smallest float, a product of one and an ordinary one may end in subnormal sums
    assert bool(((c.double() - want).abs() <= size * (k / 2 + 9) * 2.0 ** -24 + k * 2.0 ** -149).all())


# a block whose grouped float weight gradients and bias gradients take 128x128 tiles, tokens with a remainder
def test_float_stage_on_wide_tiles():
    _stage(b.F32, 768, 12, 203, 1)


# operands with NaN between their rows (64x64 and 128x128 tiles), and with rows too far apart for the tiles' offsets (32x32 tiles)
@pytest.mark.parametrize("m,n,k,gap", [(1032, 584, 72, 8), (2600, 2600, 200, 24), (1032, 584, 8, 1 << 22)])
@pytest.mark.parametrize("layout", ["fwd", "dgrad", "wgrad"])
def test_float_split_strides(m, n, k, gap, layout):
    import torch
    print("float split strides", m, n, k, gap, layout, flush=True)
    a_kc, b_kc = {"fwd": (1, 0), "dgrad": (1, 1), "wgrad": (0, 0)}[layout]
    gen = torch.Generator(device="cuda").manual_seed(m)
    A, B = torch.randn((m, k), generator=gen, device="cuda"), torch.randn((k, n), generator=gen, device="cuda")

    def spread(X, wide):
        rows, cols = X.shape
        Y = torch.full((rows, cols + (gap if wide else 8)), float("nan"), device="cuda")
        Y[:, :cols] = X
        return Y

    few = gap > 1 << 20                                           # only eight rows of an operand may lie that far apart
    da, db = spread(A if a_kc else A.T, not few or not a_kc), spread(B.T if b_kc else B, not few or not b_kc)
    c = torch.zeros((m, n), device="cuda")
    b.chimera_op_gemm(da, db, c, m, n, k, a_kc, b_kc, b.EPI_NONE if a_kc else b.EPI_ACCUM_F32, lda=da.shape[1], ldb=db.shape[1])
    want, size = A.double() @ B.double(), A.double().abs() @ B.double().abs()
    # as above; the float instructions round once for every second product
    assert bool(((c.double() - want).abs() <= size * (12 + (k / 2 if few else k / 16)) * 2.0 ** -24).all())
