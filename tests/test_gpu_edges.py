"""GPU parity of the pipeline's two ends (embedding; LM head and loss) against the oracle."""
import numpy as np
import pytest

from oracle import edges_oracle as eo
from paper_2107_06925_amd import binding as b
from paper_2107_06925_amd import synth
from gpu_util import assert_close, to_dev, to_np

pytestmark = pytest.mark.gpu
DTYPES = [b.F32, b.BF16]


def _rand(shape, seed, dtype, scale=1.0):
    a = np.random.default_rng(seed).standard_normal(shape).astype(np.float32) * scale
    return synth.round_to_bf16(a) if dtype == b.BF16 else a


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("batch,seq,hidden,vocab", [(2, 64, 128, 50), (3, 40, 320, 1000), (8, 512, 1024, 50304), (1, 8, 8, 8)])
def test_embedding(dtype, batch, seq, hidden, vocab):
    import torch
    print("embedding", dtype, batch, seq, hidden, vocab, flush=True)
    M = batch * seq
    rng = np.random.default_rng(1)
    tokens = rng.integers(0, vocab, size=M).astype(np.int32)          # small vocabularies repeat tokens many times
    wte, wpe, dx = _rand((vocab, hidden), 2, dtype), _rand((seq, hidden), 3, dtype), _rand((M, hidden), 4, dtype)
    dtok = torch.from_numpy(tokens).cuda()
    x = torch.empty((M, hidden), dtype=to_dev(dx, dtype).dtype, device="cuda")
    b.chimera_op_embedding_fwd(dtok, seq, to_dev(wte, dtype), to_dev(wpe, dtype), x)
    assert_close(to_np(x), eo.embedding_fwd(tokens, seq, wte, wpe), dtype, "x")
    g0 = np.random.default_rng(5).standard_normal((vocab, hidden)).astype(np.float32)
    p0 = np.random.default_rng(6).standard_normal((seq, hidden)).astype(np.float32)
    dwte, dwpe = torch.from_numpy(g0.copy()).cuda(), torch.from_numpy(p0.copy()).cuda()
    b.chimera_op_embedding_bwd(dtok, seq, to_dev(dx, dtype), dwte, dwpe)
    torch.cuda.synchronize()
    want_te, want_pe = eo.embedding_bwd(dx, tokens, seq, vocab)
    assert_close(to_np(dwte) - g0, want_te, b.F32 if dtype == b.F32 else dtype, "dwte")
    assert_close(to_np(dwpe) - p0, want_pe, b.F32 if dtype == b.F32 else dtype, "dwpe")
    # reproducible bit for bit
    dwte2, dwpe2 = torch.from_numpy(g0.copy()).cuda(), torch.from_numpy(p0.copy()).cuda()
    b.chimera_op_embedding_bwd(dtok, seq, to_dev(dx, dtype), dwte2, dwpe2)
    torch.cuda.synchronize()
    assert torch.equal(dwte, dwte2) and torch.equal(dwpe, dwpe2)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("rows,vocab", [(37, 1000), (16, 50304), (300, 264), (2, 8)])
def test_softmax_xent(dtype, rows, vocab):
    import torch
    print("xent", dtype, rows, vocab, flush=True)
    z = _rand((rows, vocab), 7, dtype, 3.0)
    targets = np.random.default_rng(8).integers(0, vocab, size=rows).astype(np.int32)
    scale = 1.0 / rows
    dz = to_dev(z, dtype)
    loss_rows = torch.empty(rows, device="cuda")
    loss = torch.full((1,), 2.5, device="cuda")
    b.chimera_op_softmax_xent(dz, torch.from_numpy(targets).cuda(), scale, loss_rows, loss)
    torch.cuda.synchronize()
    want_loss, want_dz = eo.softmax_xent(z, targets, scale)
    assert abs(float(loss.item()) - 2.5 - want_loss) <= 1e-4 * max(1.0, abs(want_loss))
    assert_close(to_np(dz), want_dz, dtype, "dz")
    per_row = [eo.softmax_xent(z[t:t + 1], targets[t:t + 1], scale)[0] for t in range(min(rows, 8))]
    assert_close(to_np(loss_rows)[:len(per_row)], np.array(per_row), b.F32, "loss per row")


@pytest.mark.parametrize("vocab", [2048, 2056, 4096, 4104, 8192, 8200, 16384, 16392, 32768, 32776, 65536, 65544])
def test_softmax_xent_row_sizes(vocab):
    # ends of the ranges of the row kernels' sizes, extreme logits, targets at both ends of the row
    import torch
    print("xent row", vocab, flush=True)
    rows = 5
    z = _rand((rows, vocab), 21, b.BF16, 3.0)
    z[1] = synth.round_to_bf16(z[1] * 30)                     # one entry holds nearly all of the probability
    z[2] = -3.0e38
    z[2, vocab - 3] = 3.0e38                                  # the widest finite range
    z[2] = synth.round_to_bf16(z[2])
    z[3, ::2] = -np.inf                                       # masked entries
    targets = np.array([0, vocab - 1, vocab - 3, 1, vocab // 2], dtype=np.int32)
    dz = to_dev(z, b.BF16)
    loss_rows, loss = torch.empty(rows, device="cuda"), torch.zeros(1, device="cuda")
    b.chimera_op_softmax_xent(dz, torch.from_numpy(targets).cuda(), 0.25, loss_rows, loss)
    torch.cuda.synchronize()
    x = z.astype(np.float64)
    m = x.max(axis=1, keepdims=True)
    s = np.exp(x - m).sum(axis=1, keepdims=True)
    p = np.exp(x - m) / s
    rng = np.arange(rows)
    want_loss = 0.25 * ((m + np.log(s))[:, 0] - x[rng, targets])
    p[rng, targets] -= 1
    # float sums and exponentials: 1e-5 of the larger of the loss and the row's logits it is a difference of
    bound = 1e-5 * np.maximum(np.abs(want_loss), 0.25 * np.abs(m[:, 0]))
    assert np.all(np.abs(to_np(loss_rows) - want_loss) <= bound)
    assert_close(to_np(dz), 0.25 * p, b.BF16, "dz")


@pytest.mark.parametrize("dtype,tokens,hidden,vocab", [(b.F32, 256, 128, 1024), (b.BF16, 512, 256, 2048), (b.BF16, 200, 136, 1000),
                                                       (b.BF16, 4096, 1024, 50304)])
def test_head_loss(dtype, tokens, hidden, vocab):
    import torch
    print("head", dtype, tokens, hidden, vocab, flush=True)
    y = _rand((tokens, hidden), 11, dtype, 1.5)
    g = (1 + 0.1 * _rand((hidden,), 12, dtype)).astype(np.float32)
    g = synth.round_to_bf16(g) if dtype == b.BF16 else g
    be = _rand((hidden,), 13, dtype, 0.1)
    w = _rand((hidden, vocab), 14, dtype, 0.05)
    targets = np.random.default_rng(15).integers(0, vocab, size=tokens).astype(np.int32)
    scale = 1.0 / tokens
    td = to_dev(y, dtype).dtype
    dy = torch.empty((tokens, hidden), dtype=td, device="cuda")
    dg = torch.zeros(hidden, device="cuda"); db = torch.zeros(hidden, device="cuda")
    dw = torch.zeros((hidden, vocab), device="cuda")
    loss = torch.zeros(1, device="cuda")
    args = (to_dev(y, dtype), torch.from_numpy(targets).cuda(), to_dev(g, dtype), to_dev(be, dtype), to_dev(w, dtype), scale,
            dy, dg, db, dw, loss)
    ws = b.chimera_head_loss(*args)
    b.chimera_head_loss(*args, workspace=ws)                  # a second micro-batch accumulates
    torch.cuda.synchronize()
    want = eo.head_fwd_bwd(y, targets, g, be, w, scale)
    assert abs(float(loss.item()) - 2 * want["loss"]) <= (1e-4 if dtype == b.F32 else 2e-2) * abs(2 * want["loss"])
    assert_close(to_np(dy), want["dy"], dtype, "dy")
    assert_close(to_np(dw), 2 * want["dw_head"], dtype, "dw_head")
    assert_close(to_np(dg), 2 * want["dlnf_g"], dtype, "dlnf_g")
    assert_close(to_np(db), 2 * want["dlnf_b"], dtype, "dlnf_b")


@pytest.mark.parametrize("tokens,hidden,vocab", [(130, 136, 20008), (1, 8, 16384), (264, 520, 30072), (40, 1032, 65528), (1100, 392, 12296)])
def test_head_split_data_gradient(tokens, hidden, vocab):
    # Few output tiles over a long vocabulary: the data gradient is cut along it where the workspace has
    # room for the partial sums, and whole where it only holds the rest.
    import torch
    print("head split", tokens, hidden, vocab, flush=True)
    y, w = _rand((tokens, hidden), 31, b.BF16, 1.5), _rand((hidden, vocab), 32, b.BF16, 0.05)
    g, be = synth.round_to_bf16((1 + 0.1 * _rand((hidden,), 33, b.BF16)).astype(np.float32)), _rand((hidden,), 34, b.BF16, 0.1)
    targets = np.random.default_rng(35).integers(0, vocab, size=tokens).astype(np.int32)
    want = eo.head_fwd_bwd(y, targets, g, be, w, 1.0 / tokens)
    full = b.lib().chimera_head_workspace_bytes(b.BF16, tokens, hidden, vocab)
    b.check(b.lib().chimera_op_gemm_tuning(0, 0, 0, 1))         # register-staged products only: never cut
    try:
        least = b.lib().chimera_head_workspace_bytes(b.BF16, tokens, hidden, vocab)
    finally:
        b.check(b.lib().chimera_op_gemm_tuning(0, 0, 0, 0))
    assert full > least and (full - least) % (tokens * hidden * 4) < 256        # whole slabs, rounded up to 256 bytes
    for size in (full, full - 1, least):
        dy = torch.empty((tokens, hidden), dtype=torch.bfloat16, device="cuda")
        dg, db = torch.zeros(hidden, device="cuda"), torch.zeros(hidden, device="cuda")
        dw, loss = torch.zeros((hidden, vocab), device="cuda"), torch.zeros(1, device="cuda")
        ws = torch.full((size,), 0xff, dtype=torch.uint8, device="cuda")         # NaN wherever nothing is written
        b.chimera_head_loss(to_dev(y, b.BF16), torch.from_numpy(targets).cuda(), to_dev(g, b.BF16), to_dev(be, b.BF16),
                            to_dev(w, b.BF16), 1.0 / tokens, dy, dg, db, dw, loss, workspace=ws)
        torch.cuda.synchronize()
        assert_close(to_np(dy), want["dy"], b.BF16, "dy")
        assert_close(to_np(dg), want["dlnf_g"], b.BF16, "dlnf_g")
        assert_close(to_np(dw), want["dw_head"], b.BF16, "dw_head")


def test_edge_argument_errors():
    import torch
    tok = torch.zeros(16, dtype=torch.int32, device="cuda")
    w = torch.zeros((8, 12), device="cuda")
    with pytest.raises(b.ChimeraError):
        b.chimera_op_embedding_fwd(tok, 8, w, w, torch.zeros((16, 12), device="cuda"))        # hidden not a multiple of 8
    w = torch.zeros((8, 16), device="cuda")
    with pytest.raises(b.ChimeraError):
        b.chimera_op_embedding_fwd(tok, 5, w, w, torch.zeros((16, 16), device="cuda"))        # tokens not a multiple of seq
    z = torch.zeros((4, 12), device="cuda")
    with pytest.raises(b.ChimeraError):
        b.chimera_op_softmax_xent(z, tok, 1.0, torch.zeros(4, device="cuda"), torch.zeros(1, device="cuda"))
    y = torch.zeros((16, 16), device="cuda")
    wh = torch.zeros((16, 64), device="cuda")
    small = torch.zeros(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(b.ChimeraError) as e:
        b.chimera_head_loss(y, tok, y[0], y[0], wh, 1.0, torch.zeros_like(y), torch.zeros(16, device="cuda"),
                            torch.zeros(16, device="cuda"), torch.zeros_like(wh), torch.zeros(1, device="cuda"), workspace=small)
    assert e.value.code == b.ENOMEM


# Token lists of the embedding backward: one token everywhere, every second position, more positions of one owner's tokens than a
# list holds, frequent tokens beside rare ones of the same bucket, rows that end inside a slice.  Integers, so that float sums are exact.
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("tokens,hidden,vocab,kind", [
    (17, 8, 5, "same"), (2049, 136, 70000, "same"), (4096, 264, 1000, "padding"), (5000, 136, 40000, "owner"), (6144, 72, 40000, "bucket"),
    (16384, 128, 3000, "log"), (4097, 1032, 50304, "log"), (600, 2048, 40, "log"),
    (463, 24, 900, "log"), (65, 192, 3, "uniform"), (4096, 64, 125, "uniform"), (8193, 64, 250, "uniform"), (70000, 40, 30000, "dense"), (70001, 24, 90, "uniform")])
def test_embedding_backward_lists(tokens, hidden, vocab, kind, dtype):
    import torch
    print("embedding backward lists", tokens, hidden, vocab, kind, dtype, flush=True)
    rng = np.random.default_rng(tokens)
    ids = np.minimum(np.exp(rng.random(tokens) * np.log(vocab)).astype(np.int64) - 1, vocab - 1).clip(0)
    if kind == "same":
        ids[:] = 3
    elif kind == "padding":
        ids[::2] = 1
    elif kind == "owner":
        ids = rng.integers(0, vocab // 1024, tokens) * 1024 + 5
    elif kind == "bucket":
        ids[::3], ids[1::700] = 7, 7 + 16384
    elif kind == "uniform":                        # as many positions per token as make one frequent, a few more or fewer
        ids = rng.integers(0, vocab, tokens)
    elif kind == "dense":                          # one owner's tokens, none frequent, fill a stretch of positions and are few around it
        ids = rng.integers(0, vocab, tokens)
        ids[20000:23500] = rng.integers(0, 16, 3500) * 1024 + 5
        ids[60000::3] = rng.integers(0, 16, 3334) * 1024 + 5
    ids = ids.astype(np.int32)
    dx = rng.integers(-4, 5, (tokens, hidden)).astype(np.float32)
    dwte, dwpe = torch.ones((vocab, hidden), device="cuda"), torch.zeros((1, hidden), device="cuda")
    b.chimera_op_embedding_bwd(torch.from_numpy(ids).cuda(), 1, to_dev(dx, dtype), dwte, dwpe)
    want = np.ones((vocab, hidden), np.float32)
    np.add.at(want, ids, dx)
    assert np.array_equal(dwte.cpu().numpy(), want)
    assert np.array_equal(dwpe.cpu().numpy()[0], dx.sum(0))


# Many positions spread evenly over the vocabulary: no token is frequent among them, so every row is one owner's few additions.  Measured,
# gradients of 128 MiB: 0.6 ms, four of a copy's per byte; 8.4 ms when every token of a busy bucket was taken for a frequent one.
def test_embedding_backward_of_many_even_positions():
    import torch
    M, H, V = 262144, 256, 30000
    ids = torch.randint(0, V, (M,), device="cuda", dtype=torch.int32)
    dx, other = torch.zeros((M, H), device="cuda", dtype=torch.bfloat16), torch.empty((M, H), device="cuda", dtype=torch.bfloat16)
    dwte, dwpe = torch.zeros((V, H), device="cuda"), torch.zeros((2048, H), device="cuda")

    def best(fn):
        times = []
        for _ in range(5):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record(), fn(), t1.record()
            t1.synchronize()
            times.append(t0.elapsed_time(t1))
        return min(times)

    copy = best(lambda: other.copy_(dx))
    bwd = best(lambda: b.chimera_op_embedding_bwd(ids, 2048, dx, dwte, dwpe))
    print("embedding backward %.3f ms, copy %.3f ms" % (bwd, copy), flush=True)
    assert bwd <= 40 * copy
