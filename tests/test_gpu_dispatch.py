"""GPU parity at the edges of dispatch rules: sizes where a kernel variant begins or ends, and the
replay with its stages beside each other against the replay in turn."""
import numpy as np
import pytest

from oracle import edges_oracle as eo
from paper_2107_06925_amd import binding as b
from paper_2107_06925_amd import synth
from gpu_util import assert_close, make_stage, to_dev, to_np

pytestmark = pytest.mark.gpu


def _worker(overlap, shared_dx):
    import torch
    D, N, rank, L, H, heads, S, B = 4, 8, 1, 2, 128, 2, 72, 1
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
    torch.cuda.synchronize()
    return [t.clone() for t in outs] + [st.grads.clone() for st in stages]


@pytest.mark.parametrize("shared", [False, True])
def test_replay_beside_equals_replay_in_turn(shared):
    import torch
    print("replay lanes, shared dx", shared, flush=True)
    dx = torch.zeros((72, 128), device="cuda", dtype=torch.bfloat16) if shared else None
    for a, c in zip(_worker(True, dx), _worker(False, dx)):
        assert torch.equal(a, c)


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
