"""One evaluation workspace used for calls of changing shapes and modes: a call must never take a
word that an earlier call left for one of its own, so no call may leave a word that carries the
next call's tag anywhere but in the control block, whose place is the same for every shape."""
import numpy as np
import pytest
import torch

import paper_2510_20064_amd as hs

pytestmark = pytest.mark.gpu

CONTROL = 64 + 32 * 4096  # bytes of the control block
# (B, N, K, V): growing and shrinking; the counts of the first of each pair would lie among the
# second's slice sums, partials or argmax words if both kept their own place for them
SHAPES = [(32, 8, 16, 2048), (32, 8, 4, 33000), (1, 8, 7, 30001), (1, 8, 8, 30001), (48, 8, 32, 2048),
          (16, 8, 4, 33000), (40, 3, 5, 20000), (2, 64, 2, 9000), (64, 8, 6, 33000), (3, 1, 1, 5)]


def logits(B, N, K, V, seed):
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    x = torch.randn((N + 1, B, K, (V + 7) // 8 * 8), generator=g, device="cuda:0") * 3.0
    x[1:] = x[:1] + 0.7 * x[1:]
    x[N] = x[0]
    return x.to(torch.bfloat16)


def outputs(x, V, mode, fn, **kw):
    if mode == hs.GREEDY:
        B, N, K = x.shape[1], x.shape[0] - 1, x.shape[2]
        out = {"agree": torch.empty((B, N, K), dtype=torch.uint8, device=x.device),
               "argmax_t": torch.empty((B, K), dtype=torch.int32, device=x.device),
               "argmax_d": torch.empty((B, N, K), dtype=torch.int32, device=x.device)}
        return fn(x, V=V, mode=mode, out=out, **kw)
    return fn(x, V=V, temperature=0.7, mode=mode, out={}, **kw)


def check_no_word_of_the_next_call(ws):
    torch.cuda.synchronize()
    epoch = int(ws[:4].cpu().numpy().view(np.uint32)[0])
    tag = epoch % 0x7FFFFFFF + 1
    n = (ws.numel() - CONTROL) // 8 * 8
    words = ws[CONTROL:CONTROL + n].cpu().numpy().view(np.uint64)
    bad = np.nonzero((words & np.uint64(0x7FFFFFFF)) == np.uint64(tag))[0]
    assert bad.size == 0, (bad[:4], epoch)


def test_one_workspace_for_changing_shapes_and_modes():
    dt = hs.HS_BF16
    size = max(hs.eval_workspace_size(B, N, K, V, dt) for B, N, K, V in SHAPES)
    ws = torch.zeros(size, dtype=torch.uint8, device="cuda:0")
    for i, (B, N, K, V) in enumerate(SHAPES + SHAPES[::-1]):
        x = logits(B, N, K, V, i)
        for mode in ((hs.GREEDY,) if i % 2 == 0 else (hs.SAMPLE, hs.GREEDY, hs.GREEDY, hs.SAMPLE)):
            print("\n[case] B=%d N=%d K=%d V=%d mode=%d" % (B, N, K, V, mode), flush=True)
            got = outputs(x, V, mode, hs.eval_alpha, workspace=ws)
            check_no_word_of_the_next_call(ws)
            ref = outputs(x, V, mode, hs.eval_alpha)
            for k in ref:
                assert torch.equal(got[k], ref[k]), k
            if mode == hs.GREEDY:
                assert bool(got["agree"][:, N - 1].all())


def test_noalloc_for_changing_shapes_and_modes():
    for i, (B, N, K, V) in enumerate(SHAPES + SHAPES[::-1]):
        x = logits(B, N, K, V, i)
        mode = hs.SAMPLE if i % 2 else hs.GREEDY
        print("\n[case] noalloc B=%d N=%d K=%d V=%d mode=%d" % (B, N, K, V, mode), flush=True)
        ref = outputs(x, V, mode, hs.eval_alpha)
        for _ in range(4):
            got = outputs(x, V, mode, hs.eval_alpha_noalloc)
            torch.cuda.synchronize()
            for k in ref:
                assert torch.equal(got[k], ref[k]), k


@pytest.mark.parametrize("B,N,K,V", [(64, 8, 6, 4000), (48, 3, 8, 20011), (3, 19, 2, 700)])
def test_streamed_greedy_call_with_a_wait_that_gave_up(B, N, K, V):
    """A fold that loses a word marks its call's count of folded groups (byte 24, top bit) and every
    output is invalid, those of the groups that lost nothing too. The mark is set here by the host."""
    x = logits(B, N, K, V, V)
    ws = hs.alloc_workspace(B, N, K, V, hs.HS_BF16, "cuda:0")
    ref = outputs(x, V, hs.GREEDY, hs.eval_alpha, workspace=ws)
    assert bool(ref["agree"][:, N - 1].all())
    print("\n[case] failed fold B=%d N=%d K=%d V=%d" % (B, N, K, V), flush=True)
    ws[31] |= 0x80
    got = outputs(x, V, hs.GREEDY, hs.eval_alpha, workspace=ws)
    assert int(got["agree"].sum()) == 0
    assert bool((got["argmax_t"] == -2).all()) and bool((got["argmax_d"] == -2).all())
    check_no_word_of_the_next_call(ws)
    got = outputs(x, V, hs.GREEDY, hs.eval_alpha, workspace=ws)
    for k in ref:
        assert torch.equal(got[k], ref[k]), k
