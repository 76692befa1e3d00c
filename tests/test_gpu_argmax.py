"""Greedy calls without alpha (the streaming argmax kernel and the team kernel's argmax variant), the
alpha kernel's sums against a common offset and against a thread's own, and the row statistics, at
the sizes where their dispatch turns.

The argmax kernel cuts rows into units of 512 16-byte vectors and gives waves spans of units, so
the edges are rows of one vector, of a partial vector only, of one unit and one logit more, and
batches whose spans cross rows and groups. The alpha kernel with several items per workgroup takes
a thread's sums of up to 8 terms against a common offset of 8 binary orders at T = 1 (5.5 logits)
and an item again, by its threads' largest logits, where a sum leaves [2^-56, 2^96]: logits near
-33 and +72, which shifts by multiples of 40 cross for some rows of an item and not for others.
"""
import numpy as np
import pytest
import torch

import paper_2510_20064_amd as hs

pytestmark = pytest.mark.gpu

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def note(what):
    print("\n[case] " + what, flush=True)


def logits(shape, dtype, seed, kind):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(shape, generator=g) * 3.0
    if kind == "ties":
        x = x.round()
    elif kind == "zeros":
        x = x.sign() * 0.0  # +0 and -0 tie
    elif kind == "masked":
        x[torch.rand(shape, generator=g) < 0.4] = -float("inf")
    elif kind == "nan":
        x[torch.rand(shape, generator=g) < 0.02] = float("nan")
    return x.to(DTYPES[dtype])


def reference(x, V):
    """Lowest index of each row's maximum, NaN ignored."""
    z = x[..., :V].float().numpy()
    z = np.where(np.isnan(z), -np.inf, z)
    return np.argmax(z, axis=-1).astype(np.int32)


@pytest.mark.parametrize("dtype", list(DTYPES))
@pytest.mark.parametrize("kind", ["plain", "ties", "zeros", "masked", "nan"])
@pytest.mark.parametrize("B,N,K,V", [
    (1, 1, 1, 1), (2, 3, 2, 7), (1, 2, 1, 8), (3, 5, 2, 2049), (2, 8, 3, 4096), (2, 4, 1, 4097),
    (1, 64, 2, 8200), (5, 7, 3, 33001), (24, 3, 2, 20011)])
def test_argmax_and_agreement(B, N, K, V, kind, dtype):
    note("argmax %s %s B=%d N=%d K=%d V=%d" % (dtype, kind, B, N, K, V))
    x = logits((N + 1, B, K, (V + 7) // 8 * 8), dtype, 7 * V + N, kind)
    x[N] = x[0]  # one drafter always agrees
    ref = reference(x, V)
    live = (x[..., :V] > -float("inf")).any(-1).numpy()
    xd = x.to("cuda:0")
    ws = hs.alloc_workspace(B, N, K, V, hs._dtype_code(xd), "cuda:0")
    for mode in (hs.GREEDY, hs.SAMPLE, hs.GREEDY):  # one workspace, both kernels in turn
        out = hs.eval_alpha(xd, V=V, temperature=1.0, mode=mode, want_agree=True,
                            want_alpha=mode == hs.SAMPLE, want_argmax=True, workspace=ws)
        torch.cuda.synchronize()
        at = out["argmax_t"].cpu().numpy()
        ad = out["argmax_d"].cpu().numpy()
        rows, d = live[0], live[1:].transpose(1, 0, 2)
        assert np.array_equal(at[rows], ref[0][rows])
        assert np.array_equal(ad[d], ref[1:].transpose(1, 0, 2)[d])
        agree = out["agree"].cpu().numpy()
        assert np.array_equal(agree, (ad == at[:, None]).astype(np.uint8))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shift", [-120.0, -80.0, -40.0, 40.0, 80.0])
@pytest.mark.parametrize("B,N,K,V", [(1, 8, 2, 4104), (1, 3, 2, 4104), (48, 8, 4, 32000)])
def test_sums_outside_the_plain_range(B, N, K, V, shift, dtype):
    # some rows shifted (a softmax does not see it), so that rows against the common offset and
    # against their threads' own share items; 48 queries run the pipelined kernel, one the kernel
    # with one item per workgroup, whose exponents lie near 0: 2^-25 each, with exp2, two sums and
    # two logarithms 2^-24 each, within 1.5e-6. The pipelined kernel's exponents reach 96 against the
    # common offset (rounded at 2^-18: 2.6e-6 of a term after the factor ln 2, at random from term
    # to term), and the min-sums' 64, for target and drafter (2^-19, 1.3e-6 each): within 5e-6
    note("shift %g %s B=%d N=%d" % (shift, dtype, B, N))
    x = logits((N + 1, B, K, V), "f32", 11, "plain")
    x = (x * 8).round() / 8
    x[1:] = (x[:1] + 0.5 * x[1:]).mul(4).round() / 4
    x[0, :, 0] += shift
    x[1, :, K - 1] += shift
    x[N] += shift
    x = x.to(DTYPES[dtype])
    z = x.double()
    p, q = torch.softmax(z[0], -1), torch.softmax(z[1:], -1)
    ref = torch.minimum(p, q).sum(-1).permute(1, 0, 2)
    out = hs.eval_alpha(x.to("cuda:0"), V=V, temperature=1.0, mode=hs.SAMPLE, want_alpha=True)
    torch.cuda.synchronize()
    err = (out["alpha"].cpu().double() - ref).abs().max().item()
    assert err <= (1.5e-6 if B == 1 else 5e-6), err


@pytest.mark.parametrize("dtype,rows", [("bf16", 1), ("bf16", 511), ("bf16", 512), ("f16", 3),
                                        ("f32", 5), ("f32", 3071), ("f32", 3072)])
@pytest.mark.parametrize("V", [3, 2050, 8193, 16391])
def test_row_statistics_by_row_count(rows, V, dtype):
    # fp32 sums of up to 16391 terms in a few hundred partial sums: relative 1e-6, over log terms
    note("stats %s rows=%d V=%d" % (dtype, rows, V))
    x = logits((rows, (V + 7) // 8 * 8), dtype, rows + V, "ties" if V == 2050 else "plain")
    mx, lse, am = hs.softmax_stats(x.to("cuda:0"), V=V, temperature=0.7)
    torch.cuda.synchronize()
    z = x[:, :V].double()
    assert torch.equal(mx.cpu().double(), z.amax(1))
    assert np.array_equal(am.cpu().numpy(), np.argmax(x[:, :V].float().numpy(), axis=1))
    ref = torch.logsumexp(z / 0.7, dim=1)
    assert ((lse.cpu().double() - ref).abs() <= 1e-6 * (1 + ref.abs())).all()


# both sides of every line of the rule: short and long rows of few, 16-bit rows of 64000 logits around
# 1024 of them, fp32 rows of 50000 around 1200 and 3072. Bound as above, with 1.5e-6 for the longest
# rows: sixteen times the terms per thread, whose sums round in turn
@pytest.mark.parametrize("dtype,rows,V", [
    ("bf16", 256, 13103), ("bf16", 256, 13112), ("f32", 256, 13100), ("f32", 256, 13108),
    ("bf16", 257, 24569), ("bf16", 511, 24576), ("f32", 300, 24570), ("f32", 511, 24577),
    ("f16", 1023, 64000), ("bf16", 1024, 64001), ("bf16", 700, 63990), ("f16", 512, 64007),
    ("f32", 1199, 50001), ("f32", 1200, 50000), ("f32", 1200, 49995), ("f32", 512, 50003),
    ("f32", 3071, 50000), ("f32", 3072, 50000)])
def test_row_statistics_at_the_lines_of_the_rule(rows, V, dtype):
    note("stats %s rows=%d V=%d" % (dtype, rows, V))
    g = torch.Generator(device="cuda:0").manual_seed(rows + V)
    x = (torch.randn((rows, (V + 7) // 8 * 8), generator=g, device="cuda:0") * 3.0).to(DTYPES[dtype])
    x[rows // 2, V - 1] = 40.0
    mx, lse, am = hs.softmax_stats(x, V=V, temperature=0.7)
    torch.cuda.synchronize()
    for r in range(0, rows, 256):
        z = x[r:r + 256, :V].float()
        top = z.amax(1)
        first = torch.where(z == top[:, None], torch.arange(V, device=z.device), V).amin(1)
        assert torch.equal(mx[r:r + 256], top)
        assert torch.equal(am[r:r + 256].long(), first)
        ref = torch.logsumexp(z.double() / 0.7, dim=1)
        assert ((lse[r:r + 256].double() - ref).abs() <= 1.5e-6 * (1 + ref.abs())).all()
