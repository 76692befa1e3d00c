"""alpha whatever offset a row's logits have: a softmax does not see one, and neither may the kernels
that take exponentials against offsets of their own, at any temperature, for rows of one call
far apart from each other.

Bounds. Rounding c = log2(e)/T moves an exponent z c by 2^-25 of its distance to the row's largest:
6.2e-7 of a term 30 binary orders below it, of which alpha holds next to nothing. Exponents of
the kept form lie near 0 for the terms that matter (the offset is a thread's own maximum): 2^-25
each, with the roundings of exp2, of two sums and two logarithms 2^-24 each. So the kept form (one
item per workgroup) stays within 1.5e-6, and over many outputs within 2^-22 in the 2-norm. The
pipelined form keeps an offset and a difference of normalisers in one addend of up to 64 and exponents
of up to 64: 2^-19 (1.3e-6 of a term) each, for target and drafter, and sums against the common offset
have exponents of up to 96 (2^-18, 2.6e-6, at random from term to term): within 5e-6, and 2e-6 in the
2-norm.
"""
import pytest
import torch

import paper_2510_20064_amd as hs

pytestmark = pytest.mark.gpu

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
PIPELINED = [(48, 8, 4, 32000), (64, 3, 4, 20001), (30, 12, 3, 33001), (256, 1, 8, 9000)]
SINGLE = [(1, 8, 2, 4104), (1, 3, 2, 4097), (2, 5, 3, 20011), (1, 1, 4, 2050)]
# (temperature, target's shift, drafters' shift)
SHIFTS = [(1.0, 0.0, 0.0), (1.0, 20.0, 20.0), (1.0, -60.0, -60.0), (1.0, -40.0, 55.0),
          (1.0, 60.0, -40.0), (0.5, -25.0, 20.0), (0.5, 20.0, 20.0), (0.3, 12.0, -18.0),
          (0.3, -15.0, 12.0), (0.2, 10.0, -11.0), (0.2, 0.0, 0.0), (0.1, 0.0, 9.0), (0.1, 0.0, 0.0)]


def rows(B, N, K, V, seed):
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    t = torch.randn((B, K, V), generator=g, device="cuda:0") * 2.5
    boost = torch.randint(0, V, (B, K, 5), generator=g, device="cuda:0")
    t = t.scatter_add_(2, boost, torch.full(boost.shape, 6.0, device="cuda:0"))
    scale = torch.logspace(-1.5, 0.3, N, device="cuda:0").view(N, 1, 1, 1)
    d = t + scale * torch.randn((N, B, K, V), generator=g, device="cuda:0")
    return torch.cat([t[None], d])


def reference(x, V, T):
    p = torch.softmax(x[0, :, :, :V].double() / T, -1)
    q = [torch.softmax(x[1 + i, :, :, :V].double() / T, -1) for i in range(x.shape[0] - 1)]
    return torch.stack([torch.minimum(p, qi).sum(-1) for qi in q], 1)


@pytest.mark.parametrize("dtype", list(DTYPES))
@pytest.mark.parametrize("B,N,K,V", SINGLE + PIPELINED)
@pytest.mark.parametrize("arg", [False, True])
def test_alpha_under_shifts(B, N, K, V, dtype, arg):
    kept = (B, N, K, V) in SINGLE
    x0 = rows(B, N, K, V, V + N)
    for T, st, sd in SHIFTS:
        print("\n[case] T=%g shifts %g %g %s B=%d N=%d K=%d V=%d" % (T, st, sd, dtype, B, N, K, V),
              flush=True)
        x = torch.zeros((N + 1, B, K, (V + 7) // 8 * 8), dtype=DTYPES[dtype], device="cuda:0")
        x[0, :, :, :V] = x0[0] + st
        x[1:, :, :, :V] = x0[1:] + sd
        out = hs.eval_alpha(x, V=V, temperature=T, mode=hs.SAMPLE, want_argmax=arg)["alpha"].double()
        ref = reference(x, V, T)
        err = (out - ref).abs().max().item()
        assert err <= (1.5e-6 if kept else 5e-6), (T, st, sd, err)
        rel = ((out - ref).norm() / ref.norm()).item()
        assert rel <= (2.0 ** -22 if kept else 2e-6), (T, st, sd, rel)


@pytest.mark.parametrize("dtype", list(DTYPES))
@pytest.mark.parametrize("B,N,K,V", [(1, 8, 2, 4104), (48, 8, 4, 32000)])
def test_masked_and_far_apart_rows(B, N, K, V, dtype):
    """Threads and slices without a finite logit next to ordinary ones, on either side, at low
    temperature: the parts of one side that the other masks count nothing."""
    lowest = torch.finfo(DTYPES[dtype]).min
    x0 = rows(B, N, K, V, 3)
    for T, st, sd, fill in [(1.0, -40.0, 55.0, -float("inf")), (0.2, 10.0, -11.0, lowest),
                            (0.1, 0.0, 9.0, -float("inf")), (1.0, 60.0, -40.0, lowest)]:
        print("\n[case] masked T=%g shifts %g %g %s B=%d" % (T, st, sd, dtype, B), flush=True)
        x = torch.empty((N + 1, B, K, V), dtype=DTYPES[dtype], device="cuda:0")
        x[0] = x0[0] + st
        x[1:] = x0[1:] + sd
        x[0, :, 0, : V // 3] = fill              # the target masks a third
        x[1, :, :, V // 2:] = fill               # drafter 0 masks half
        x[2, :, 1, : V - 1] = fill               # drafter 1 all but one token
        x[3, :, 0, V // 3:] = fill               # drafter 2 shares no token with the target
        out = hs.eval_alpha(x, V=V, temperature=T, mode=hs.SAMPLE)["alpha"].double()
        err = (out - reference(x, V, T)).abs().max().item()
        assert err <= (1.5e-6 if B == 1 else 5e-6), (T, st, sd, err)
        assert (out[:, 2, 0] == 0).all()


def test_results_do_not_depend_on_the_items_before():
    """A wave takes an item against its threads' own offsets or the common one by that item alone:
    queries whose logits need the one, the other, or both within a row, in orders that change which
    item follows which, give bitwise the same alpha."""
    B, N, K, V = 96, 8, 4, 20001
    x0 = rows(B, N, K, V, 5).to(torch.bfloat16).float()
    x0[:, 1::4] -= 64.0                     # below the common range
    x0[:, 2::8] += 96.0                     # above it
    x0[:, 3::8, :, : V // 2] -= 64.0        # half of the slices below
    x0[1, 6::8] = x0[1, 6::8] * 0 - float("inf")
    x0[2, 7::8, :, ::3] = -float("inf")
    x0[3, 4::8, 0, 5000:12000] = -30.0      # near the lower end, where the test is not the rule
    x0[3, 0::8, 1, :] = -37.5
    x = torch.zeros((N + 1, B, K, (V + 7) // 8 * 8), dtype=torch.bfloat16, device="cuda:0")
    x[..., :V] = x0
    refs = {}  # with an argmax every wave takes its threads' own offsets
    for seed in range(6):
        g = torch.Generator().manual_seed(seed)
        perm = torch.randperm(B, generator=g) if seed else torch.arange(B)
        print("\n[case] order %d" % seed, flush=True)
        y = x[:, perm.to("cuda:0")].contiguous()
        for arg in (False, True):
            out = hs.eval_alpha(y, V=V, temperature=1.0, mode=hs.SAMPLE, want_argmax=arg)["alpha"]
            back = torch.empty_like(out)
            back[perm.to("cuda:0")] = out
            ref = refs.setdefault(arg, back)
            if seed == 0:
                d = (ref.double() - reference(x, V, 1.0)).abs()
                assert torch.equal(torch.isnan(ref), torch.isnan(d))
                assert d[~torch.isnan(d)].max().item() <= 5e-6
            assert torch.equal(torch.nan_to_num(back, nan=-1.0), torch.nan_to_num(ref, nan=-1.0)), (seed, arg)
