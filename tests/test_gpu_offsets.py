"""alpha whatever offset a row's logits have: a softmax does not see one, and neither may the kernels
that take exponentials against offsets of their own, at any temperature, for rows of one call
far apart from each other.

Bounds. Rounding c = log2(e)/T moves an exponent z c by 2^-25 of its distance to the row's largest:
6.2e-7 of a term 30 binary orders below it, of which alpha holds next to nothing. Exponents of
the kept form lie near 0 for the terms that matter (the offset is a thread's own maximum): 2^-25
each, with the roundings of exp2, of two sums and two logarithms 2^-24 each. So the kept form (one
item per workgroup) stays within 1.5e-6, and over many outputs within 2^-22 in the 2-norm.
"""
import pytest
import torch

import paper_2510_20064_amd as hs

pytestmark = pytest.mark.gpu

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
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
@pytest.mark.parametrize("B,N,K,V", SINGLE)
@pytest.mark.parametrize("arg", [False, True])
def test_alpha_under_shifts(B, N, K, V, dtype, arg):
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
        assert err <= 1.5e-6, (T, st, sd, err)
        rel = ((out - ref).norm() / ref.norm()).item()
        assert rel <= 2.0 ** -22, (T, st, sd, rel)


@pytest.mark.parametrize("dtype", list(DTYPES))
@pytest.mark.parametrize("B,N,K,V", [(1, 8, 2, 4104)])
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
        assert err <= 1.5e-6, (T, st, sd, err)
        assert (out[:, 2, 0] == 0).all()
