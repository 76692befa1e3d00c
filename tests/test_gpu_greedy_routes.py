"""Greedy calls on both sides of the line between the team kernel and the streaming argmax kernel:
groups of few and of many units and waves, few and many row sets, teams with at most two items, with
up to six and with more, rows of few slices, rows that end inside a vector, slices and units that end
inside a row. Argmaxes and agreements are whole numbers: exact. Interleaved on one workspace with
calls that need alpha."""
import numpy as np
import pytest
import torch

import paper_2510_20064_amd as hs

pytestmark = pytest.mark.gpu

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def reference(x, V):
    """Lowest index of each row's maximum, NaN ignored."""
    z = x[..., :V].float()
    z = torch.where(torch.isnan(z), torch.full_like(z, -float("inf")), z)
    i = torch.arange(V, device=z.device, dtype=torch.int32)
    i = torch.where(z == z.amax(-1, keepdim=True), i, V)
    return i.amin(-1).cpu().numpy()


@pytest.mark.parametrize("dtype", list(DTYPES))
@pytest.mark.parametrize("N,K,V", [(8, 3, 20489), (5, 7, 50257), (1, 4, 8200), (20, 3, 30001),
                                   (3, 2, 4097), (8, 8, 4000), (17, 2, 37314), (47, 3, 33001),
                                   (43, 9, 8032)])
def test_greedy_over_the_batch_sizes(N, K, V, dtype):
    for B in (1, 2, 5, 12, 17, 33):
        ld = (V + 7) // 8 * 8
        if (N + 1) * B * K * ld > 1 << 28:
            continue
        print("\n[case] greedy %s B=%d N=%d K=%d V=%d" % (dtype, B, N, K, V), flush=True)
        g = torch.Generator(device="cuda:0").manual_seed(B * 100 + N)
        x = torch.randn((N + 1, B, K, ld), generator=g, device="cuda:0") * 3.0
        x[N] = x[0]
        x[0, 0, 0, ::7] = -float("inf")
        x[N, B - 1, K - 1, 5] = float("nan")
        x[1, 0, 0] = x[1, 0, 0].round()  # ties
        x = x.to(DTYPES[dtype])
        ref = reference(x, V)
        ws = hs.alloc_workspace(B, N, K, V, hs._dtype_code(x), "cuda:0")
        for mode in (hs.GREEDY, hs.SAMPLE, hs.GREEDY, hs.GREEDY):
            out = hs.eval_alpha(x, V=V, mode=mode, want_alpha=mode == hs.SAMPLE, want_agree=True,
                                want_argmax=True, workspace=ws)
            torch.cuda.synchronize()
            at, ad = out["argmax_t"].cpu().numpy(), out["argmax_d"].cpu().numpy()
            assert np.array_equal(at, ref[0])
            assert np.array_equal(ad, ref[1:].transpose(1, 0, 2))
            assert np.array_equal(out["agree"].cpu().numpy(), (ad == at[:, None]).astype(np.uint8))
