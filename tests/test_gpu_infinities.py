"""Infinite inputs: what they reach, and what stays finite."""
import math

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("c", [6, 7])
def test_an_infinite_kept_channel_leaves_a_pairs_residual_loss_finite(dtype, d, c):
    """The channel is among the token's top-k, so the residual deviation drops it, and its neighbours'
    deviations are finite: the loss is Eq. (2) without it, at the 2e-5 of the parity cases."""
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import probe
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    hkv, G, P, T, k = 2, 2, 24, 200, 4
    g = torch.Generator("cuda").manual_seed(d + c)
    kl = [torch.randn(hkv, T, d, generator=g, device="cuda").to(tdt) for _ in range(2)]
    q = [torch.randn(hkv * G, P, d, generator=g, device="cuda").to(tdt) for _ in range(2)]
    kl[0][0, 57, c] = math.inf
    kl[1][1, 130, c] = -math.inf
    err, _ = probe(B.dims(2, hkv, hkv * G, d, k, dtype), T, kl, q, P)
    for h in range(hkv):
        x = kl[0][h].double() - kl[1][h].double()
        top = (kl[0][h].float() - kl[1][h].float()).abs().sort(dim=1, descending=True, stable=True)[1][:, :k]
        kept = torch.zeros_like(x, dtype=torch.bool).scatter_(1, top, True)
        dev = torch.where(kept, torch.zeros_like(x), x / 2)
        want = sum(float(((dev @ q[p].double().reshape(hkv, G * P, d)[h].T.contiguous()) ** 2).sum()) for p in range(2))
        want /= 2 * G * P * d
        got = err[0, h].tolist()
        assert not math.isfinite(got[0]) and abs(got[1] - want) <= 2e-5 * want, (h, got, want)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
def test_an_infinite_layer_reaches_both_losses_of_a_block_of_four(dtype, d):
    """The mean of the four layers and every coefficient are infinite there: so is what decode would rebuild."""
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import probe
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator("cuda").manual_seed(d)
    kl = [torch.randn(2, 100, d, generator=g, device="cuda").to(tdt) for _ in range(4)]
    q = [torch.randn(4, 24, d, generator=g, device="cuda").to(tdt) for _ in range(4)]
    kl[2][1, 33, 5] = math.inf
    err, _ = probe(B.dims(4, 2, 4, d, 8, dtype, B.QUADS), 100, kl, q, 24)
    assert torch.isfinite(err[0, 0]).all() and not torch.isfinite(err[0, 1]).any()


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("rows", [32, 64, 96])
def test_an_infinite_deviation_makes_the_shared_loss_of_a_token_set_infinite(d, rows):
    """bf16 probe rows in multiples of 32 are not padded with rows of zeros, whose product with an infinite
    deviation is NaN: the token's score and the shared loss are infinite."""
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import probe
    G, T = 2, 200
    g = torch.Generator("cuda").manual_seed(d + rows)
    kl = [torch.randn(1, T, d, generator=g, device="cuda").bfloat16() for _ in range(2)]
    q = [torch.randn(G, rows // G, d, generator=g, device="cuda").bfloat16() for _ in range(2)]
    kl[0][0, 57, 3] = math.inf
    err, score = probe(B.dims(2, 1, G, d, 0, "bf16", B.PAIRS, B.RES_TOKENS, 50000), T, kl, q, rows // G)
    assert score[0, 0, 57] == math.inf and err[0, 0, 0] == math.inf
    assert int(torch.isfinite(score).sum()) == T - 1
