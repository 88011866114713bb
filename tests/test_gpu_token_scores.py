"""The token scores of the probe at the edges of their rounds of probe rows (64)
and of the waves' and workgroups' tokens, for every block size and type: the
largest |q . dev| over the probe rows in float64, with the deviations rounded to
bf16 as the kernel's products take them.  What is left is the fp32 sum of d
exact products (fp32 queries: of their bf16 pairs, 2^-17 relative): 2^-16 of
sum |q| |dev|."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,schedule", [("bf16", 128, 0), ("bf16", 64, 0), ("bf16", 128, 2), ("bf16", 64, 2),
                                              ("f32", 64, 0)])
def test_scores_at_the_edges_of_rounds_and_workgroups(dtype, d, schedule):
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import probe
    g = torch.Generator("cuda").manual_seed(d + schedule)
    size, hkv = (4 if schedule else 2), 2
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    full = [torch.randn(hkv, 1100, d, generator=g, device="cuda").to(tdt) for _ in range(size)]
    for G, P in ((1, 1), (1, 31), (2, 16), (1, 33), (1, 63), (4, 16), (1, 65), (2, 65)):
        dm = B.dims(size, hkv, hkv * G, d, 0, dtype, schedule, B.RES_TOKENS, 50000)
        q = [torch.randn(hkv * G, P, d, generator=g, device="cuda").to(tdt) for _ in range(size)]
        for T in (1, 63, 65, 255, 257, 511, 513, 1100):
            k = [x[:, :T].contiguous() for x in full]
            _, got = probe(dm, T, k, q, P)
            x = torch.stack([t.float() for t in k])
            if size == 2:
                dev = torch.stack([(x[0] - x[1]) * 0.5, (x[1] - x[0]) * 0.5])
            else:
                dev = x - ((x[0] + x[3]) + (x[1] + x[2])) * 0.25
            dev = dev.bfloat16().double()
            for h in range(hkv):
                rows = torch.stack([t.double().reshape(hkv, G * P, d)[h] for t in q])          # [B][GP][d]
                logit = torch.stack([dev[p, h] @ rows[p].T.contiguous() for p in range(size)])
                scale = torch.stack([dev[p, h].abs() @ rows[p].abs().T.contiguous() for p in range(size)])
                want, bar = logit.abs().amax((0, 2)), scale.amax((0, 2)) * 2.0 ** -16
                assert bool(((got[0, h].double() - want).abs() <= bar).all()), (G, P, T, h)
