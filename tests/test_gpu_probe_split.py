"""The routing loss at the edges of the probe's steps (64 or 32 tokens) and of
its split of a unit over workgroups, against Eq. (2) through Gram matrices in
float64; with no residual entries (k = 0) the residual loss equals the shared
one.  Bar: the 2e-5 of the parity cases (each half difference as a bf16 pair,
2^-18 relative, the dropped product of the low halves as small)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,schedule", [("bf16", 128, 0), ("bf16", 64, 0), ("bf16", 128, 2), ("bf16", 64, 2),
                                              ("f32", 128, 0), ("f32", 64, 2)])
def test_loss_at_the_edges_of_steps_and_workgroups(dtype, d, schedule):
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import probe
    g = torch.Generator("cuda").manual_seed(d + schedule)
    size, layers, hkv, G, P = (4, 8, 3, 2, 24) if schedule else (2, 4, 3, 2, 24)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    dm = B.dims(layers, hkv, hkv * G, d, 0, dtype, schedule)
    q = [torch.randn(hkv * G, P, d, generator=g, device="cuda").to(tdt) for _ in range(layers)]
    S = [torch.stack([x.double().reshape(hkv, G * P, d)[h].T @ x.double().reshape(hkv, G * P, d)[h] for h in range(hkv)])
         for x in q]
    full = [torch.randn(hkv, 5000, d, generator=g, device="cuda").to(tdt) for _ in range(layers)]
    for T in (1, 31, 32, 33, 63, 64, 65, 1023, 1024, 1025, 1057, 2049, 3073, 5000):
        k = [x[:, :T].contiguous() for x in full]
        err, _ = probe(dm, T, k, q, P)
        for b in range(layers // size):
            x = torch.stack([t.double() for t in k[b * size:(b + 1) * size]])
            dev = x.mean(0) - x
            for h in range(hkv):
                want = sum(float(((dev[p, h].T @ dev[p, h]) * S[b * size + p][h]).sum()) for p in range(size))
                want /= size * G * P * d
                got = err[b, h].tolist()
                assert abs(got[0] - want) <= 2e-5 * want and abs(got[1] - got[0]) <= 2e-5 * want, (T, b, h, got, want)
