"""The routing loss at the edges of the probe's steps (64 or 32 tokens) and of
its split of a unit over workgroups (csrc/probe_split.h), against Eq. (2)
through Gram matrices in float64; with no residual entries (k = 0) the residual
loss equals the shared one.  Bar: the 2e-5 of the parity cases (each half
difference as a bf16 pair, 2^-18 relative, the dropped product of the low halves
as small).  Between splits a unit's loss differs by the rounding of fp32 sums of
up to 1024 tokens: twice sqrt(1024) 2^-24."""
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


RESPLIT = 4e-6


@pytest.mark.parametrize("layers,schedule,T", [(32, 0, 5000), (32, 0, 12345), (24, 2, 12345), (32, 1, 12345), (2, 0, 513)])
def test_a_units_loss_in_every_split(layers, schedule, T):
    """8 KV heads: 128 units of two layers, 48 of four, and both sizes in one probe (which split apart),
    with the workspace of the query and with one partial per 1024 tokens, against probes of one block
    alone; and the shared loss of a unit against float64."""
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import probe
    hkv, d, P = 8, 128, 16
    g = torch.Generator("cuda").manual_seed(T + layers)
    k = [torch.randn(hkv, T, d, generator=g, device="cuda").bfloat16() for _ in range(layers)]
    q = [torch.randn(hkv, P, d, generator=g, device="cuda").bfloat16() for _ in range(layers)]
    dm = B.dims(layers, hkv, hkv, d, 16, "bf16", schedule)
    err, _ = probe(dm, T, k, q, P)
    first, size = B.blocks(dm)
    least = layers * hkv * d * d * 4 + -(-len(first) * hkv * -(-T // 1024) * 8 // 256) * 256
    assert least <= B.probe_workspace(dm, T, P)
    ws = torch.full((least + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    few = torch.empty_like(err)
    B.probe(dm, T, k, q, P, few, ws[:least])
    assert bool((ws[least:] == 0xA5).all())
    with pytest.raises(B.FdkvError):
        B.probe(dm, T, k, q, P, few, ws[:least - 256])
    for b in sorted({0, len(first) // 2, len(first) - 1}):
        f, n = int(first[b]), int(size[b])
        one, _ = probe(B.dims(n, hkv, hkv, d, 16, "bf16", B.QUADS if n == 4 else B.PAIRS), T, k[f:f + n], q[f:f + n], P)
        for other in (one[0], few[b]):
            assert float(((other.double() - err[b].double()) / err[b].double()).abs().max()) <= RESPLIT, b
        x = torch.stack([t[5].double() for t in k[f:f + n]])
        want = sum(float((((x.mean(0) - x[p]) @ q[f + p][5].double().T.contiguous()) ** 2).sum()) for p in range(n))
        want /= n * P * d
        assert abs(float(err[b, 5, 0]) - want) <= 2e-5 * want, b
