"""The split-K decode (csrc/decode_shape.h) at the edges of its chunks, waves and
tiles.  A bf16 sequence's outputs are the same bits whatever the call around it:
any workspace, the two-phase call, a bound on the lengths that makes more than
192 chunks, alone or in a batch.  Of an fp32 cache that holds between small
calls (chunks spread over workgroups, or their groups of waves in one), and up
to the rounding of fp32 sums against calls of more than 192 chunks (one
workgroup of four waves).  The outputs of every launch shape are held to the
oracle's decode."""
import math

import numpy as np
import pytest

import oracle as O
from synth import WORKLOADS, gen, scaled

from gpu_cases import oracle_decode_layer, rel_l2

pytestmark = pytest.mark.gpu

GROUPS = {"g1": 1, "g2": 2, "g4": 4, "g8": 8}
LONG = 65 * 512                     # a bound on the lengths: more than 192 chunks with three KV heads
# fp32 sums in another order: about sqrt(terms) roundings of 2^-24 on sums over some 1000 tokens and
# 128 channels, which the exponential of a logit of up to some 30 multiplies
REORDERED = 2e-6


def _cache(w, modes):
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import CompressedCache, probe, to_device
    dm = B.dims(**w.dims())
    cache = CompressedCache(dm, w.seq_lens, modes)
    data = []
    for s, T in enumerate(w.seq_lens):
        if T == 0:
            data.append(None)
            continue
        one = scaled(w, seq_lens=(T,))
        K, V = gen.layer_cache(one, 0)
        kl, vl = ([to_device(X, w.dtype)[l] for l in range(w.n_layers)] for X in (K, V))
        scores = None
        if w.residual:
            qp = to_device(gen.probe_queries(one, 0), w.dtype)
            _, scores = probe(dm, T, kl, [qp[l] for l in range(w.n_layers)], w.n_probe)
        cache.compress(s, kl, vl, token_scores=scores)
        data.append((one, K, V))
    return cache, data


def _records(dm, chunks):
    """Bytes of one record per chunk."""
    return chunks * (dm.n_q_heads // dm.n_kv_heads) * (dm.head_dim + 4) * 4


def _nan(n):
    import torch
    return torch.full((n // 4,), float("nan"), device="cuda")


@pytest.mark.parametrize("g,hkv", [(g, 3) for g in GROUPS] + [("g2", 9)])
@pytest.mark.parametrize("d,dtype,schedule,tok", [(128, "bf16", 0, 0), (64, "bf16", 0, 0), (128, "bf16_e4m3", 2, 0),
                                                  (64, "bf16_e4m3", 0, 0), (128, "bf16", 2, 200000),
                                                  (64, "bf16", 0, 300000), (128, "f32", 0, 0), (64, "f32", 2, 0),
                                                  (64, "f32", 0, 300000)])
def test_a_sequence_gives_the_same_bits_in_every_call(g, hkv, d, dtype, schedule, tok):
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import to_device
    G = GROUPS[g]
    # below, at and above a tile, a wave's tokens, a chunk
    lens = (1, 8, 33, 127, 129, 256, 511, 513, 0, 1100) if hkv == 3 else (8, 129, 513)
    w = scaled(WORKLOADS["prefill8b"], n_layers=4, n_kv_heads=hkv, n_q_heads=hkv * G, head_dim=d, dtype=dtype, topk=d // 8,
               schedule=schedule, seq_lens=lens, n_needles=1, n_probe=8, **(dict(residual=1, res_ppm=tok) if tok else {}))
    modes = np.stack([np.stack([(np.arange(hkv) + 2 * (s + b)) % 3 for b in range(w.n_blocks)])
                      for s in range(w.batch)]).astype(np.uint8)
    cache, data = _cache(w, modes)
    dm, chunks = cache.dims, -(-cache.max_seq_len // 512)
    small, full = w.batch * hkv * chunks, w.batch * hkv * (LONG // 512)
    assert small <= 192 < full
    scale = 1.0 / math.sqrt(d)
    qs = gen.decode_queries(w, 0, scale=8.0)
    for layer in (0, w.n_layers - 1):
        q = to_device(qs[layer], dtype)

        def decode(ws, bound=cache.max_seq_len):
            out = torch.full_like(q, 7.0)
            B.decode_attn(dm, w.batch, cache.seq_lens, bound, cache.modes, cache.offsets, cache.buf, layer, q, out, scale, ws)
            return out

        one = decode(_nan(_records(dm, small)))
        roomy = decode(_nan(4 * _records(dm, small)))
        long = decode(_nan(B.decode_workspace(dm, w.batch, LONG)), LONG)
        ws, two = _nan(_records(dm, small)), torch.full_like(q, 7.0)
        B.decode_partial(dm, w.batch, cache.seq_lens, cache.max_seq_len, cache.modes, cache.offsets, cache.buf,
                         layer, q, scale, ws)
        B.decode_combine(dm, w.batch, chunks, two, ws)
        for name, other in (("four records a chunk", roomy), ("two phases", two),
                            ("the cache's own workspace", cache.decode(layer, q))):
            assert torch.equal(one, other), (name, layer)
        if dtype == "f32":
            assert float((one - long).norm() / one.norm()) <= REORDERED, layer
        else:
            assert torch.equal(one, long), layer
        for s, T in enumerate(lens):
            mode = torch.zeros(-(-w.n_blocks * hkv // 4) * 4, dtype=torch.uint8, device="cuda")
            mode[: w.n_blocks * hkv] = cache.modes[s].flatten()
            alone = torch.full_like(q[s], 7.0)
            B.decode_attn(dm, 1, cache.seq_lens[s:s + 1], T, mode, cache.offsets[s], cache.buf, layer, q[s].contiguous(),
                          alone, scale, _nan(B.decode_workspace(dm, 1, T)))
            assert torch.equal(one[s], alone), (T, layer)
        outs = [x.float().cpu().numpy() for x in (one, long)]
        for s, T in enumerate(lens):
            if T == 0:
                assert all(np.all(out[s] == 0.0) for out in outs)
                continue
            if tok:
                assert all(np.all(np.isfinite(out[s])) for out in outs)  # values: the parity cases of token-level sets
                continue
            one_w, K, V = data[s]
            units = {(b, h): O.compress_unit(K[f:f + nb, h], V[f:f + nb, h], int(modes[s, b, h]), w.topk, dtype)
                     for b, (f, nb) in enumerate(w.blocks) for h in range(hkv)}
            want = oracle_decode_layer(units, modes[s], layer, qs[layer][s].astype(np.float64), one_w)
            for hq in range(w.n_q_heads):
                for out in outs:
                    assert rel_l2(out[s, hq], want[hq]) <= (1e-5 if dtype == "f32" else 1e-2), (T, layer, hq)


@pytest.mark.parametrize("T", [12288, 12289])
def test_the_two_sides_of_the_small_call_rule(T):
    """8 KV heads: 24 chunks a head are the last small call; both sides against exact attention over
    exact heads (every unit exact, so that the reference is plain softmax attention in float64)."""
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import CompressedCache
    for dtype, tol in (("f32", 1e-5), ("bf16", 1e-2)):
        tdt = torch.float32 if dtype == "f32" else torch.bfloat16
        dm = B.dims(2, 8, 32, 128, 16, dtype)
        g = torch.Generator("cuda").manual_seed(T)
        k, v = ([torch.randn(8, T, 128, generator=g, device="cuda").to(tdt) for _ in range(2)] for _ in range(2))
        cache = CompressedCache(dm, [T], np.full((1, 1, 8), 2, np.uint8))
        cache.compress(0, k, v)
        q = torch.randn(1, 32, 128, generator=g, device="cuda").to(tdt)
        out = cache.decode(1, q).double().view(8, 4, 128)
        p = torch.softmax(torch.bmm(k[1].double(), q.double().view(8, 4, 128).transpose(1, 2).contiguous()) / math.sqrt(128), 1)
        want = torch.bmm(p.transpose(1, 2).contiguous(), v[1].double())
        # bf16: probabilities and outputs 2^-9 each, relative to the weighted magnitude of V; fp32: the parity bar
        assert float((out - want).norm() / want.norm()) <= tol


@pytest.mark.parametrize("d,dtype,schedule,G", [(128, "bf16", 0, 4), (128, "bf16_e4m3", 2, 8), (64, "bf16", 0, 1),
                                                (64, "bf16_e4m3", 0, 2), (128, "f32", 2, 2), (64, "f32", 0, 8)])
def test_spans_and_a_tail_give_the_same_bits_in_every_call(d, dtype, schedule, G):
    """Two sequences cut into four spans, the second one without a tail row: the same bits (fp32: up to
    the order of sums) with one and with four records a chunk and with a longer bound on the last span
    (more than 192 chunks; only tail rows come after it); and, where there are no tail rows, what one
    cache of all the tokens gives (which the other cases hold to the oracle), up to the rounding of
    probabilities against other reference maxima."""
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import CompressedCache
    hkv, tdt = 3, torch.float32 if dtype == "f32" else torch.bfloat16
    n = 4 if schedule == 2 else 2
    dm = B.dims(n, hkv, hkv * G, d, d // 8, dtype, schedule)
    g = torch.Generator("cuda").manual_seed(d + G)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(tdt)
    cuts = (700, 512, 1, 130)
    T = sum(cuts)
    modes = np.array([[[0, 1, 2]], [[1, 2, 0]]], np.uint8)
    whole = CompressedCache(dm, [T, T], modes)
    spans = [CompressedCache(dm, [t, t], modes) for t in cuts]
    for s in range(2):
        k, v = ([rnd(hkv, T, d) for _ in range(n)] for _ in range(2))
        whole.compress(s, k, v)
        at = 0
        for c, t in zip(spans, cuts):
            c.compress(s, *([x[:, at:at + t].contiguous() for x in y] for y in (k, v)))
            at += t
    tk, tv = rnd(2, hkv, 200, d), rnd(2, hkv, 200, d)
    lens = torch.tensor([77, 0], dtype=torch.int32, device="cuda")
    tail = B.Tail(int(lens.data_ptr()), 200, int(tk.data_ptr()), int(tv.data_ptr()))
    q, scale = rnd(2, hkv * G, d), 1.0 / math.sqrt(d)

    def decode(room, with_tail, bound=None):
        bounds = [*cuts[:-1], bound or cuts[-1]]
        desc = [B.Span(int(c.seq_lens.data_ptr()), m, int(c.modes.data_ptr()), int(c.offsets.data_ptr()),
                       int(c.buf.data_ptr())) for c, m in zip(spans, bounds)]
        chunks = 2 * hkv * (sum(-(-m // 512) for m in bounds) + with_tail)
        assert (chunks <= 192) == (bound is None)
        out = torch.full_like(q, 7.0)
        B.decode_spans(dm, 2, desc, tail if with_tail else None, n - 1, q, out, scale, _nan(room * _records(dm, chunks)))
        return out

    for with_tail in (0, 1):
        one = decode(1, with_tail)
        assert torch.isfinite(one).all()
        same = lambda x, y: float((x - y).norm() / x.norm()) <= REORDERED if dtype == "f32" else torch.equal(x, y)
        assert same(one, decode(4, with_tail)), with_tail
        long = decode(1, with_tail, LONG)
        want = whole.decode(n - 1, q)
        for s in range(2) if not with_tail else (1,):
            assert same(one[s], long[s]), (with_tail, s)
            rel = float((one[s].double() - want[s].double()).norm() / want[s].double().norm())
            assert rel <= (1e-5 if dtype == "f32" else 1e-2), (with_tail, s, rel)
