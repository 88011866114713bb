"""The launch shapes of the split-K decode (csrc/decode_shape.h) at
the edges of their chunks, groups and tiles: the chunks of a small call spread
over workgroups (a workspace with room for a record per group), held in one
workgroup (a workspace of exactly the queried size, and the two-phase call),
and one workgroup of four waves (calls of more than 192 chunks).  The first two
give the same bits; each is held to the oracle by the parity cases, and here
to the oracle's decode at the edges."""
import math

import numpy as np
import pytest

import oracle as O
from synth import WORKLOADS, gen, scaled

from gpu_cases import oracle_decode_layer, rel_l2

pytestmark = pytest.mark.gpu

GROUPS = {"g1": 1, "g2": 2, "g4": 4, "g8": 8}


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


@pytest.mark.parametrize("g", list(GROUPS))
@pytest.mark.parametrize("d,dtype,schedule,tok", [(128, "bf16", 0, 0), (64, "bf16", 0, 0), (128, "bf16_e4m3", 2, 0),
                                                  (64, "bf16_e4m3", 0, 0), (128, "bf16", 2, 200000),
                                                  (64, "bf16", 0, 300000), (128, "f32", 0, 0), (64, "f32", 2, 0),
                                                  (64, "f32", 0, 300000)])
def test_a_spread_chunk_gives_the_bits_of_one_workgroup(g, d, dtype, schedule, tok):
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import to_device
    G = GROUPS[g]
    # below, at and above a tile, a wave's and a group's tokens, a chunk
    lens = (1, 8, 33, 127, 129, 256, 511, 513, 0, 1100)
    w = scaled(WORKLOADS["prefill8b"], n_layers=4, n_kv_heads=3, n_q_heads=3 * G, head_dim=d, dtype=dtype, topk=d // 8,
               schedule=schedule, seq_lens=lens, n_needles=1, n_probe=8, **(dict(residual=1, res_ppm=tok) if tok else {}))
    modes = np.stack([np.stack([np.roll([0, 1, 2], s + b) for b in range(w.n_blocks)]) for s in range(w.batch)]).astype(np.uint8)
    cache, data = _cache(w, modes)
    need = B.decode_workspace(cache.dims, w.batch, cache.max_seq_len)
    assert w.batch * 3 * 3 <= 192 and cache.ws.numel() * 4 >= 4 * need
    scale = 1.0 / math.sqrt(d)
    qs = gen.decode_queries(w, 0, scale=8.0)
    for layer in (0, w.n_layers - 1):
        q = to_device(qs[layer], dtype)
        wide = torch.full((need // 4,), float("nan"), device="cuda")
        got = [torch.full_like(q, 7.0) for _ in range(3)]
        B.decode_attn(cache.dims, w.batch, cache.seq_lens, cache.max_seq_len, cache.modes, cache.offsets, cache.buf,
                      layer, q, got[0], scale, torch.full((need,), float("nan"), device="cuda"))
        B.decode_attn(cache.dims, w.batch, cache.seq_lens, cache.max_seq_len, cache.modes, cache.offsets, cache.buf,
                      layer, q, got[1], scale, wide)
        wide.fill_(float("nan"))
        B.decode_partial(cache.dims, w.batch, cache.seq_lens, cache.max_seq_len, cache.modes, cache.offsets, cache.buf,
                         layer, q, scale, wide)
        B.decode_combine(cache.dims, w.batch, 3, got[2], wide)
        assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2]), layer
        out = got[0].float().cpu().numpy()
        for s, T in enumerate(lens):
            if T == 0:
                assert np.all(out[s] == 0.0)
                continue
            if tok:
                assert np.all(np.isfinite(out[s]))  # the set's values: the parity cases of token-level sets
                continue
            one, K, V = data[s]
            units = {(b, h): O.compress_unit(K[f:f + nb, h], V[f:f + nb, h], int(modes[s, b, h]), w.topk, dtype)
                     for b, (f, nb) in enumerate(w.blocks) for h in range(3)}
            want = oracle_decode_layer(units, modes[s], layer, qs[layer][s].astype(np.float64), one)
            for hq in range(w.n_q_heads):
                assert rel_l2(out[s, hq], want[hq]) <= (1e-5 if dtype == "f32" else 1e-2), (T, layer, hq)


@pytest.mark.parametrize("T", [12288, 12289])
def test_the_two_sides_of_the_small_call_rule(T):
    """8 KV heads: 24 chunks a head are the last small call; both sides against exact attention over
    exact heads (every unit exact, so that the reference is plain softmax attention in float64)."""
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import CompressedCache
    dm = B.dims(2, 8, 32, 128, 16, "bf16")
    g = torch.Generator("cuda").manual_seed(T)
    k, v = ([torch.randn(8, T, 128, generator=g, device="cuda").bfloat16() for _ in range(2)] for _ in range(2))
    cache = CompressedCache(dm, [T], np.full((1, 1, 8), 2, np.uint8))
    cache.compress(0, k, v)
    q = torch.randn(1, 32, 128, generator=g, device="cuda").bfloat16()
    out = cache.decode(1, q).double().view(8, 4, 128)
    p = torch.softmax(torch.bmm(k[1].double(), q.double().view(8, 4, 128).transpose(1, 2).contiguous()) / math.sqrt(128), 1)
    want = torch.bmm(p.transpose(1, 2).contiguous(), v[1].double())
    # probabilities and outputs in bf16: 2^-9 each, relative to the weighted magnitude of V
    assert float((out - want).norm() / want.norm()) <= 1e-2


def test_spans_with_and_without_room_for_the_groups():
    """A call over spans and a tail spreads its chunks only where the workspace holds a record per
    group: both launches agree within the bf16 bar (they split a chunk differently)."""
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import CompressedCache
    dm = B.dims(2, 3, 12, 128, 16, "bf16")
    g = torch.Generator("cuda").manual_seed(7)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    spans = []
    for i, T in enumerate((700, 512, 1, 130)):
        c = CompressedCache(dm, [T, T], np.array([[[0, 1, 2]], [[1, 2, 0]]], np.uint8))
        for s in range(2):
            c.compress(s, [rnd(3, T, 128) for _ in range(2)], [rnd(3, T, 128) for _ in range(2)])
        spans.append(c)
    desc = [B.Span(int(c.seq_lens.data_ptr()), c.max_seq_len, int(c.modes.data_ptr()), int(c.offsets.data_ptr()),
                   int(c.buf.data_ptr())) for c in spans]
    tk, tv = rnd(2, 3, 200, 128), rnd(2, 3, 200, 128)
    lens = torch.tensor([77, 0], dtype=torch.int32, device="cuda")
    need = B.decode_spans_workspace(dm, 2, [c.max_seq_len for c in spans], 200)
    q = rnd(2, 12, 128)
    outs = []
    for n in (need // 4, need):
        out = torch.full_like(q, 7.0)
        B.decode_spans(dm, 2, desc, B.Tail(int(lens.data_ptr()), 200, int(tk.data_ptr()), int(tv.data_ptr())), 1, q, out,
                       1.0 / math.sqrt(128), torch.full((n,), float("nan"), device="cuda"))
        outs.append(out.double())
    assert torch.isfinite(outs[0]).all()
    assert float((outs[0] - outs[1]).norm() / outs[1].norm()) <= 1e-2
