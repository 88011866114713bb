"""Decode over residual heads whose entries per row are fewer or more than the
lanes that hold a row (16 at 128 channels, 8 at 64; blocks of four: of 3d
coefficients), at the edges of what travels ahead of a tile (one and two
entries a lane), whatever the workspace and the bound on the lengths, against the oracle's decode."""
import math

import numpy as np
import pytest

import oracle as O
from synth import WORKLOADS, gen, scaled

from gpu_cases import oracle_decode_layer, rel_l2
from test_gpu_launch_shapes import _cache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,dtype,schedule,G", [(128, "bf16", 0, 4), (64, "bf16", 0, 2), (128, "bf16_e4m3", 0, 8),
                                                (128, "bf16", 2, 1), (64, "bf16_e4m3", 2, 4)])
@pytest.mark.parametrize("lanes,more", [(0, 1), (1, -1), (1, 0), (1, 1), (2, -1), (2, 0), (2, 1), (3, 1)])
def test_entries_per_row_at_the_edges_of_the_lanes(d, dtype, schedule, G, lanes, more):
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import to_device
    k = lanes * d // 8 + more
    lens = (1, 9, 130, 515, 1030)
    w = scaled(WORKLOADS["prefill8b"], n_layers=4, n_kv_heads=3, n_q_heads=3 * G, head_dim=d, dtype=dtype, topk=k,
               schedule=schedule, seq_lens=lens, n_needles=1, n_probe=8)
    modes = np.stack([np.stack([np.roll([1, 1, 0], s + b) for b in range(w.n_blocks)]) for s in range(w.batch)]).astype(np.uint8)
    cache, data = _cache(w, modes)
    need = B.decode_workspace(cache.dims, w.batch, cache.max_seq_len)
    scale = 1.0 / math.sqrt(d)
    qs = gen.decode_queries(w, 0, scale=8.0)
    for layer in (0, w.n_layers - 1):
        q = to_device(qs[layer], dtype)
        got = [torch.full_like(q, 7.0) for _ in range(3)]
        for out, room in zip(got, (1, 4)):      # a record per chunk, and room for more
            B.decode_attn(cache.dims, w.batch, cache.seq_lens, cache.max_seq_len, cache.modes, cache.offsets, cache.buf,
                          layer, q, out, scale, torch.full((room * need // 4,), float("nan"), device="cuda"))
        assert torch.equal(got[0], got[1]), layer
        # a longer bound on the lengths: more than 192 chunks
        big = torch.full((B.decode_workspace(cache.dims, w.batch, 65 * 512) // 4,), float("nan"), device="cuda")
        B.decode_attn(cache.dims, w.batch, cache.seq_lens, 65 * 512, cache.modes, cache.offsets, cache.buf,
                      layer, q, got[2], scale, big)
        assert torch.equal(got[0], got[2]), layer
        for out in (x.float().cpu().numpy() for x in (got[0], got[2])):
            for s in range(w.batch):
                one, K, V = data[s]
                units = {(b, h): O.compress_unit(K[f:f + nb, h], V[f:f + nb, h], int(modes[s, b, h]), w.topk, dtype)
                         for b, (f, nb) in enumerate(w.blocks) for h in range(3)}
                want = oracle_decode_layer(units, modes[s], layer, qs[layer][s].astype(np.float64), one)
                for hq in range(w.n_q_heads):
                    assert rel_l2(out[s, hq], want[hq]) <= 1e-2, (k, lens[s], layer, hq)
