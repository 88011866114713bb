"""The wavefront top-k (csrc/rowtopk.h) at the edges of its search: rows whose
magnitudes span many octaves (past the 255 prefix steps), rows of equal or zero
keys, prefixes shared by many keys that differ in their low bits, single
outliers, and k at the edges of its lower bounds (one, two and four groups a
lane), in every layout that pairs take.  The selections written by compress
equal the oracle's, and those taken from the probe give the same cache."""
import numpy as np
import pytest

import oracle as O

from gpu_cases import TYPES, BYTES, coef_plane_bytes

pytestmark = pytest.mark.gpu


def _rows(rng, T, d, f32):
    """Layer differences of T rows, as (x0, x1) with x0 - x1 exact in fp32."""
    kinds = 9
    out = np.zeros((T, d), np.float32)
    for t in range(T):
        kind, s = t % kinds, rng.choice([-1.0, 1.0], size=d)
        if kind == 0:      # ordinary
            v = rng.standard_normal(d)
        elif kind == 1:    # every octave from 2^-40 to 2^20
            v = np.ldexp(1 + rng.integers(0, 128, d) / 128, rng.integers(-40, 20, d))
        elif kind == 2:    # all equal
            v = np.full(d, 1.5)
        elif kind == 3:    # zeros, and a few values
            v = np.zeros(d)
            v[rng.choice(d, size=int(rng.integers(0, 5)), replace=False)] = 1.0
        elif kind == 4:    # two values
            v = np.where(rng.random(d) < 0.2, 2.0, 1.0)
        elif kind == 5:    # one prefix, unlike low bits (fp32); ties in bf16
            v = 1.0 + rng.integers(0, 1 << 16, d) * 2.0 ** -23
        elif kind == 6:    # most keys small, outliers two to eight octaves up
            v = rng.standard_normal(d) * 0.01
            v[rng.choice(d, size=d // 4, replace=False)] = np.ldexp(1.0, rng.integers(2, 9, d // 4))
        elif kind == 7:    # ascending, so that the k-th key sits at a lane's edge
            v = 1.0 + np.arange(d) / 64
        else:              # few distinct values
            v = rng.integers(0, 4, d) * 0.25
        out[t] = (v * s).astype(np.float32)
    x0 = out if f32 else O.round_bf16(out.astype(np.float64)).astype(np.float32)
    return x0, np.zeros_like(x0)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64), ("bf16_e4m3", 128)])
def test_selection_at_the_edges_of_the_search(dtype, d):
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import CompressedCache, probe, to_device
    T, rng = 9 * 15, np.random.default_rng(d)
    xs = [_rows(rng, T, d, dtype == "f32") for _ in range(4)]     # two heads of K, two of V
    lay = lambda i: [to_device(np.stack([xs[i][l], xs[i + 1][l]]), dtype) for l in (0, 1)]
    kl, vl = lay(0), lay(2)
    rows = [torch.ones(2, 4, d, device="cuda").to(kl[0].dtype) for _ in (0, 1)]
    c = BYTES[TYPES[dtype][1]]
    for k in (1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64 if d == 128 else 62, d - 1):
        dm = B.dims(2, 2, 2, d, k, dtype)
        got = []
        for reuse in (False, True):
            cache = CompressedCache(dm, [T], np.full((1, 1, 2), 1, np.uint8))
            cache.buf.zero_()
            cache.compress(0, kl, vl, k_select=probe(dm, T, kl, rows, 4)[1] if reuse else None)
            got.append(cache.host_bytes().copy())
        assert np.array_equal(got[0], got[1]), k
        pad = lambda n: -(-n // 256) * 256
        for h in range(2):
            o = int(cache.offsets_host[0, 0, h]) + 2 * coef_plane_bytes(T, d, c)
            for x in (xs[h], xs[2 + h]):
                idx = got[0][o: o + T * k].reshape(T, k)
                want = O.residual_channels(x[0].astype(np.float64), x[1].astype(np.float64), k)
                np.testing.assert_array_equal(idx, want, err_msg=f"k={k} head {h}")
                o += pad(T * k) + pad(T * k * c)
