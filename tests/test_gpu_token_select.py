"""The selection of token-level sets at the edges of what a workgroup holds of a
unit's scores (32768), of the waves' runs of 128-token chunks and of the radix
digits: spread scores, scores that share their upper digits, ties in bulk, zeros
and infinities.  The set written by compress equals the oracle's (the highest
scores, ties to the lower token), and so do the running counts."""
import numpy as np
import pytest

import oracle as O

from test_gpu_tokres import unpack_tok_unit

pytestmark = pytest.mark.gpu

KINDS = 6


def _scores(rng, T, kind):
    if kind == 0:      # ordinary: a few octaves
        s = np.abs(rng.standard_normal(T))
    elif kind == 1:    # every octave
        s = np.ldexp(1 + rng.random(T), rng.integers(-120, 120, T))
    elif kind == 2:    # alike but for the last digit
        s = 1.0 + rng.integers(0, 256, T) * 2.0 ** -23
    elif kind == 3:    # ties in bulk
        s = rng.integers(0, 3, T).astype(np.float64)
    elif kind == 4:    # all equal
        s = np.full(T, 0.75)
    else:              # zeros, and infinities (a logit past the type's range)
        s = np.where(rng.random(T) < 0.02, np.inf, 0.0)
    return s.astype(np.float32)


@pytest.mark.parametrize("T", [1, 65, 500, 2049, 16385, 32767, 32768, 32769, 33281, 70001])
def test_sets_at_the_edges_of_runs_and_digits(T):
    import torch
    from paper_2607_06519_amd import binding as B
    from paper_2607_06519_amd.cache import CompressedCache
    rng, d = np.random.default_rng(T), 64
    s = np.stack([_scores(rng, T, i) for i in range(KINDS)])
    scores = torch.from_numpy(s[None].copy()).cuda()
    x = [torch.zeros(KINDS, T, d, dtype=torch.bfloat16, device="cuda") for _ in (0, 1)]
    for ppm in (1, 50000, 500000, 1000000):
        dm = B.dims(2, KINDS, KINDS, d, 0, "bf16", 0, B.RES_TOKENS, ppm)
        cache = CompressedCache(dm, [T], np.full((1, 1, KINDS), O.RESIDUAL, np.uint8))
        cache.compress(0, x, x, token_scores=scores)
        torch.cuda.synchronize()
        buf, n = cache.host_bytes(), O.n_residual_tokens(T, ppm)
        for h in range(KINDS):
            got, counts = unpack_tok_unit(buf, int(cache.offsets_host[0, 0, h]), O.RESIDUAL, T, d, ppm, "bf16", 2)
            want = O.residual_tokens(s[h], n)
            np.testing.assert_array_equal(got["TS"], want, err_msg=str((T, ppm, h)))
            np.testing.assert_array_equal(counts[:-1], np.searchsorted(want, np.arange(0, T, 128)))
            assert counts[-1] == n
