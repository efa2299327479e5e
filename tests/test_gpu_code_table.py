"""The table of a blob from given populations of the buckets: the deepest trees, ties of every kind, one symbol, none kept, all
kept, and kept sets that pass over the smallest exponents; binary32 and binary64, one vector, a batch and a cached call.
Against the oracle's blobs byte for byte."""
import numpy as np
import pytest
import torch

from oracle import lc_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

FIB = [1, 1, 2, 3, 5, 8, 13, 21, 34, 55, 89, 144, 233, 377, 610, 987]
# populations of the buckets in order of priority (+ before - at equal exponent), the last: elements that stay unchanged
POPULATIONS = {
    "deepest": FIB, "deepest, other way round": FIB[::-1], "deepest from the middle": FIB[8:] + FIB[:8],
    "all equal": [7] * 16, "all ones": [1] * 16, "powers": [2 ** k for k in range(12)], "pairs": [1, 1, 2, 2, 4, 4, 8, 8, 16, 16, 32, 32, 64, 64, 128, 128],
    "leaf against node": [3, 3, 6, 6, 12, 12, 24], "one kept": [5000, 0], "one and the rest": [1, 20000], "rest only": [0, 300],
    "nothing merged": FIB + [0], "signs apart": [0, 5, 0, 4, 0, 3, 3, 0, 9], "more than fit": list(range(1, 60)), "nine": [9, 9, 9, 9, 9, 9, 9, 9, 9],
}


def vector(pop, dtype, seed):
    vals = []
    for k, c in enumerate(pop[:-1]):
        # larger exponent first, down through the types' whole ranges where there are many
        e = (100 if dtype == np.float32 else 900) - (k // 2) * (1 if len(pop) < 40 else 3)
        vals.append(np.full(c, (-1.0 if k % 2 else 1.0) * 2.0 ** e) * (1 + np.arange(c) / (2.0 * max(c, 1))))
    vals.append(np.zeros(pop[-1]))
    x = np.concatenate(vals).astype(dtype)
    return x[np.random.RandomState(seed).permutation(x.size)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("name", sorted(POPULATIONS))
def test_table_of_given_populations(name, dtype):
    from paper_2009_13003_amd import lc
    print("table", name, dtype, flush=True)
    w_h = vector(POPULATIONS[name], dtype, len(name))
    w = torch.from_numpy(w_h).to(DEV)
    ref_h, ref = np.zeros_like(w_h), torch.zeros_like(w)
    plain, cached = (orc.encode, orc.encode_cached) if dtype == np.float32 else (orc.encode64, orc.encode_cached64)
    for nbits in (1, 2, 3, 4):
        want = plain(w_h, ref_h, nbits)
        out = lc.alloc_out(w.numel(), nbits, DEV)
        size = lc.lc_encode_t(w, ref, nbits, out)
        assert np.array_equal(out[:size].cpu().numpy(), want), (name, nbits)
        outs = [lc.alloc_out(w.numel(), nbits, DEV) for _ in range(2)]
        sizes = lc.lc_encode_batch([w, w[:1]], [ref, ref[:1]], nbits, outs)
        assert np.array_equal(outs[0][:sizes[0]].cpu().numpy(), want), (name, nbits, "batch")
        cache, cache_h = lc.new_cache(DEV), orc.new_cache()
        for turn in range(2):                              # the second call finds this very table in the cache
            size, used = lc.lc_encode_cached_t(w, ref, nbits, out, cache)
            want, used_h = cached(w_h, ref_h, nbits, cache_h)
            assert used == used_h and np.array_equal(out[:size].cpu().numpy(), want), (name, nbits, turn)
