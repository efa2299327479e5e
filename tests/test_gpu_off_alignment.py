"""Encodes of arrays aligned to their elements only, which take the same vector loads as aligned ones: full chunks, ragged ends, parts and
chunks that are not read again, lists of the chunks left to code, either array alone off alignment; plain, cached and binary64.
Against the blob of the same elements in aligned arrays, byte for byte (integer statistics: no tolerance)."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV, CHUNK = "cuda:0", 16384


@pytest.fixture(scope="module")
def lc():
    from paper_2009_13003_amd import lc as mod
    return mod


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16, torch.float64])
@pytest.mark.parametrize("n", [5, 1023, 1024 * 9 + 3, CHUNK, 600 * CHUNK, 600 * CHUNK + 7 * 1024 + 1, 1600 * CHUNK - 1])
def test_same_blob(lc, dtype, n):
    print("off alignment", dtype, n, flush=True)
    g = torch.Generator(device=DEV); g.manual_seed(n % 1009)
    ref = (0.05 * torch.randn(n, generator=g, device=DEV)).to(dtype)
    some = torch.rand(n, generator=g, device=DEV)
    dense = 1e-3 * torch.randn(n, generator=g, device=DEV)
    updates = [dense, dense * (some < 0.3) * 10.0 ** (-6 * some),
               dense * (torch.arange(n, device=DEV) % (3 * CHUNK) < 1500)]                  # parts, and whole chunks, of zeros
    for d in updates:
        w = (ref.to(torch.float64) + d).to(dtype)
        want = lc.alloc_out(n, 3, DEV); size = lc.lc_encode_t(w, ref, 3, want)
        caches = [lc.new_cache(DEV) for _ in range(2)]
        for k, (off, off_ref) in enumerate([(1, 1), (0, 1), (3, 0)] if n < 100 * CHUNK else [(1, 1), (0, 3)]):
            bw, br = (torch.full((n + 4,), float("nan"), dtype=dtype, device=DEV) for _ in range(2))
            bw[off:off + n] = w; br[off_ref:off_ref + n] = ref                              # (a NaN outside would show)
            bw, br = bw[off:off + n], br[off_ref:off_ref + n]
            got = lc.alloc_out(n, 3, DEV)
            assert lc.lc_encode_t(bw, br, 3, got) == size and torch.equal(got[:size], want[:size]), (off, off_ref)
            if dtype != torch.float64 and k == 0:
                want2 = torch.empty_like(want)
                for turn in range(3):                                                       # without a table, then by it
                    size2, hit = lc.lc_encode_cached_t(w, ref, 3, want2, caches[0])
                    assert lc.lc_encode_cached_t(bw, br, 3, got, caches[1]) == (size2, hit), turn
                    assert torch.equal(got[:size2], want2[:size2]), turn


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n", [4096 * CHUNK, 4096 * CHUNK + 1029])
def test_same_blob_on_both_sides_of_the_counts_limit(lc, dtype, n):
    """2-byte elements between two dwords: counted element by element up to 4,096 chunks, by vectors beyond."""
    print("between dwords", dtype, n, flush=True)
    g = torch.Generator(device=DEV); g.manual_seed(n % 1009)
    ref = torch.randn(n, generator=g, device=DEV).to(dtype)
    w = (ref.float() + 0.1 * torch.randn(n, generator=g, device=DEV) * (torch.rand(n, generator=g, device=DEV) < 0.2)).to(dtype)
    want = lc.alloc_out(n, 3, DEV); size = lc.lc_encode_t(w, ref, 3, want)
    for off, off_ref in ((1, 1), (0, 3), (1, 2)):
        bw, br = (torch.full((n + 4,), float("nan"), dtype=dtype, device=DEV) for _ in range(2))
        bw[off:off + n] = w; br[off_ref:off_ref + n] = ref
        got = lc.alloc_out(n, 3, DEV)
        assert lc.lc_encode_t(bw[off:off + n], br[off_ref:off_ref + n], 3, got) == size and torch.equal(got[:size], want[:size]), (off, off_ref)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16, torch.float64])
@pytest.mark.parametrize("n", [1023, 600 * CHUNK, 600 * CHUNK + 7 * 1024 + 1, 2100 * CHUNK - 1])
def test_same_restore(lc, dtype, n):
    """Restores, alone and in a batch with a short vector: the bits of the aligned restore, and nothing written beside the array."""
    print("restore off alignment", dtype, n, flush=True)
    g = torch.Generator(device=DEV); g.manual_seed(n % 1009)
    ref = (0.05 * torch.randn(n, generator=g, device=DEV)).to(dtype)
    dense = 1e-3 * torch.randn(n, generator=g, device=DEV)
    layers = dense * 10.0 ** -(torch.arange(n, device=DEV) // CHUNK % 7).float()            # long codes in some chunks
    for nbits, d in ((3, dense), (4, layers), (1, dense * (torch.rand(n, generator=g, device=DEV) < 0.002))):
        w = (ref.to(torch.float64) + d).to(dtype)
        blob = lc.alloc_out(n, nbits, DEV); blob = blob[:lc.lc_encode_t(w, ref, nbits, blob)].contiguous()
        want = ref.clone(); lc.lc_decode_t(blob, want)
        whole = {2: torch.int16, 4: torch.int32, 8: torch.int64}[ref.element_size()]
        for batch in (False, True) if dtype != torch.float64 else (False,):
            for off in (1, 2, 3):
                buf = torch.full((n + 8,), float("nan"), dtype=dtype, device=DEV)
                guard = buf.view(whole)[:1].clone()
                buf[off:off + n] = ref
                if batch:
                    lc.DecodeBatch([blob, blob], [buf[off:off + n], ref.clone()]).run()
                else:
                    lc.lc_decode_t(blob, buf[off:off + n])
                assert torch.equal(buf[off:off + n].view(whole), want.view(whole)), (nbits, off, batch)
                beside = torch.cat([buf.view(whole)[:off], buf.view(whole)[off + n:]])
                assert bool((beside == guard).all()), (nbits, off, batch)
