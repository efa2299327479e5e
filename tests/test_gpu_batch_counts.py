"""The counting sweep of lc_encode_batch, a workgroup per chunk or per run of chunks: tensors that end inside a run, runs inside a
tensor, tensors smaller than a row, empty and unchanged ones, one that is not finite, arrays off alignment, one chunk less than the
staying workgroups take and one more.  Against an encode per tensor, byte for byte (integer statistics: no tolerance)."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV, CHUNK = "cuda:0", 16384


@pytest.fixture(scope="module")
def lc():
    from paper_2009_13003_amd import lc as mod
    return mod


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("dtype,chunks", [(torch.float32, 5), (torch.bfloat16, 5), (torch.float16, 40), (torch.float32, 3071), (torch.float32, 3072),
                                          (torch.bfloat16, 6144), (torch.float16, 6143)])
def test_counts(lc, dtype, chunks, offset):
    print("batch counts", dtype, chunks, offset, flush=True)
    g = torch.Generator(device=DEV); g.manual_seed(chunks + offset)
    sizes = [0, 1, 3, 255, 256, 257, CHUNK - 1, CHUNK, CHUNK + 5, 1029]
    left = chunks - sum((m + CHUNK - 1) // CHUNK for m in sizes)
    while left > 0:                                        # large ones between small ones, ragged and whole
        k = min(left, int(torch.randint(1, 700, (1,), generator=g, device=DEV)))
        sizes.insert(len(sizes) // 2, k * CHUNK - (k % 3) * 7)
        left -= k
    ws, refs, outs = [], [], []
    for i, m in enumerate(sizes):
        d = 10.0 ** (i % 5 - 5) * torch.randn(m, generator=g, device=DEV)
        if i % 4 == 1:
            d = d * (torch.rand(m, generator=g, device=DEV) < 0.01)       # chunks and parts that are not read again
        if i % 7 == 6:
            d = torch.zeros(m, device=DEV)
        ref, w = (torch.zeros(m + offset, dtype=dtype, device=DEV) for _ in range(2))
        ref[offset:] = (0.05 * torch.randn(m, generator=g, device=DEV)).to(dtype)
        w[offset:] = (ref[offset:].float() + d).to(dtype)
        if i == 8:
            w[offset + m // 2] = float("inf")
        ws.append(w[offset:]); refs.append(ref[offset:]); outs.append(lc.alloc_out(m, 3, DEV))
    batch = lc.EncodeBatch(ws, refs, 3, outs)
    for turn in range(2):
        for got in outs:
            got.fill_(0xAB)
        got_sizes = batch.run()
        for i, (w, ref, got, size) in enumerate(zip(ws, refs, outs, got_sizes)):
            if not bool(torch.isfinite(w.float()).all()):
                assert size == -lc.ERR_NONFINITE, (i, size)
                continue
            one = lc.alloc_out(w.numel(), 3, DEV)
            assert lc.lc_encode_t(w, ref, 3, one) == size, (i, sizes[i])
            assert torch.equal(one[:size], got[:size]), (i, sizes[i])


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
def test_short_tensors(lc, dtype, offset):
    """The form for chunks of few rows: ends at every edge of rows, parts and wavefronts, whole chunks between them."""
    g = torch.Generator(device=DEV); g.manual_seed(offset)
    sizes = [m + d for m in (1, 64, 256, 512, 1024, 2048, 4096, 6144, 8192, 10240, CHUNK) for d in (-1, 0, 1)] + [0, 2 * CHUNK, CHUNK + 1025] + [300] * 40
    assert sum(sizes) / sum((m + CHUNK - 1) // CHUNK for m in sizes) < CHUNK // 2
    ws, refs, outs = [], [], []
    for i, m in enumerate(sizes):
        d = 10.0 ** (i % 5 - 5) * torch.randn(m, generator=g, device=DEV)
        if i % 3 == 1:
            d = d * (torch.rand(m, generator=g, device=DEV) < 0.01)
        ref, w = (torch.full((m + offset + 1,), float("nan"), dtype=dtype, device=DEV) for _ in range(2))     # (a NaN beside would show)
        ref[offset:offset + m] = (0.05 * torch.randn(m, generator=g, device=DEV)).to(dtype)
        w[offset:offset + m] = (ref[offset:offset + m].float() + d).to(dtype)
        if i == 20:
            w[offset + m // 2] = float("inf")
        ws.append(w[offset:offset + m]); refs.append(ref[offset:offset + m]); outs.append(lc.alloc_out(m, 3, DEV))
    sizes_got = lc.EncodeBatch(ws, refs, 3, outs).run()
    for i, (w, ref, got, size) in enumerate(zip(ws, refs, outs, sizes_got)):
        if i == 20:
            assert size == -lc.ERR_NONFINITE, (i, size)
            continue
        one = lc.alloc_out(w.numel(), 3, DEV)
        assert lc.lc_encode_t(w, ref, 3, one) == size, (i, sizes[i])
        assert torch.equal(one[:size], got[:size]), (i, sizes[i])
