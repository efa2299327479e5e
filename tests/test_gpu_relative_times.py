"""Inputs that take a kernel off its usual path, against inputs of the same size that do not: the ratio of the two times on one
box, the fastest of many calls each, so that neither the box nor a neighbour matters.  The bounds lie midway between what the
paths measured when they were slow and what they measure now; outputs are compared with the oracle's."""
import time

import numpy as np
import pytest
import torch

from oracle import lc_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def lc():
    from paper_2009_13003_amd import lc as mod
    return mod


def best_us(call, reps=60):
    for _ in range(10):
        call()
    best = 1e9
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        call()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    return 1e6 * best


def in_binades(e, seed, dtype=torch.float32):
    """A vector with |w| in the binade 2^(e - 30) where e > 0, 0 elsewhere, against zeros."""
    g = torch.Generator(device=DEV); g.manual_seed(seed)
    d = torch.exp2(e - 30) * (1 + 0.5 * torch.rand(e.numel(), generator=g, device=DEV))
    w = torch.where(e > 0, d, torch.zeros_like(e)).to(dtype)
    return w, torch.zeros_like(w)


def blob_of(lc, w, ref, nbits):
    out = lc.alloc_out(w.numel(), nbits, DEV)
    return out[:lc.lc_encode_t(w, ref, nbits, out)].clone()


def code_lengths(blob):
    h = blob[:512].cpu().numpy()
    return h[66:66 + 16 * (int(h[20]) + 1):16].tolist()


def restored_as_the_oracle(lc, blob, n):
    want, got = np.zeros(n, np.float32), torch.zeros(n, device=DEV)
    orc.decode(blob.cpu().numpy(), want)
    lc.lc_decode(blob, got)
    return np.array_equal(got.cpu().numpy().view(np.uint32), want.view(np.uint32))


def test_codes_longer_than_the_look_up(lc):
    """The first chunk holds 8 rare symbols in 0.4 of its places, the others none of them: their codes have 11 bits behind 2^21
    elements and 9 behind 2^18.  The restore takes as long as that chunk's wavefront, so the two differ by the second
    look-up of the longer codes alone."""
    times = {}
    for n, bits in ((1 << 18, 9), (1 << 21, 11)):
        g = torch.Generator(device=DEV); g.manual_seed(n)
        i = torch.arange(n, device=DEV)
        k = torch.floor(-torch.log2(torch.rand(n, generator=g, device=DEV).clamp_(min=2.0 ** -20)))
        common = torch.where((k > 0) & (k < 8), 8 - k, torch.zeros_like(k))
        rare = torch.randint(8, 16, (n,), generator=g, device=DEV).float() * (torch.rand(n, generator=g, device=DEV) < 0.4)
        blob = blob_of(lc, *in_binades(torch.where(i < 16384, rare, common), n), 4)
        assert sorted(code_lengths(blob))[-8:] == [bits] * 8, code_lengths(blob)
        assert restored_as_the_oracle(lc, blob, n)
        rec = torch.zeros(n, device=DEV)
        times[bits] = best_us(lambda: lc.lc_decode(blob, rec))
    print("restore with 9-bit and 11-bit codes: %.1f us, %.1f us" % (times[9], times[11]), flush=True)
    assert times[11] < 2.5 * times[9], times             # (5.2 with a search through the symbols, 1.5 with a table)


def test_few_kept_symbols_spread_over_most_rows(lc):
    """Laplace updates of one scale: with 2 promotion bits about one element in a hundred is kept, with 3 most chunks are full
    of kept symbols.  The first take no longer to restore, although hardly a row is free of them."""
    n, times = 1 << 20, {}
    g = torch.Generator(device=DEV); g.manual_seed(11)
    ref = 0.05 * torch.randn(n, generator=g, device=DEV)
    u = torch.rand(n, generator=g, device=DEV) - 0.5
    w = ref - 1e-3 * torch.sign(u) * torch.log1p(-2 * u.abs().clamp_(max=0.49999997))
    for nbits in (2, 3):
        blob = blob_of(lc, w, ref, nbits)
        assert restored_as_the_oracle(lc, blob, n)
        rec = ref.clone()
        times[nbits] = best_us(lambda: lc.lc_decode(blob, rec))
    print("restore with 2 and 3 bits: %.1f us, %.1f us" % (times[2], times[3]), flush=True)
    assert times[2] < 1.2 * times[3], times               # (1.7 with rows looked up symbol by symbol, 0.8 without)


def test_encode_of_a_chunk_of_long_codes(lc):
    """One chunk of 256 whose codes are too long for the areas that a workgroup codes into at first, as a layer above the others'
    scale has them, against the same vector without it."""
    n, times = 1 << 22, {}
    g = torch.Generator(device=DEV); g.manual_seed(5)
    i = torch.arange(n, device=DEV)
    k = torch.floor(-torch.log2(torch.rand(n, generator=g, device=DEV).clamp_(min=2.0 ** -20)))
    common = torch.where((k > 0) & (k < 8), 8 - k, torch.zeros_like(k))
    rare = torch.randint(8, 16, (n,), generator=g, device=DEV).float() * (torch.rand(n, generator=g, device=DEV) < 0.7)
    for kind, where in (("long", i < 16384), ("spread", i % 256 == 0)):      # as many rare symbols, in one chunk or over all
        w, ref = in_binades(torch.where(where, rare, common), 5)
        out = lc.alloc_out(n, 4, DEV)
        size = lc.lc_encode(w, ref, 4, out)
        assert np.array_equal(out[:size].cpu().numpy(), orc.encode(w.cpu().numpy(), ref.cpu().numpy(), 4))
        times[kind] = best_us(lambda: lc.lc_encode(w, ref, 4, out))
    print("encode with a long chunk and without: %.1f us, %.1f us" % (times["long"], times["spread"]), flush=True)
    assert times["long"] < 1.6 * times["spread"], times    # (2.1 when one wavefront coded such a chunk again, 1.1 now)


def test_encode_of_chunks_with_few_parts_to_read(lc):
    """A vector short enough to go without a list of chunks, of whose 16 parts of 4 KiB per chunk one holds kept elements: the second
    sweep reads that one, and the call takes well less than one that has to read every part."""
    n, times = 1 << 24, {}
    g = torch.Generator(device=DEV); g.manual_seed(6)
    i = torch.arange(n, device=DEV)
    e = torch.randint(1, 8, (n,), generator=g, device=DEV).float()
    for kind, where in (("one", (i // 1024) % 16 == 5), ("all", i % 16 == 5)):
        w, ref = in_binades(torch.where(where, e, torch.zeros_like(e)), 6)
        out = lc.alloc_out(n, 3, DEV)
        size = lc.lc_encode(w, ref, 3, out)
        assert np.array_equal(out[:size].cpu().numpy(), orc.encode(w.cpu().numpy(), ref.cpu().numpy(), 3))
        times[kind] = best_us(lambda: lc.lc_encode(w, ref, 3, out))
    print("encode with one part in 16 and with all: %.1f us, %.1f us" % (times["one"], times["all"]), flush=True)
    assert times["one"] < 0.92 * times["all"], times         # (0.99 when all parts were read, 0.85 now)


def test_encode_of_halves_between_dwords(lc):
    """An unchanged bf16 vector of 3,000 chunks that starts between two dwords, against one that starts on a dword off alignment."""
    n, times = 3000 * 16384, {}
    buf, out = torch.zeros(2, n + 64, device=DEV, dtype=torch.bfloat16), lc.alloc_out(n, 3, DEV)
    for offset in (1, 2):
        w, ref = buf[0, offset:offset + n], buf[1, offset:offset + n]
        size = lc.lc_encode_t(w, ref, 3, out)
        if offset == 1:
            want = out[:size].clone()
        assert torch.equal(out[:size], want)
        times[offset] = best_us(lambda: lc.lc_encode_t(w, ref, 3, out))
    print("encode off dwords and on them: %.1f us, %.1f us" % (times[1], times[2]), flush=True)
    assert times[1] < 1.1 * times[2], times               # (1.19 by vectors)


def test_long_lists_of_sparse_updates(lc):
    """Five checkpoints of 2^27 elements in one call, none changed, or with a few heavy tails in a tenth of their chunks, against
    four, which another kernel restores: a blob more costs no more than its share."""
    n = 1 << 27
    g = torch.Generator(device=DEV); g.manual_seed(9)
    for kind, slow, now in (("unchanged", 1.47, 0.87), ("heavy tails", 1.42, 1.09)):
        d = torch.zeros(n, device=DEV)
        if kind == "heavy tails":
            for _ in range(3):
                d += torch.randn(n, generator=g, device=DEV) ** 2
            d = 1e-4 * torch.randn(n, generator=g, device=DEV) / torch.sqrt(d / 3 + 1e-30) * (torch.rand(n, generator=g, device=DEV) >= 0.1)
        blob, times, single, many = blob_of(lc, d, torch.zeros_like(d), 3), {}, torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
        blobs = [blob.clone() for _ in range(5)]
        for b in blobs:
            lc.lc_decode(b, single)
        lc.lc_decode_many(blobs, many)
        assert torch.equal(single, many)
        for count in (4, 5):
            times[count] = best_us(lambda: lc.lc_decode_many(blobs[:count], many), reps=30)
        print("%s, 4 and 5 blobs: %.1f us, %.1f us" % (kind, times[4], times[5]), flush=True)
        assert times[5] < 0.5 * (slow + now) * times[4], (kind, times)


@pytest.mark.parametrize("chunks,ragged,count,bound", [(3, 3 * 16384 - 777, 8, 1.2),           # (1.44 by elements, 1.0 by rows)
                                                       (4, 3 * 16384 + 4460, 7, 1.05)])        # (1.15 by payloads from memory, 0.95)
def test_short_lists_that_end_in_a_ragged_chunk(lc, chunks, ragged, count, bound):
    """A few chunks' checkpoints in one call, the last chunk whole or ragged: that one is a wavefront's work from start to end, as the others
    are, and does not keep their payloads out of the LDS."""
    times = {}
    for n in (chunks * 16384, ragged):
        g = torch.Generator(device=DEV); g.manual_seed(13)
        u = torch.rand(n, generator=g, device=DEV) - 0.5
        d = -1e-3 * torch.sign(u) * torch.log1p(-2 * u.abs().clamp_(max=0.49999997))
        blob, many, single = blob_of(lc, d, torch.zeros_like(d), 3), torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
        blobs = [blob.clone() for _ in range(count)]
        for b in blobs:
            lc.lc_decode(b, single)
        lc.lc_decode_many(blobs, many)
        assert torch.equal(single, many)
        times[n] = best_us(lambda: lc.lc_decode_many(blobs, many))
    print("%d blobs, whole and ragged: %.1f us, %.1f us" % (count, times[chunks * 16384], times[ragged]), flush=True)
    assert times[ragged] < bound * times[chunks * 16384], times


def test_lists_whose_dense_chunks_lie_together(lc):
    """Four checkpoints of 2^27 elements off alignment, of which three layers out of eleven change: their chunks come one after the other to
    the workgroups, and each wavefront of those takes one when it is free.  Against checkpoints that change everywhere."""
    n, times = 1 << 27, {}
    g = torch.Generator(device=DEV); g.manual_seed(15)
    for kind in ("dense", "layers"):
        u = torch.rand(n, generator=g, device=DEV) - 0.5
        d = -1e-3 * torch.sign(u) * torch.log1p(-2 * u.abs().clamp_(max=0.49999997))
        if kind == "layers":
            d *= 10.0 ** -((torch.arange(n, device=DEV) * 11 // n) * 3 % 4).float()
        blob, many, single = blob_of(lc, d, torch.zeros_like(d), 3), torch.zeros(n + 1, device=DEV)[1:], torch.zeros(n, device=DEV)
        blobs = [blob.clone() for _ in range(4)]
        for b in blobs:
            lc.lc_decode(b, single)
        lc.lc_decode_many(blobs, many)
        assert torch.equal(single, many)
        times[kind] = best_us(lambda: lc.lc_decode_many(blobs, many), reps=30)
    print("dense and in layers: %.1f us, %.1f us" % (times["dense"], times["layers"]), flush=True)
    assert times["layers"] < 0.45 * times["dense"], times     # (0.49 where a chunk was taken as the one before it began, 0.41 now)


def test_batch_of_tiny_tensors(lc):
    """A thousand tensors of 64 elements: the counting sweep has a workgroup for each, whose empty rows cost nothing."""
    times, batches = {}, {}
    for dtype in (torch.float32, torch.bfloat16):
        ws = [torch.full((64,), 0.5 + i, device=DEV, dtype=dtype) for i in range(1000)]
        refs, outs = [torch.zeros_like(w) for w in ws], [lc.alloc_out(64, 3, DEV) for _ in ws]
        batch = batches[dtype] = lc.EncodeBatch(ws, refs, 3, outs)
        one = lc.alloc_out(64, 3, DEV)
        sizes = batch.run()
        for i in (0, 500, 999):
            assert lc.lc_encode_t(ws[i], refs[i], 3, one) == sizes[i] and torch.equal(one[:sizes[i]], outs[i][:sizes[i]])
    for _ in range(3):                                       # (in turn: the two are a few percent apart)
        for dtype, batch in batches.items():
            times[dtype] = min(times.get(dtype, 1e9), best_us(batch.run))
    print("1,000 tensors, fp32 and bf16: %.1f us, %.1f us" % (times[torch.float32], times[torch.bfloat16]), flush=True)
    assert times[torch.float32] < 1.03 * times[torch.bfloat16], times        # (1.05 where three workgroups fit a compute unit, 1.01 where four do)
