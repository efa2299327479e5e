"""Chunks whose code strings outgrow what a workgroup of the coding sweep holds at first (5 bits per element, 7 in one lane's
part), against the oracle's blobs byte for byte: payloads on both sides of one, two and three windows of 2560 words, up to the
longest there is (15 bits for every element); from the inputs and from staged keys; in a vector and in a batch."""
import numpy as np
import pytest
import torch

from oracle import lc_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CHUNK = 16384
# elements with a code of 15 bits in the first chunks, the others have 1 bit: (16384 + 14 x) / 32 words
RARE = [4681, 4682, 10532, 10533, 16384]                       # 2560, 2561, 5120, 5121, 7680 words


@pytest.fixture(scope="module")
def lc():
    from paper_2009_13003_amd import lc as mod
    return mod


def long_chunks(dtype, tail):
    """Populations that make the code lengths 15, 15, 14, ... 1; the two rarest symbols fill RARE places of the first chunks, dealt
    evenly over the parts that the wavefronts' lanes code; a ragged last chunk holds some as well."""
    g = torch.Generator(device=DEV); g.manual_seed(tail)
    c = (sum(RARE) + tail) // 2 + 1
    counts = [c, c, c + c // 50]
    while len(counts) < 16:
        counts.append(int(1.01 * sum(counts[:-1])) + 1)
    n = (sum(counts) + CHUNK - 1) // CHUNK * CHUNK + tail
    e = torch.zeros(n, device=DEV)                             # binade 16 - rank of the population; 0: the largest, merged
    i = torch.arange(CHUNK, device=DEV)
    row, lane, v = i // 256, (i // 4) % 64, i % 4
    order = torch.argsort((row % 8 * 4 + v) * 512 + (row // 8) * 64 + lane)
    rare = lambda m: 14 + torch.randint(0, 2, (m,), generator=g, device=DEV).float()
    for k, x in enumerate(RARE):
        e[k * CHUNK + order[:x]] = rare(x)
    if tail:
        e[n - tail:] = rare(tail)
    # the rest of every population, anywhere behind the first chunks
    lo, hi = len(RARE) * CHUNK, n - tail
    rest = torch.cat([torch.full((m,), float(15 - k), device=DEV) for k, m in enumerate(counts[:15]) if k >= 2])
    assert rest.numel() < hi - lo
    e[lo + torch.randperm(hi - lo, generator=g, device=DEV)[:rest.numel()]] = rest
    w = torch.where(e > 0, torch.exp2(e - 20) * (1 + 0.5 * torch.rand(n, generator=g, device=DEV)), torch.zeros_like(e)).to(dtype)
    return w, torch.zeros_like(w)


@pytest.mark.parametrize("dtype,tail", [(torch.float32, 0), (torch.float32, 2311), (torch.bfloat16, 4000)])
def test_chunks_of_several_windows(lc, dtype, tail):
    w, ref = long_chunks(dtype, tail)
    n = w.numel()
    print("long chunks", dtype, n, flush=True)
    if dtype == torch.float32:
        want = orc.encode(w.cpu().numpy(), ref.cpu().numpy(), 4)
    else:
        raw = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)
        want = orc.encode_t(raw(w), raw(ref), 4, orc.DT_BF16)
    lens = want[66:66 + 16 * 16:16].tolist()
    assert lens[:2] == [15, 15] and lens[15] == 1, lens
    offs = want[512:512 + 4 * 6].view(np.uint32).astype(int)
    assert (np.diff(offs) - 32).tolist() == [2560, 2561, 5120, 5121, 7680]
    out = lc.alloc_out(n, 4, DEV)
    for staging in ([lc.STAGING_NEVER, lc.STAGING_ALWAYS] if dtype == torch.float32 else [lc.STAGING_AUTO]):
        lc.lc_set_option(lc.OPT_KEY_STAGING, staging)
        try:
            out.fill_(0xA5)
            size = lc.lc_encode_t(w, ref, 4, out)
        finally:
            lc.lc_set_option(lc.OPT_KEY_STAGING, lc.STAGING_AUTO)
        assert size == want.size and np.array_equal(out[:size].cpu().numpy(), want), staging
    out.fill_(0xA5)
    sizes = lc.lc_encode_batch([w], [ref], 4, [out])
    assert sizes == [want.size] and np.array_equal(out[:want.size].cpu().numpy(), want)
    # behind a cached table that this vector voids, by workgroups that take several chunks each
    cache, other = lc.new_cache(DEV), torch.zeros_like(w[:CHUNK])
    other[::3] = 1000.0
    lc.lc_encode_cached_t(other, torch.zeros_like(other), 4, lc.alloc_out(CHUNK, 4, DEV), cache)
    out.fill_(0xA5)
    size, used = lc.lc_encode_cached_t(w, ref, 4, out, cache)
    assert not used and size == want.size and np.array_equal(out[:size].cpu().numpy(), want)
    rec = torch.zeros_like(w)                                  # and their restore, whose payloads are the longest there are
    assert lc.lc_verify(out[:want.size], n, dtype) == want.size
    assert lc.lc_decode_t(out[:want.size], rec) == want.size
    if dtype == torch.float32:
        back = np.zeros(n, np.float32); orc.decode(want, back)
        got = rec.cpu().numpy()
    else:
        back = np.zeros(n, np.uint16); orc.decode_t(want, back, orc.DT_BF16)
        got = rec.view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(got.view(np.uint8), back.view(np.uint8))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [(1 << 22) + 5, 20_000_001, 40_000_000])
def test_restore_of_payloads_of_every_length(lc, dtype, n):
    """A workgroup of a restore has room for payloads of 15, 8 or 4 bits per element, by how many share a compute unit: payloads of
    2 to 5.6 thousand words in launches of each kind."""
    print("payloads", dtype, n, flush=True)
    g = torch.Generator(device=DEV); g.manual_seed(n)
    i = torch.arange(n, device=DEV)
    k = torch.floor(-torch.log2(torch.rand(n, generator=g, device=DEV).clamp_(min=2.0 ** -20)))
    common = torch.where((k > 0) & (k < 8), 8 - k, torch.zeros_like(k))
    share = 0.3 + (i // CHUNK) * (0.7 / 60)
    rare = torch.randint(8, 16, (n,), generator=g, device=DEV).float() * (torch.rand(n, generator=g, device=DEV) < share)
    e = torch.where((i < 60 * CHUNK) & (i // CHUNK % 10 == 0), rare, common)
    w = torch.where(e > 0, torch.exp2(e - 30), torch.zeros_like(e)).to(dtype)
    ref = torch.zeros_like(w)
    out = lc.alloc_out(n, 4, DEV)
    size = lc.lc_encode_t(w, ref, 4, out)
    blob = out[:size].clone()
    h = blob.cpu().numpy()
    words = np.diff(h[512:512 + 4 * 61].view(np.uint32).astype(int)) - 32
    assert words.max() > 4300, words
    rec, want = torch.zeros_like(w), np.zeros(n, np.float64 if dtype == torch.float64 else np.float32)
    assert lc.lc_decode_t(blob, rec) == size
    (orc.decode64 if dtype == torch.float64 else orc.decode)(h, want)
    assert np.array_equal(rec.cpu().numpy().view(np.uint8), want.view(np.uint8))
