"""The restore's decoding, where lanes advance at very different rates: several symbols per look-up in some lanes, codes
longer than the look-up's 10 bits in others, so that the fast lanes run into the end of their symbol ring while the slow
ones lag; at the edges of the groups of 8 rows, of chunks, and of ragged and unaligned vectors.  Against the oracle, bit for
bit (a restore is one addition per element: no tolerance)."""
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


def uneven(n, seed, dtype, offset):
    """Even lanes hold the merged symbol only, odd lanes rare binades (codes of up to 15 bits), a quarter of the rows both."""
    g = torch.Generator(device=DEV); g.manual_seed(seed)
    i = torch.arange(n, device=DEV)
    lane, row = (i // 4) % 64, (i // 256) % 64
    common = torch.floor(-torch.log2(torch.rand(n, generator=g, device=DEV).clamp_(min=2.0 ** -13)))
    rare = torch.randint(8, 14, (n,), generator=g, device=DEV).float()
    e = torch.where((lane % 2 == 1) & (row % 4 != 3) & (i < 16384), rare, common)
    d = torch.exp2(e - 20) * (1 + 0.5 * torch.rand(n, generator=g, device=DEV))       # rare = large exponent
    d = torch.where((lane % 2 == 0) & (row % 4 != 3), torch.zeros_like(d), d)
    ref = torch.zeros(n + offset, device=DEV, dtype=dtype)
    w = ref.clone()
    w[offset:] = d.to(dtype)
    return w[offset:], ref[offset:]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float64])
@pytest.mark.parametrize("n,offset", [(2048 - 1, 0), (2048 + 3, 0), (16384 - 1, 0), (16384, 1), (16384 + 2047, 0),
                                      (3 * 16384 + 5 * 2048 + 257, 0), (3 * 16384 + 11, 1)])
def test_lanes_that_advance_at_different_rates(lc, dtype, n, offset):
    w, ref = uneven(n, n + offset, dtype, offset)
    for nbits in (3, 4):
        print("uneven lanes", dtype, n, offset, nbits, flush=True)
        out = lc.alloc_out(n, nbits, DEV)
        size = lc.lc_encode_t(w, ref, nbits, out)
        blob = out[:size].clone()
        h = blob.cpu().numpy()
        rec = torch.zeros(n + offset, device=DEV, dtype=dtype)
        assert lc.lc_verify(blob, n, dtype) == size
        assert lc.lc_decode_t(blob, rec[offset:]) == size
        other = rec.clone()
        assert lc.lc_decode_batch([blob, blob], [rec[offset:], other[offset:]]) == [size, size]
        assert torch.equal(rec.view(torch.uint8), other.view(torch.uint8))
        if dtype == torch.float64:
            want = np.zeros(n)
            for _ in range(2):
                orc.decode64(h, want)
            got = rec[offset:].cpu().numpy()
        elif dtype == torch.float32:
            want = np.zeros(n, np.float32)
            for _ in range(2):
                orc.decode(h, want)
            got = rec[offset:].cpu().numpy()
        else:
            want = np.zeros(n, np.uint16)
            for _ in range(2):
                orc.decode_t(h, want, orc.DT_BF16)
            got = rec[offset:].view(torch.int16).cpu().numpy().view(np.uint16)
        assert np.array_equal(np.ascontiguousarray(got).view(np.uint8), want.view(np.uint8))


@pytest.mark.parametrize("tail", [52, 999, 3 * 256 + 17, 5 * 256, 9 * 256 + 100, 13 * 256, 16 * 256 + 225, 18 * 256 - 3])
def test_ragged_chunks_whose_strings_end_within_a_word(lc, tail):
    """Many strings that end in the middle of a word of the ring, each by another last step."""
    n = 16384 + tail
    for seed in range(6):
        g = torch.Generator(device=DEV); g.manual_seed(100 * seed + tail)
        e = torch.floor(-torch.log2(torch.rand(n, generator=g, device=DEV).clamp_(min=2.0 ** -12)))
        w = torch.where(e > seed % 3, torch.exp2(e - 30), torch.zeros_like(e))
        ref = torch.zeros(n, device=DEV)
        out = lc.alloc_out(n, 3, DEV)
        blob = out[:lc.lc_encode(w, ref, 3, out)].clone()
        want, rec, many = np.zeros(n, np.float32), torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
        orc.decode(blob.cpu().numpy(), want)
        lc.lc_decode(blob, rec)
        assert np.array_equal(rec.cpu().numpy().view(np.uint32), want.view(np.uint32)), seed
        for count in (1, 5):
            many.zero_()
            lc.lc_decode_many([blob] * count, many)
            want = np.zeros(n, np.float32)
            for _ in range(count):
                orc.decode(blob.cpu().numpy(), want)
            assert np.array_equal(many.cpu().numpy().view(np.uint32), want.view(np.uint32)), (seed, count)


def test_a_string_that_the_group_before_has_finished(lc):
    """A ragged last chunk of 17 rows in which every lane's symbols run out in the look-up that passes the end of row 15: two
    codes of 5 bits, then merged symbols (1 bit, 6 to a look-up): 2 + 11 x 6 = 68.  Nothing is left to decode for row 16,
    whose symbols fill half a word."""
    n, nbits = 16384 + 17 * 256, 3
    i = torch.arange(n, device=DEV)
    e = torch.zeros(n, device=DEV)
    # populations of chunk 0: codes of 1 bit (merged), 2, 3, 4, 5 and 5 bits
    for binade, start, count in ((1, 0, 4000), (2, 4000, 2000), (3, 6000, 1000), (4, 7000, 100), (5, 7100, 100)):
        e[start:start + count] = binade
    first = (i >= 16384) & (i < 16384 + 256)
    e[first & (i % 4 == 0)] = 4
    e[first & (i % 4 == 1)] = 5
    w = torch.where(e > 0, torch.exp2(e - 30), torch.zeros_like(e))
    ref = torch.zeros(n, device=DEV)
    out = lc.alloc_out(n, nbits, DEV)
    size = lc.lc_encode(w, ref, nbits, out)
    blob = out[:size].clone()
    lens = sorted(blob.cpu().numpy()[66:66 + 16 * 6:16].tolist())
    assert lens == [1, 2, 3, 4, 5, 5], lens
    want = np.zeros(n, np.float32)
    orc.decode(blob.cpu().numpy(), want)
    rec = torch.zeros(n, device=DEV)
    assert lc.lc_decode(blob, rec) == size
    assert np.array_equal(rec.cpu().numpy().view(np.uint32), want.view(np.uint32))
    rec.zero_()
    assert lc.lc_decode_many([blob, blob], rec) == 2 * size
    orc.decode(blob.cpu().numpy(), want)
    assert np.array_equal(rec.cpu().numpy().view(np.uint32), want.view(np.uint32))
