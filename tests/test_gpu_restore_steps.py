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
