"""Restores of chunks of few kept symbols, which go from one kept symbol to the next and touch nothing else: at the ends of a
lane's string, more of them in a lane than its notes hold, ragged ends, unaligned arrays, every element type, and merged
symbols' codes of one bit and of two.  Against the oracle, bit for bit (a restore is one addition per element: no tolerance)."""
import numpy as np
import pytest
import torch

from oracle import lc_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CHUNK = 16384


@pytest.fixture(scope="module")
def lc():
    from paper_2009_13003_amd import lc as mod
    return mod


def few(n, merged, seed):
    """Binades (0: unchanged) of a vector: chunk 0 fixes the code, a share `merged` of it merged; the others hold few kept."""
    g = torch.Generator(device=DEV); g.manual_seed(seed)
    pick = lambda m: torch.randint(1, 7, (m,), generator=g, device=DEV).float()
    e = torch.zeros(n, device=DEV)
    e[:CHUNK] = torch.where(torch.rand(CHUNK, generator=g, device=DEV) < merged, e[:CHUNK], pick(CHUNK))

    def keep(chunk, lane, first, count):                   # symbols first .. first + count - 1 of a lane's string
        p = torch.arange(first, first + count, device=DEV)
        e[chunk * CHUNK + (p // 4) * 256 + lane * 4 + p % 4] = pick(count)

    keep(1, 0, 0, 1); keep(1, 63, 255, 1); keep(1, 7, 0, 8); keep(1, 8, 100, 9); keep(1, 9, 248, 8); keep(1, 10, 31, 2)
    keep(2, 5, 0, 16); keep(2, 6, 64, 17); keep(2, 7, 200, 20)
    keep(3, 11, 0, 256)                                    # a lane that holds nothing else: the usual path
    at = torch.randperm(CHUNK, generator=g, device=DEV)[:150]
    e[4 * CHUNK + at] = pick(150)
    e[5 * CHUNK + 37 * 256:5 * CHUNK + 38 * 256] = pick(256)
    e[6 * CHUNK] = 3
    e[n - 1] = 2                                           # the last element of all, and a few of the chunk that it ends
    if n > 7 * CHUNK + 300:
        e[7 * CHUNK + 299] = 4
    return e


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16, torch.float64])
@pytest.mark.parametrize("n,offset", [(7 * CHUNK, 0), (7 * CHUNK + 1, 0), (7 * CHUNK + 2047, 1), (8 * CHUNK - 3, 0), (7 * CHUNK + 514, 0)])
@pytest.mark.parametrize("merged", [0.6, 0.27])
def test_few_kept_symbols(lc, dtype, n, offset, merged):
    print("few kept", dtype, n, offset, merged, flush=True)
    g = torch.Generator(device=DEV); g.manual_seed(n)
    e = few(n, merged, n + offset)
    if merged < 0.5:                                       # more chunks of the dense kind, or the code of the merged symbol is one bit
        dense = few(CHUNK * 7, merged, 9)[:CHUNK]
        e = torch.cat([dense.repeat(60), e])
    total = e.numel()
    d = torch.where(e > 0, torch.exp2(e - 8) * (1 + 0.5 * torch.rand(total, generator=g, device=DEV)), torch.zeros_like(e))
    w, ref = torch.zeros(total + offset, device=DEV, dtype=dtype), torch.zeros(total + offset, device=DEV, dtype=dtype)
    w[offset:] = d.to(dtype)
    out = lc.alloc_out(total, 3, DEV)
    size = lc.lc_encode_t(w[offset:], ref[offset:], 3, out)
    blob = out[:size].clone()
    h = blob.cpu().numpy()
    lens = h[66:66 + 16 * (int(h[20]) + 1):16].tolist()
    assert lens[-1] == (1 if merged > 0.5 else 2) and min(lens[:-1]) > lens[-1], lens
    # onto values of every kind, so that an element that is not its own would show
    start = torch.randn(total + offset, generator=g, device=DEV).to(dtype)
    rec, batch = start.clone(), start.clone()
    assert lc.lc_decode_t(blob, rec[offset:]) == size
    assert lc.lc_decode_batch([blob], [batch[offset:]]) == [size] or dtype == torch.float64
    assert torch.equal(rec[:offset].view(torch.uint8), start[:offset].view(torch.uint8))
    if dtype == torch.float64:
        want = start[offset:].cpu().numpy(); orc.decode64(h, want)
    elif dtype == torch.float32:
        want = start[offset:].cpu().numpy(); orc.decode(h, want)
    elif dtype == torch.float16:
        want = start[offset:].cpu().numpy().copy(); orc.decode_t(h, want, orc.DT_F16)
    else:
        want = start[offset:].view(torch.int16).cpu().numpy().view(np.uint16).copy()
        orc.decode_t(h, want, orc.DT_BF16)
    raw = lambda t: np.ascontiguousarray(t[offset:].view(torch.uint8).cpu().numpy())
    assert np.array_equal(raw(rec), want.view(np.uint8))
    assert np.array_equal(raw(batch), want.view(np.uint8))
