"""Restores of short vectors, which run in one launch whose workgroups take every string in eight segments at once, against the
oracle, bit for bit: whole, ragged and single chunks, unaligned arrays, every element type; codes that never fall into step
with themselves (all of one length), of one bit, of more than 10 bits; strings whose segments differ widely; damaged blobs;
the largest size and the first beyond; many threads; workgroups that give up meeting."""
import os
import subprocess
import sys
import threading

import numpy as np
import pytest
import torch

from oracle import lc_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CHUNK = 16384
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DT = {torch.float32: orc.DT_F32, torch.bfloat16: orc.DT_BF16, torch.float16: orc.DT_F16}


@pytest.fixture(scope="module")
def lc():
    from paper_2009_13003_amd import lc as mod
    return mod


def host(t):
    if t.dtype == torch.bfloat16:
        return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16).copy()
    return t.cpu().numpy().copy()


def restored(blob, start):
    """The oracle's restore of start (a device tensor) as bytes, or its status."""
    want = host(start)
    try:
        if start.dtype == torch.float64:
            orc.decode64(blob, want)
        elif start.dtype == torch.float32:
            orc.decode(blob, want)
        else:
            orc.decode_t(blob, want, DT[start.dtype])
    except orc.OracleError as e:
        return e.status
    return want.view(np.uint8)


def binades(kind, n, g):
    """Exponents above the reference (0: unchanged) of n elements."""
    if kind == "one length":                                 # 16 symbols (with nbits 4), all as frequent
        return torch.arange(n, device=DEV).remainder(16).float()[torch.randperm(n, generator=g, device=DEV)]
    if kind == "one bit":
        return (torch.rand(n, generator=g, device=DEV) < 0.4).float()
    if kind == "one symbol":
        return torch.zeros(n, device=DEV)
    if kind == "few":                                        # behind chunk 0, which fixes the code (merged: 1 bit, the others 2), few kept ones
        e = torch.zeros(n, device=DEV)
        e[:CHUNK] = torch.floor(2.5 * torch.rand(min(n, CHUNK), generator=g, device=DEV))
        for chunk in range(1, (n + CHUNK - 1) // CHUNK - 1):
            # (32 symbols of a lane are noted, a lane of more than 64 bits above its merged ones takes the usual path)
            for lane, count in ((3, 1), (chunk % 64, 30 + chunk), (63, 5)):
                p = torch.randperm(256, generator=g, device=DEV)[:count]
                e[chunk * CHUNK + (p // 4) * 256 + lane * 4 + p % 4] = 1 + (p % 2).float()
        e[n - 1] = 2
        return e
    k = torch.floor(-torch.log2(torch.rand(n, generator=g, device=DEV).clamp_(min=2.0 ** -20)))
    e = torch.where((k > 0) & (k < 16), 16 - k, torch.zeros_like(k))
    if kind == "uneven":                                     # every lane: kept symbols in the first quarter of its rows, few behind
        quiet = (torch.arange(n, device=DEV) // 256) % 64 >= 16
        e = torch.where(quiet & (torch.rand(n, generator=g, device=DEV) < 0.999), torch.zeros_like(e), e)
    return e                                                 # "deep": codes of 1 to 15 bits


def case(lc, kind, n, offset, dtype, nbits, seed=0):
    g = torch.Generator(device=DEV); g.manual_seed(n + offset + seed)
    e = binades(kind, n, g)
    d = torch.where(e > 0, torch.exp2(e - 9) * (1 + 0.5 * torch.rand(n, generator=g, device=DEV)), torch.zeros_like(e))
    w, ref = torch.zeros(n + offset, device=DEV, dtype=dtype), torch.zeros(n + offset, device=DEV, dtype=dtype)
    w[offset:] = d.to(dtype)
    out = lc.alloc_out(n, nbits, DEV)
    blob = out[:lc.lc_encode_t(w[offset:], ref[offset:], nbits, out)].clone()
    start = torch.randn(n + offset, generator=g, device=DEV).to(dtype)
    return blob, start


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16, torch.float64])
@pytest.mark.parametrize("n,offset", [(1, 0), (5, 1), (1025, 0), (CHUNK, 0), (CHUNK + 3, 1), (3 * CHUNK - 1, 0), (18 * CHUNK + 777, 0), (33 * CHUNK, 1)])
@pytest.mark.parametrize("kind", ["one length", "one bit", "one symbol", "deep", "uneven", "few"])
def test_short_restores(lc, kind, n, offset, dtype):
    for nbits in (4, 3) if kind in ("deep", "one length") else (4,):
        print("short", kind, n, offset, dtype, nbits, flush=True)
        blob, start = case(lc, kind, n, offset, dtype, nbits)
        rec = start.clone()
        assert lc.lc_decode_t(blob, rec[offset:]) == blob.numel()
        assert np.array_equal(host(rec[offset:]).view(np.uint8), restored(blob.cpu().numpy(), start[offset:]))
        assert torch.equal(rec[:offset].view(torch.uint8), start[:offset].view(torch.uint8))


@pytest.mark.parametrize("chunks", [16, 17, 512, 513])
def test_largest(lc, chunks):
    for dtype in (torch.float32, torch.float64):
        print("largest", chunks, dtype, flush=True)
        blob, start = case(lc, "deep", chunks * CHUNK, 0, dtype, 3)
        rec = start.clone()
        lc.lc_decode_t(blob, rec)
        assert torch.equal(rec.view(torch.uint8), torch.from_numpy(restored(blob.cpu().numpy(), start)).to(DEV))


@pytest.mark.parametrize("kind", ["one length", "deep", "one symbol", "few"])
def test_damaged_blobs(lc, kind):
    """The verifying sweep's and the oracle's verdict on blobs with one bit flipped; found before the first store in the header and the offsets."""
    n = 5 * CHUNK + 1234
    blob, start = case(lc, kind, n, 0, torch.float32, 4)
    h = blob.cpu().numpy()
    area = 512 + (4 * 7 + 15) // 16 * 16
    rng = np.random.RandomState(len(kind))
    places = [int(x) for x in rng.randint(0, 512 * 8, 40)] + [int(x) for x in rng.randint(512 * 8, area * 8, 20)] + \
             [int(x) for x in rng.randint(area * 8, (area + 128) * 8, 20)] + [int(x) for x in rng.randint((area + 128) * 8, 8 * h.size, 60)]
    for at in places:
        bad = h.copy(); bad[at // 8] ^= 1 << (at % 8)
        rec, dev = start.clone(), torch.from_numpy(bad).to(DEV)
        status = lambda call: (call(), 0)[1]
        try:
            want = status(lambda: lc.lc_verify(dev, n, torch.float32))       # (not this path)
        except lc.LcError as e:
            want = e.status
        try:
            got = status(lambda: lc.lc_decode(dev, rec))
        except lc.LcError as e:
            got = e.status
        assert got == want, (at, got, want)
        if got and at < area * 8:                            # (a lane's length may be wrong and the record's size right)
            assert torch.equal(rec, start), at
        if at >= 512 * 8 or not got:                         # (the oracle does not look at every reserved byte of the header)
            values = restored(bad, start)
            assert got == values if isinstance(values, int) else not got and np.array_equal(host(rec).view(np.uint8), values), at
    rec = start.clone()                                      # and nothing of it stays behind
    lc.lc_decode(blob, rec)
    assert np.array_equal(host(rec).view(np.uint8), restored(h, start))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16, torch.float64])
@pytest.mark.parametrize("n,offset,kinds", [(7, 0, ["deep", "one bit"]), (CHUNK + 900, 1, ["deep", "uneven", "one symbol", "few"]), (5 * CHUNK, 0, ["one length"] * 3),
                                            (21 * CHUNK - 2, 0, ["deep", "one symbol", "one bit", "uneven", "deep", "one length", "deep", "uneven", "deep"])])
def test_several_blobs(lc, dtype, n, offset, kinds):
    """lc_decode_many in one launch: as one restore after the other (16-bit values rounded after every blob)."""
    print("several", dtype, n, offset, len(kinds), flush=True)
    blobs, start = [], None
    for k, kind in enumerate(kinds):
        blob, start = case(lc, kind, n, offset, dtype, 4 - k % 2, seed=k)
        blobs.append(blob)
    rec = start.clone()
    assert lc.lc_decode_many_t(blobs, rec[offset:]) == sum(b.numel() for b in blobs)
    want = start.clone()
    for blob in blobs:
        h = restored(blob.cpu().numpy(), want[offset:])
        want[offset:].view(torch.uint8).copy_(torch.from_numpy(h))
    assert torch.equal(rec.view(torch.uint8), want.view(torch.uint8))
    for at in sorted({0, len(blobs) // 2, len(blobs) - 1}):  # one of them damaged: nothing is touched
        for byte, bit, status in ((8, 1, lc.ERR_BADARG), (67, 0, lc.ERR_BAD_BLOB), (512, 4, lc.ERR_BAD_BLOB)):
            bad = [b.clone() for b in blobs]
            bad[at][byte] ^= 1 << bit
            rec = start.clone()
            with pytest.raises(lc.LcError) as e:
                lc.lc_decode_many_t(bad, rec[offset:])
            assert e.value.status == status and torch.equal(rec.view(torch.uint8), start.view(torch.uint8)), (at, byte)
    rec = start.clone()
    lc.lc_decode_many_t(blobs, rec[offset:])
    assert torch.equal(rec.view(torch.uint8), want.view(torch.uint8))


@pytest.mark.parametrize("dtype,chunks,kind,count,kernels", [
    (torch.float32, 20, "deep", 6, {"k_dec_check", "k_decode_one"}), (torch.bfloat16, 257, "deep", 4, {"k_dec_check", "k_decode_one"}),
    (torch.float64, 257, "deep", 2, {"k_dec_check", "k_decode_one"}), (torch.float64, 257, "few", 2, {"k_dec_check", "k_decode"}),
    (torch.float32, 20, "one bit", 6, {"k_dec_check", "k_decode_fused"}), (torch.float32, 257, "one bit", 3, {"k_decode_one"}),
    (torch.float64, 256, "deep", 33, {"k_decode_one"})])
def test_several_blobs_by_what_the_check_finds(lc, dtype, chunks, kind, count, kernels):
    """Lists that go into one launch only once their codes or sizes are known, and those beside them that do not."""
    print("by the check", dtype, chunks, kind, count, flush=True)
    blobs, start = [], None
    for k in range(min(count, 3)):
        blob, start = case(lc, kind, chunks * CHUNK, 0, dtype, 4, seed=k)
        blobs.append(blob)
    blobs = [blobs[k % len(blobs)] for k in range(count)]
    rec, want = start.clone(), start.clone()
    lc.lc_profile(True)
    assert lc.lc_decode_many_t(blobs, rec) == sum(b.numel() for b in blobs)
    ran = {k for k, v in lc.lc_profile_read().items() if v[1]}
    lc.lc_profile(False)
    for kernel in ("k_decode_one", "k_decode_fused"):        # (the others of a list are not timed)
        assert (kernel in ran) == (kernel in kernels), ran
    for blob in blobs[:1] if count > 8 else blobs:
        want.view(torch.uint8).copy_(torch.from_numpy(restored(blob.cpu().numpy(), want)))
    if count > 8:                                            # (the oracle for the first, single restores for the rest)
        for blob in blobs[1:]:
            lc.lc_decode_t(blob, want)
    assert torch.equal(rec.view(torch.uint8), want.view(torch.uint8))


def test_many_threads(lc):
    """More calls at once than fit the chip in one launch each, encodes among them."""
    jobs = [case(lc, "deep", k * CHUNK + 31 * k, 0, torch.float32, 3) for k in (3, 60, 130, 200, 256, 255, 90, 17)]
    want = [restored(b.cpu().numpy(), s) for b, s in jobs]
    wrong = []

    def work(i):
        blob, start = jobs[i]
        s = torch.cuda.Stream()
        out = lc.alloc_out(start.numel(), 3, DEV)
        with torch.cuda.stream(s):
            for _ in range(20):
                rec = start.clone()
                lc.lc_decode(blob, rec)
                size = lc.lc_encode(rec, start, 3, out)
                again = start.clone()
                lc.lc_decode(out[:size], again)
                if not np.array_equal(host(rec).view(np.uint8), want[i]) or size <= 512:
                    wrong.append(i)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not wrong


@pytest.mark.parametrize("looks", ["-1", "0", "1"])
def test_workgroups_that_give_up(looks):
    """-1: every call; with a little patience hardly any (their wait begins behind the decoding)."""
    code = """
import sys, torch, numpy as np
sys.path.insert(0, %r)
from tests.test_gpu_short_decode import case, restored, host, CHUNK
from paper_2009_13003_amd import lc
lc.lc_profile(True)
for k in range(60):
    n = (k * 37 %% 250 + 1) * CHUNK + k
    blob, start = case(lc, 'deep', n, 0, torch.float32, 3)
    for turn in range(3):
        rec = start.clone()
        assert lc.lc_decode(blob, rec) == blob.numel()
        assert np.array_equal(host(rec).view(np.uint8), restored(blob.cpu().numpy(), start)), (k, turn)
        many = start.clone()
        lc.lc_decode_many_t([blob, blob], many)
        lc.lc_decode(blob, rec)
        assert torch.equal(rec, many), (k, turn)
p = lc.lc_profile_read()
given_up = p['k_decode'][1], p['k_decode_fused'][1]
assert p['k_decode_one'][1] == 540 and (given_up == (360, 180) or sys.argv[1] != '-1'), p
print('same')
""" % ROOT
    env = dict(os.environ, LC_TUNE_ONE_WAIT=looks, LC_TUNE_ONE_REST="0")
    res = subprocess.run([sys.executable, "-c", code, looks], capture_output=True, text=True, env=env, cwd=ROOT, timeout=100)
    assert res.returncode == 0 and "same" in res.stdout, res.stdout[-2000:] + res.stderr[-2000:]
