"""lc_decode_many by the sweep that looks up one symbol at a time, of vectors whose last chunk is ragged: no whole row in it, one, as
many as are read ahead and one more, all but one; a rest behind them or none; every number of blobs, short codes and long ones,
payloads that fit the LDS beside others' and ones that do not, every element type.  Against the oracle's restores, one after the
other, bit for bit (one addition per element and blob: no tolerance), and its verdict where the ragged chunk is damaged.  In a
process of its own, in which all lists take this sweep."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUN = r"""
import sys, numpy as np, torch
sys.path.insert(0, %r)
from paper_2009_13003_amd import lc
from oracle import lc_oracle as orc
DEV, CHUNK = "cuda:0", 16384
dtype, name = getattr(torch, sys.argv[1]), {"float32": 0, "bfloat16": 1, "float16": 2}[sys.argv[1]]
g = torch.Generator(device=DEV); g.manual_seed(47)
rand = lambda n: torch.rand(n, generator=g, device=DEV)
raw = lambda t: t.cpu().view(torch.int32 if dtype == torch.float32 else torch.int16).numpy()

def delta(kind, n):
    sign = torch.where(rand(n) < 0.5, -1.0, 1.0)
    if kind == "flat": return sign * torch.exp2(-torch.floor(7.99 * rand(n))) * (1 + rand(n)) * 0.05
    if kind == "spread": return sign * torch.exp2(torch.floor(torch.log2(rand(n).clamp_(min=1e-6)))) * (1 + rand(n)) * 0.05
    if kind == "few": return torch.where(rand(n) < 0.001, sign * 0.01, torch.zeros(n, device=DEV))
    if kind == "end":                                  # the ragged chunk's strings far longer than the others'
        d = 1e-5 * sign * rand(n)
        d[n // CHUNK * CHUNK:] = (sign * torch.exp2(-torch.floor(15.99 * rand(n))) * 0.5)[n // CHUNK * CHUNK:]
        return d
    return torch.zeros(n, device=DEV)

def blob_of(kind, n, nbits):
    out = lc.alloc_out(n, nbits, DEV)
    return out[:lc.lc_encode_t(delta(kind, n).to(dtype), torch.zeros(n, device=DEV, dtype=dtype), nbits, out)].cpu().numpy().copy()

def compare(blobs, n, what):
    start = torch.randn(n, generator=g, device=DEV).to(dtype)
    want = raw(start).copy().view({0: np.float32, 1: np.uint16, 2: np.float16}[name])
    verdict = got = 0
    try:
        for b in blobs: orc.decode(b, want) if dtype == torch.float32 else orc.decode_t(b, want, name)
    except orc.OracleError as e: verdict = e.status
    try: lc.lc_decode_many_t([torch.from_numpy(b).to(DEV) for b in blobs], start)
    except lc.LcError as e: got = e.status
    assert got == verdict, (what, got, verdict)
    assert got or np.array_equal(raw(start).view(np.uint8), want.view(np.uint8)), what
    return got

KINDS = ["flat", "spread", "few", "none", "end", "spread", "flat", "few"]
for nbits in (3, 4):
    lc.lc_profile(True)
    for rest in (1, 255, 256, 257, 3 * 256 + 9, 4 * 256, 5 * 256 + 77, 8 * 256, 9 * 256 + 130, 63 * 256, CHUNK - 1):
        for count in (1, 2, 3, 4, 5, 6, 7, 8):
            n = (count %% 3) * CHUNK + rest
            print(sys.argv[1], n, count, nbits, flush=True)
            compare([blob_of(KINDS[(i + rest + count) %% 8], n, nbits) for i in range(count)], n, (n, count, nbits))
    ran = {k: v[1] for k, v in lc.lc_profile_read().items() if v[1]}
    lc.lc_profile(False)
    assert {"k_dec_check", "k_decode_fused"} <= ran.keys() and "k_decode_pairs" not in ran and "k_decode" not in ran, ran
    assert nbits == 4 or ran["k_decode_fused"] == ran["k_dec_check"], ran       # (of short codes only a sweep a list)
# damage in the ragged chunk that the check cannot see: strings that end elsewhere, and a full chunk's lengths with a payload of zeros
n, refused = CHUNK + 7 * 256 + 100, 0
for nbits, count in ((3, 8), (3, 2), (4, 3)):
    good = blob_of("spread", n, nbits)
    area = 512 + 16
    first, end = (area + 4 * int(w) for w in good[512 + 4:512 + 12].view(np.uint32))
    first += 128
    for at in sorted({first, first + 1, (3 * first + end) // 4, (first + end) // 2, (first + 3 * end) // 4, end - 5, end - 1}):
        for flip in (0x5A, 0xFF):
            bad = good.copy(); bad[at] ^= flip
            refused += compare([good] * (count // 2) + [bad] + [good] * (count - count // 2 - 1), n, (nbits, count, at, flip)) != 0
    b = blob_of("few", n, nbits)
    K = int(b[20:24].view(np.uint32)[0]); merged = int(b[64 + 16 * K + 2])
    head, words = b[:512 + 16 + 4 * int(b[516:520].view(np.uint32)[0])], 32 + 512 * merged
    b = np.concatenate([head, np.full(64, 256 * merged, np.uint16).view(np.uint8), np.zeros(4 * 512 * merged, np.uint8)])
    b[520:524].view(np.uint32)[0] = int(b[516:520].view(np.uint32)[0]) + words
    b[40:48].view(np.uint64)[0] = b.size
    assert compare([b] * count, n, "a full chunk's lengths") == lc.ERR_BAD_BLOB
assert refused >= 12, refused
print("ok")
"""


@pytest.mark.parametrize("dtype", ["float32", "bfloat16", "float16"])
def test_ragged_chunk(dtype):
    env = dict(os.environ, LC_TUNE_ONE_DEC_PER_CU="0", LC_TUNE_PAIRS="2", LC_TUNE_FUSED_MIN_WAVES_PER_CU="2")
    r = subprocess.run([sys.executable, "-c", RUN % ROOT, dtype], env=env, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-1500:] + r.stderr[-3000:]
