"""lc_decode_many by the sweep that takes two symbols per look-up: every number of blobs, with 8 symbols and with 16, codes that do
not fit its tables together and ones that do not fit them alone, strings that outrun the words at hand, ragged ends, arrays off
alignment, every element type.  Against the oracle's restores, one after the other, bit for bit (one addition per element and
blob: no tolerance).  In a process of its own, in which no call takes the one-launch route and every list that may takes this sweep;
how often it ran is checked as well."""
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
g = torch.Generator(device=DEV); g.manual_seed(41)
rand = lambda n: torch.rand(n, generator=g, device=DEV)

def delta(kind, n):
    sign = torch.where(rand(n) < 0.5, -1.0, 1.0)
    if kind == "flat":                                 # all symbols as frequent: the longest strings, 4 bits an element
        return sign * torch.exp2(-torch.floor(7.99 * rand(n))) * (1 + rand(n)) * 0.05
    if kind == "spread":                               # codes of up to 15 bits
        return sign * torch.exp2(torch.floor(torch.log2(rand(n).clamp_(min=1e-6)))) * (1 + rand(n)) * 0.05
    if kind == "layered":                              # chunks of rare symbols only among chunks of merged ones
        d = 1e-5 * sign * rand(n)
        d[:CHUNK // 3] = (sign * torch.exp2(-torch.floor(15.99 * rand(n))) * 0.5)[:CHUNK // 3]
        return d
    if kind == "few":
        return torch.where(rand(n) < 0.001, sign * 0.01, torch.zeros(n, device=DEV))
    if kind == "one":                                  # a single symbol, the code of which starts half the windows only
        return torch.full((n,), 0.25, device=DEV)
    return torch.zeros(n, device=DEV)                  # unchanged

KINDS = ["flat", "spread", "layered", "few", "one", "none", "flat", "spread"]
def check(n, offset, nbits, kinds, what, sweeps):
    print(what, sys.argv[1], n, offset, nbits, kinds, flush=True)
    start = torch.randn(n + offset, generator=g, device=DEV).to(dtype)
    zero = torch.zeros(n, device=DEV, dtype=dtype)
    out, blobs = lc.alloc_out(n, 4, DEV), []
    for k, b in zip(kinds, nbits):
        blobs.append(out[:lc.lc_encode_t(delta(k, n).to(dtype), zero, b, out)].clone())
    rec = start.clone()
    lc.lc_profile(True)
    assert lc.lc_decode_many_t(blobs, rec[offset:]) == sum(b.numel() for b in blobs)
    ran = {k: v[1] for k, v in lc.lc_profile_read().items() if v[1]}
    lc.lc_profile(False)
    assert (sweeps is None and ran["k_decode_pairs"] > 1) or ran == dict(sweeps if isinstance(sweeps, dict) else {"k_decode_pairs": sweeps}, k_dec_check=1), (what, ran)
    raw = lambda t: t.cpu().view(torch.int32 if dtype == torch.float32 else torch.int16).numpy()
    want = raw(start[offset:]).copy()
    want = want.view({0: np.float32, 1: np.uint16, 2: np.float16}[name])
    for b in blobs:
        if dtype == torch.float32: orc.decode(b.cpu().numpy(), want)
        else: orc.decode_t(b.cpu().numpy(), want, name)
    assert np.array_equal(raw(rec[offset:]).view(np.uint8), want.view(np.uint8)), what
    assert torch.equal(rec[:offset].view(torch.uint8), start[:offset].view(torch.uint8))

for offset in (0, 1, 3):
    for n in (5, 255, CHUNK - 1, CHUNK, 2 * CHUNK + 256 * 3 + 9, 9 * CHUNK + 514):
        for count in ((5, 6, 7, 8) if offset == 0 else (2, 3, 4, 8)):
            check(n, offset, [3] * count, [KINDS[(i + n) %% 8] for i in range(count)], "narrow", 1)
        for count in ((3, 4) if offset == 0 else (2, 3, 4)):
            check(n, offset, [4] * count, [KINDS[(2 * i + n + count) %% 8] for i in range(count)], "wide", 1)
check(3 * CHUNK + 77, 0, [3] * 5 + [4] * 6 + [3] * 9, (["flat", "spread"] * 10)[:20], "runs", 1 + 2 + 2)
check(3 * CHUNK + 77, 0, [3, 4] * 7, ["flat", "spread"] * 7, "mixed", 4)
check(3 * CHUNK + 77, 1, [3, 4] * 7, (KINDS * 2)[:14], "mixed", None)
check(3 * CHUNK, 0, [2, 3, 1, 3, 2, 3, 3, 1, 2, 3, 3, 3, 1], ["none"] * 13, "unchanged", 2)
# (off alignment, one blob that has a sweep to itself: the kernel of single restores)
check(5 * CHUNK + 9, 3, [4] + [3] * 6, ["flat", "spread"] * 3 + ["flat"], "one and several", {"k_decode": 1, "k_decode_pairs": 1})
check(5 * CHUNK + 9, 1, [3], ["spread"], "one", {"k_decode": 1})
# (more chunks than wavefronts, 8 or 16 per compute unit)
check(2101 * CHUNK + 1025, 0, [3] * 6, ["spread", "few", "none"] + ["flat"] * 3, "several chunks to a wavefront, narrow", 1)
check(4501 * CHUNK + 77, 1, [3] * 3, ["few", "spread", "none"], "several chunks to a wavefront, two workgroups per unit", 1)
check(4400 * CHUNK, 0, [3] * 5, ["none"] * 4 + ["few"], "several chunks to a wavefront, hardly a kept symbol", 1)
check(2100 * CHUNK, 0, [4] * 3, ["spread", "layered", "flat"], "several chunks to a wavefront, wide", 1)
print("ok")
"""


@pytest.mark.parametrize("dtype", ["float32", "bfloat16", "float16"])
def test_pairs_of_symbols(dtype):
    env = dict(os.environ, LC_TUNE_ONE_DEC_PER_CU="0", LC_TUNE_PAIRS="1")
    r = subprocess.run([sys.executable, "-c", RUN % ROOT, dtype], env=env, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-1500:] + r.stderr[-3000:]
