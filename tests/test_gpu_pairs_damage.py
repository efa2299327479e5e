"""lc_decode_many of damaged blobs by the sweep that takes two symbols per look-up: strings that its check cannot tell from sound
ones and that end too early, too late or in no code, in inner chunks and in the ragged last one, between sound blobs.  The verdict
is the oracle's, and where that takes the damage for data, so are the values, bit for bit.  Arrays are off alignment, of which every
list of several blobs takes that sweep, in a process of its own, in which no call takes the one-launch route."""
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
n = 4 * CHUNK + 100
g = torch.Generator(device=DEV); g.manual_seed(43)
rand = lambda: torch.rand(n, generator=g, device=DEV)
zero, out = torch.zeros(n, device=DEV), lc.alloc_out(n, 4, DEV)
start = torch.randn(n + 1, generator=g, device=DEV)

def blob_of(delta, nbits):
    return out[:lc.lc_encode(delta, zero, nbits, out)].cpu().numpy().copy()

def restore(blobs):
    rec = start.clone()
    try: lc.lc_decode_many([torch.from_numpy(b).to(DEV) for b in blobs], rec[1:])
    except lc.LcError as e: return e.status, None
    return 0, rec[1:].cpu().numpy()

def oracle(blobs):
    want = start[1:].cpu().numpy().copy()
    try:
        for b in blobs: orc.decode(b, want)
    except orc.OracleError as e: return e.status, None
    return 0, want

def compare(blobs, what):
    print(what, flush=True)
    got, want = restore(blobs), oracle(blobs)
    assert got[0] == want[0], (what, got[0], want[0])
    assert want[1] is None or np.array_equal(got[1].view(np.uint32), want[1].view(np.uint32)), what
    return got[0]

sign = torch.where(rand() < 0.5, -1.0, 1.0)
spread = sign * torch.exp2(torch.floor(torch.log2(rand().clamp_(min=1e-6)))) * (1 + rand()) * 0.05       # codes of many lengths
for nbits, count in ((3, 5), (3, 2), (4, 3), (4, 2)):
    good = blob_of(spread, nbits)
    # (where the chunk records start, and each one's place and words)
    area = 512 + (4 * 6 + 15) // 16 * 16
    off = good[512:512 + 24].view(np.uint32)
    refused = 0
    for c in (0, 2, 3, 4):
        first, end = area + 4 * int(off[c]) + 128, area + 4 * int(off[c + 1])
        for at in sorted({first, first + 1, (3 * first + end) // 4, (first + end) // 2, (first + 3 * end) // 4, end - 5, end - 1}):
            for flip in (0x5A, 0xFF):
                bad = good.copy(); bad[at] ^= flip
                refused += compare([good] * (count // 2) + [bad] + [good] * (count - count // 2 - 1), "%%d bits x%%d chunk %%d at %%d" %% (nbits, count, c, at)) != 0
        # a lane's length handed to its neighbour: the sum, all that the check sees, stays
        bad = good.copy(); lens = bad[first - 128:first].view(np.uint16); lens[20] += 9; lens[21] -= 9
        refused += compare([bad] + [good] * (count - 1), "lengths of chunk %%d" %% c) != 0
    assert refused >= 10, refused

# every lane of the ragged chunk as long as a full chunk's of merged symbols only, and a payload of zero bits
for nbits, count in ((3, 5), (3, 2), (4, 3)):
    b = blob_of(torch.where(rand() < 0.001, 0.01 * sign, zero), nbits)
    words = b[512:512 + 24].view(np.uint32)
    K = int(b[20:24].view(np.uint32)[0]); merged = int(b[64 + 16 * K + 2])
    assert merged == 1
    b = np.concatenate([b[:512 + (4 * 6 + 15) // 16 * 16 + 4 * int(words[4])], np.full(64, 256 * merged, np.uint16).view(np.uint8), np.zeros(4 * 512 * merged, np.uint8)])
    b[512 + 20:512 + 24].view(np.uint32)[0] = int(words[4]) + 32 + 512 * merged
    b[40:48].view(np.uint64)[0] = b.size
    assert compare([b] * count, "ragged chunk of a full one's lengths x%%d" %% count) == lc.ERR_BAD_BLOB
print("ok")
"""


def test_damaged_strings():
    env = dict(os.environ, LC_TUNE_ONE_DEC_PER_CU="0")
    r = subprocess.run([sys.executable, "-c", RUN % ROOT], env=env, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-1500:] + r.stderr[-3000:]
