"""Encodes of short vectors, which run in one launch whose workgroups meet twice, against the same call in four kernels (the
asynchronous one) and the oracle, byte for byte: whole, ragged and single chunks, unaligned arrays, every element type that
takes this path, chunks of long codes, deltas that are not finite, cached tables, the largest size and the first one beyond it,
calls of many threads at once, and workgroups that give up meeting, also while other threads' calls take the same scratch area."""
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


@pytest.fixture(scope="module")
def lc():
    from paper_2009_13003_amd import lc as mod
    return mod


def pair(n, dtype, offset, seed, rare=0):
    """Parameters and reference; with `rare`, the first elements hold the rarest buckets (codes far above the average)."""
    g = torch.Generator(device=DEV); g.manual_seed(seed)
    ref = 0.05 * torch.randn(n, generator=g, device=DEV)
    u = torch.rand(n, generator=g, device=DEV) - 0.5
    d = -1e-3 * torch.sign(u) * torch.log1p(-2.0 * u.abs().clamp(max=0.4999))
    if rare:
        d[:rare] *= 2.0 ** torch.randint(2, 5, (rare,), generator=g, device=DEV)
    buf = torch.zeros(2, n + offset, device=DEV, dtype=dtype)
    buf[0, offset:] = (ref + d).to(dtype)
    buf[1, offset:] = ref.to(dtype)
    return buf[0, offset:].clone() if offset == 0 else buf[0, offset:], buf[1, offset:].clone() if offset == 0 else buf[1, offset:]


def four_kernels(lc, w, ref, nbits, out, cache=None):
    size, used = lc.lc_encode_wait(lc.lc_encode_async_t(w, ref, nbits, out, cache=cache))
    return out[:size].cpu().numpy(), used


def oracle_blob(w, ref, nbits):
    if w.dtype == torch.float32:
        return orc.encode(w.cpu().numpy(), ref.cpu().numpy(), nbits)
    if w.dtype == torch.float16:
        return orc.encode_t(w.cpu().numpy(), ref.cpu().numpy(), nbits, orc.DT_F16)
    raw = lambda t: t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
    return orc.encode_t(raw(w), raw(ref), nbits, orc.DT_BF16)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n,offset", [(1, 0), (3, 1), (255, 0), (CHUNK - 1, 0), (CHUNK, 0), (CHUNK + 1, 1), (2 * CHUNK + 2048, 0), (9 * CHUNK - 3, 0),
                                      (37 * CHUNK, 3), (65 * CHUNK + 5, 0)])
def test_short_vectors(lc, dtype, n, offset):
    for nbits in (1, 3, 4):
        print("short", dtype, n, offset, nbits, flush=True)
        w, ref = pair(n, dtype, offset, n + nbits)
        out = lc.alloc_out(n, nbits, DEV)
        size = lc.lc_encode_t(w, ref, nbits, out)
        got = out[:size].cpu().numpy()
        want, _ = four_kernels(lc, w, ref, nbits, lc.alloc_out(n, nbits, DEV))
        assert np.array_equal(got, want) and np.array_equal(got, oracle_blob(w, ref, nbits))


@pytest.mark.parametrize("chunks", [256, 257, 512, 513])
def test_largest(lc, chunks):
    print("largest", chunks, flush=True)
    w, ref = pair(chunks * CHUNK, torch.float32, 0, chunks)
    out = lc.alloc_out(w.numel(), 3, DEV)
    size = lc.lc_encode(w, ref, 3, out)
    want, _ = four_kernels(lc, w, ref, 3, lc.alloc_out(w.numel(), 3, DEV))
    assert np.array_equal(out[:size].cpu().numpy(), want)


@pytest.mark.parametrize("rare", [3000, CHUNK, CHUNK + 700])
def test_chunks_of_long_codes(lc, rare):
    """Payloads of two and three windows of 2560 words, and a lane's part of more than 7 words."""
    print("long", rare, flush=True)
    for n in (40 * CHUNK, 40 * CHUNK + 300):
        w, ref = pair(n, torch.float32, 0, rare, rare)
        out = lc.alloc_out(n, 4, DEV)
        size = lc.lc_encode(w, ref, 4, out)
        got = out[:size].cpu().numpy()
        words = np.diff(got[512:512 + 4 * (n // CHUNK + 1)].view(np.uint32))
        assert rare < CHUNK or words.max() > 32 + 2560
        assert np.array_equal(got, oracle_blob(w, ref, 4))


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_deltas_that_are_not_finite(lc, bad):
    w, ref = pair(3 * CHUNK + 77, torch.float32, 0, 1)
    good = w.clone()
    for at in (0, 2 * CHUNK, 3 * CHUNK + 76):
        w.copy_(good); w[at] = bad
        out = lc.alloc_out(w.numel(), 3, DEV)
        with pytest.raises(lc.LcError) as e:
            lc.lc_encode(w, ref, 3, out)
        assert e.value.status == lc.ERR_NONFINITE
        head = out[:512].cpu().numpy()
        with pytest.raises(orc.OracleError) as want:
            orc.encode(w.cpu().numpy(), ref.cpu().numpy(), 3)
        assert np.array_equal(head, want.value.header)
        size = lc.lc_encode(good, ref, 3, out)               # nothing of it stays behind
        assert np.array_equal(out[:size].cpu().numpy(), oracle_blob(good, ref, 3))


@pytest.mark.parametrize("n", [CHUNK - 9, 11 * CHUNK + 5])
def test_cached_tables(lc, n):
    """Hit, moved kept set, other nbits, another element type's cache, caches that hold nonsense."""
    cache, cache_h = lc.new_cache(DEV), orc.new_cache()
    out = lc.alloc_out(n, 4, DEV)

    def step(seed, scale, nbits, expect=None):
        w, ref = pair(n, torch.float32, 0, seed)
        w = ref + scale * (w - ref)
        size, used = lc.lc_encode_cached_t(w, ref, nbits, out, cache)
        want, used_h = orc.encode_cached(w.cpu().numpy(), ref.cpu().numpy(), nbits, cache_h)
        assert used == used_h and (expect is None or bool(used) == expect), (seed, used, used_h)
        assert np.array_equal(out[:size].cpu().numpy(), want)
        assert np.array_equal(cache[:144].cpu().numpy().view(np.uint32), cache_h)

    step(1, 1.0, 3, False); step(1, 1.0, 3, True); step(1, 16.0, 3, False); step(1, 16.0, 4, False); step(1, 16.0, 4, True)
    for word, value in [(0, 2), (1, 3), (2, 16), (2, 0xFFFFFFFF), (4, 0), (4, 255), (4, 600), (5, 126), (20, 16), (21, 1), (35, 9)]:
        step(1, 16.0, 4)
        bad = cache_h.copy(); bad[word] = value
        cache_h[:] = bad
        cache[:144] = torch.from_numpy(bad.view(np.uint8)).to(DEV)
        step(1, 16.0, 4)


def test_many_threads(lc):
    """More calls at once than fit the chip in one launch each."""
    jobs = [pair(k * CHUNK + 31 * k, torch.float32, 0, k) for k in (3, 60, 130, 200, 256, 255, 90, 17)]
    want = [four_kernels(lc, w, r, 3, lc.alloc_out(w.numel(), 3, DEV))[0] for w, r in jobs]
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        w, r = jobs[i]
        s = torch.cuda.Stream()
        out = lc.alloc_out(w.numel(), 3, DEV)
        for _ in range(40):
            with torch.cuda.stream(s):
                size = lc.lc_encode(w, r, 3, out)
                if not np.array_equal(out[:size].cpu().numpy(), want[i]):
                    wrong.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not wrong


@pytest.mark.parametrize("looks", ["-1", "0", "1"])
def test_workgroups_that_give_up(looks):
    """With next to no patience most calls are given up at one of the meetings, by some of their workgroups (-1: all at the first):
    same blobs."""
    code = """
import sys, torch, numpy as np
sys.path.insert(0, %r)
from tests.test_gpu_short_encode import pair, four_kernels, CHUNK, DEV
from paper_2009_13003_amd import lc
lc.lc_profile(True)
for k in range(60):
    n = (k * 37 %% 250 + 1) * CHUNK + k
    w, r = pair(n, torch.float32, 0, k)
    out, cache, cache4 = lc.alloc_out(n, 3, DEV), lc.new_cache(DEV), lc.new_cache(DEV)
    want, _ = four_kernels(lc, w, r, 3, lc.alloc_out(n, 3, DEV))
    size = lc.lc_encode(w, r, 3, out)
    assert np.array_equal(out[:size].cpu().numpy(), want), k
    for turn in range(2):
        size, used = lc.lc_encode_cached_t(w, r, 3, out, cache)
        want, used4 = four_kernels(lc, w, r, 3, lc.alloc_out(n, 3, DEV), cache4)
        assert used == used4 == bool(turn) and np.array_equal(out[:size].cpu().numpy(), want) and torch.equal(cache, cache4), (k, turn)
p = lc.lc_profile_read()
given_up = p['k_hist'][1] + p['k_spec_sweep'][1]            # (waited for: the asynchronous calls are not timed)
assert given_up > 5 and given_up + p['k_encode_one'][1] == 180 and (given_up == 180 or sys.argv[1] != '-1'), p
print('same')
""" % ROOT
    env = dict(os.environ, LC_TUNE_ONE_WAIT=looks, LC_TUNE_ONE_REST="0")
    res = subprocess.run([sys.executable, "-c", code, looks], capture_output=True, text=True, env=env, cwd=ROOT, timeout=100)
    assert res.returncode == 0 and "same" in res.stdout, res.stdout[-2000:] + res.stderr[-2000:]


CROSSED = """
import sys, threading, torch, numpy as np
sys.path.insert(0, %r)
from tests.test_gpu_short_encode import pair, four_kernels, oracle_blob, CHUNK, DEV
from paper_2009_13003_amd import lc
which = sys.argv[1]
jobs = []
for k, (chunks, how) in enumerate([(40, 'wait'), (600, 'wait'), (3, 'wait'), (200, 'wait'), (700, 'async'), (12, 'wait'), (90, 'async'), (256, 'wait'), (530, 'cached'), (17, 'wait')]):
    w, r = pair(chunks * CHUNK + 11 * k, torch.float32, 0, k)
    w = r + (w - r) * 2.0 ** (3 * k - 12)                    # other buckets in every job
    want, _ = four_kernels(lc, w, r, 3, lc.alloc_out(w.numel(), 3, DEV))
    if chunks < 100:
        assert np.array_equal(want, oracle_blob(w, r, 3))
    jobs.append((w, r, how, torch.from_numpy(want).to(DEV)))
torch.cuda.synchronize()
streams = [torch.cuda.Stream() for _ in range({'one stream': 1, 'own streams': len(jobs), 'one area': 3}[which])]
if which == 'one area':
    size = lc.lc_workspace_bytes(701 * CHUNK, 3)
    area = torch.empty((size + 255) // 256 * 256, dtype=torch.uint8, device=DEV)
    lc.lc_set_workspace(area)
wrong = []

def work(i):
    w, r, how, want = jobs[i]
    out, spare = lc.alloc_out(w.numel(), 3, DEV), lc.alloc_out(w.numel(), 3, DEV)
    with torch.cuda.stream(streams[i %% len(streams)]):
        for turn in range(25):
            out.zero_()
            if how == 'wait':
                size = lc.lc_encode(w, r, 3, out)
            elif how == 'async':
                size, _ = lc.lc_encode_wait(lc.lc_encode_async_t(w, r, 3, out))
            else:
                size, _ = lc.lc_encode_cached_t(w, r, 3, out, lc.new_cache(DEV))
            if size != want.numel() or not torch.equal(out[:size], want):
                wrong.append((i, turn))

threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
[t.start() for t in threads]
[t.join() for t in threads]
assert not wrong, wrong
print('same')
"""


@pytest.mark.parametrize("which", ["one stream", "own streams", "one area"])
def test_calls_that_give_up_beside_other_threads_calls(which):
    """A call that is given up leaves counts behind in its scratch area; other threads' calls, long, asynchronous and cached ones, take the
    area before its own thread knows: on one stream, on more streams than there are areas, and in a caller's one area."""
    env = dict(os.environ, LC_TUNE_ONE_WAIT="0", LC_TUNE_ONE_REST="0")
    res = subprocess.run([sys.executable, "-c", CROSSED % ROOT, which], capture_output=True, text=True, env=env, cwd=ROOT, timeout=100)
    assert res.returncode == 0 and "same" in res.stdout, res.stdout[-2000:] + res.stderr[-2000:]
