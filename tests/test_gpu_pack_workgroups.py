"""Sweep 2 by workgroups, against the oracle's blobs byte for byte: chunks whose strings fit the workgroup's areas beside
chunks that outgrow them, quiet chunks and quiet 4 KiB parts, ragged ends, on both sides of the number of chunks from which
the chunks to read are listed, from the inputs and from staged keys."""
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


def mixed(n, dtype, offset, seed):
    """Ordinary chunks; chunk 1 rare binades only (its payload does not fit), chunk 2 rare ones in the first lanes of a few
    rows (one part does not fit), chunk 3 quiet, chunk 4 quiet but for one row."""
    g = torch.Generator(device=DEV); g.manual_seed(seed)
    i = torch.arange(n, device=DEV)
    c, row, lane = i // 16384, (i // 256) % 64, (i // 4) % 64
    e = torch.floor(-torch.log2(torch.rand(n, generator=g, device=DEV).clamp_(min=2.0 ** -13)))
    rare = torch.randint(8, 13, (n,), generator=g, device=DEV).float()
    e = torch.where((c == 1) | ((c == 2) & (row < 8) & (lane < 2)), rare, e)
    d = torch.exp2(e - 20) * (1 + 0.5 * torch.rand(n, generator=g, device=DEV))        # rare = large exponent
    d = torch.where((c == 3) | ((c == 4) & (row != 37)), torch.zeros_like(d), d)
    w, ref = torch.empty(n + offset, device=DEV, dtype=dtype), torch.zeros(n + offset, device=DEV, dtype=dtype)
    w[offset:] = d.to(dtype)
    return w[offset:], ref[offset:]


def oracle_blob(w, ref, nbits):
    if w.dtype == torch.float32:
        return orc.encode(w.cpu().numpy(), ref.cpu().numpy(), nbits)
    raw = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)
    return orc.encode_t(raw(w), raw(ref), nbits, orc.DT_BF16)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("nbits", [2, 4])
@pytest.mark.parametrize("n,offset", [(5 * 16384, 0), (5 * 16384 + 1029, 0), (5 * 16384 + 255, 1), (2048 * 16384, 0), (2049 * 16384 + 3, 0)])
def test_chunks_that_fit_and_chunks_that_do_not(lc, dtype, nbits, n, offset):
    print("workgroups", dtype, nbits, n, offset, flush=True)
    w, ref = mixed(n, dtype, offset, n + nbits)
    want = oracle_blob(w, ref, nbits)
    out = lc.alloc_out(n, nbits, DEV)
    for staging in ([lc.STAGING_NEVER, lc.STAGING_ALWAYS] if dtype == torch.float32 else [lc.STAGING_AUTO]):
        lc.lc_set_option(lc.OPT_KEY_STAGING, staging)
        try:
            out.fill_(0xA5)
            size = lc.lc_encode_t(w, ref, nbits, out)
        finally:
            lc.lc_set_option(lc.OPT_KEY_STAGING, lc.STAGING_AUTO)
        assert size == want.size and np.array_equal(out[:size].cpu().numpy(), want), staging
    out.fill_(0xA5)
    half = 3 * 16384 + 77                              # the same again as two tensors with a table each
    outs = [lc.alloc_out(half, nbits, DEV), out]
    sizes = lc.lc_encode_batch([w[:half], w], [ref[:half], ref], nbits, outs)
    assert np.array_equal(outs[0][:sizes[0]].cpu().numpy(), oracle_blob(w[:half], ref[:half], nbits))
    assert sizes[1] == want.size and np.array_equal(out[:sizes[1]].cpu().numpy(), want)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n,offset", [(5 * 16384 + 1029, 0), (5 * 16384 + 255, 1), (600 * 16384, 0), (2 * 2048 * 16384 + 3, 0)])
def test_behind_a_cache_that_does_not_hold(lc, dtype, n, offset):
    """An empty cache, and one of other data: the sweep in which a workgroup may take several chunks (the largest), again and again on
    the scratch area that the call before has left, against the plain encode's blob, which has a sweep 2 of its own."""
    nbits = 4
    print("cache", dtype, n, offset, flush=True)
    w, ref = mixed(n, dtype, offset, n)
    other = (w.float() * 2.0 ** -7).to(dtype)
    out = lc.alloc_out(n, nbits, DEV)
    plain = {}
    for name, x in (("w", w), ("other", other)):
        size, _ = lc.lc_encode_wait(lc.lc_encode_async_t(x, ref, nbits, out))
        plain[name] = out[:size].clone()
    if n < 10 * 16384 and dtype != torch.float16:
        assert np.array_equal(plain["w"].cpu().numpy(), oracle_blob(w, ref, nbits))
    for turn in range(4):
        cache = lc.new_cache(DEV)
        for name, x in (("w", w), ("other", other), ("w", w)):
            out.fill_(0xA5)
            size, used = lc.lc_encode_wait(lc.lc_encode_async_t(x, ref, nbits, out, cache=cache))
            assert not used and torch.equal(out[:size], plain[name]), (turn, name)
