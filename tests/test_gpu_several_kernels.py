"""The kernels of longer vectors on the small ones that other tests try them with: a vector of up to two chunks per compute unit
is encoded and restored in one launch, and several files' edge cases (rings, lanes at different rates, chunks of few kept
symbols, payloads that overflow their area, quiet chunks and parts) were written for the kernels that take over beyond that, or
where such a call is given up.  Here they run once more in a process with that route switched off."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import sys
import torch
sys.path.insert(0, %r)
from paper_2009_13003_amd import lc
ref = torch.zeros(5 * 16384 + 3, device="cuda:0")
w = torch.exp2(-torch.arange(ref.numel(), device="cuda:0") %% 9.0)
out = lc.alloc_out(ref.numel(), 3, "cuda:0")
lc.lc_profile(True)
blob = out[:lc.lc_encode(w, ref, 3, out)].clone()
lc.lc_encode_cached(w, ref, 3, out, lc.new_cache("cuda:0"))
lc.lc_decode(blob, ref.clone())
lc.lc_decode_many([blob, blob], ref.clone())
ran = {k for k, v in lc.lc_profile_read().items() if v[1]}
lc.lc_profile(False)
assert {"k_hist", "k_pack", "k_place", "k_spec_sweep", "k_decode", "k_decode_fused"} <= ran and not {"k_encode_one", "k_decode_one"} & ran, ran
import pytest
rc = pytest.main(["-x", "-q", "-m", "gpu", "-p", "no:cacheprovider", "--timeout", "100", "--timeout-method", "thread"] + sys.argv[1:])
print("child's tests:", int(rc), flush=True)
sys.exit(int(rc))
"""


@pytest.mark.parametrize("args", [
    ["tests/test_gpu_restore_steps.py", "tests/test_gpu_sparse_restore.py", "tests/test_gpu_pack_workgroups.py", "tests/test_gpu_code_table.py"],
    ["tests/test_gpu_parity.py", "-k", "fused_restore or checkpoint_chain or seeded or verify or verifies or damaged"],
    ["tests/test_gpu_parity.py", "-k", "sizes_and_bit or unaligned or degenerate or symbol or heterogeneous or quiet or below or merged or long"],
    ["tests/test_gpu_parity.py", "-k", "16_bit or bf16 or fp64 or cached or nonfinite or threads"],
    ["tests/test_gpu_short_encode.py", "tests/test_gpu_short_decode.py", "-k", "not give_up and not by_what_the_check_finds"],
], ids=["restores", "fused", "chunks", "types", "short"])
def test_with_the_one_launch_route_off(args):
    env = dict(os.environ, LC_TUNE_ONE_PER_CU="0", LC_TUNE_ONE_DEC_PER_CU="0")
    res = subprocess.run([sys.executable, "-c", CHILD % ROOT] + args, capture_output=True, text=True, env=env, cwd=ROOT, timeout=110)
    assert res.returncode == 0 and "child's tests: 0" in res.stdout, res.stdout[-3000:] + res.stderr[-2000:]
