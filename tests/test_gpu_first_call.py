"""A process pays for loading the attention kernels in its first attention call:
the first draft after a verify finds its code on the GPU."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.gpu

SCRIPT = """
import time, torch
import paper_2408_11049_amd as md
B, S, Hkv, G, d = 64, 8192, 8, 4, 128
k = torch.zeros((B, S, Hkv, d), dtype=torch.bfloat16, device="cuda:0")
q = torch.zeros((B, 5, Hkv * G, d), dtype=torch.bfloat16, device="cuda:0")
n = torch.full((B,), S, dtype=torch.int32, device="cuda:0")
out, lse = torch.empty_like(q), torch.empty((B, 5, Hkv * G), device="cuda:0")
kw = dict(max_kv_len=S, out=out, lse=lse)
calls = [lambda: md.md_verify_attn(q, k, k, n, **kw), lambda: md.md_draft_attn(q, k, k, n, 16, 496, **kw)]
calls[FIRST]()
torch.cuda.synchronize()
t = time.perf_counter()
calls[1 - FIRST]()
torch.cuda.synchronize()
print("second call ms", (time.perf_counter() - t) * 1e3)
"""


@pytest.mark.parametrize("first", [0, 1], ids=["verify_then_draft", "draft_then_verify"])
def test_second_kind_of_call_loads_no_code(first):
    """The balanced verify of two row tiles and the drafts come from two code
    objects.  Loading the drafts' takes 4.3 ms (6 in a larger process), the
    calls 0.1-0.4: whichever comes second ends well before a load would."""
    best = float("inf")
    for _ in range(3):  # a busy host can delay any one process
        r = subprocess.run([sys.executable, "-c", SCRIPT.replace("FIRST", str(first))], cwd=ROOT,
                           capture_output=True, text=True, timeout=100,
                           env={**os.environ, "PYTHONPATH": ROOT})
        assert r.returncode == 0, r.stderr[-2000:]
        best = min(best, float(r.stdout.split()[-1]))
        print(f"[first call] {best:.2f} ms", flush=True)
        if best < 2.5:
            return
    assert False, f"the second kind of call took {best:.2f} ms"
