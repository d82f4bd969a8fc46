"""The split-KV merge done inside the attention launch (MD_FUSED_MERGE = 1):
when a unit's range is cut into chunks, the last workgroup of each head group
to finish merges the chunks' partials by log-sum-exp (the split-KV identity,
paper Sec. 2).  Its arrival counters live in the caller's workspace and carry
a per-call tag, so the workspace needs no clearing: these tests hand the
kernels workspaces full of garbage (including values shaped like counters of
other calls), reuse one workspace across calls of different plans, and check
every result against the fp64 oracle -- for the fused merge and for the
default second launch alike."""
import numpy as np
import pytest
import torch

import oracle
import paper_2408_11049_amd as md
from gpu_util import TOL, compare, run_oracle, say
from paper_2408_11049_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _case(B, L, Hq, Hkv, lens, page, seed):
    return wl.make_case(B=B, q_len=L, Hq=Hq, Hkv=Hkv, d=128, kv_lens=lens, dtype="bf16",
                        page_size=page, seed=seed, device=DEV,
                        S_alloc=None if page else max(lens) + 5)


def _call(mode, c, ws, n_sink=0, window=1):
    out = torch.full_like(c["q"], float("nan"))
    lse = torch.full(c["q"].shape[:3], float("nan"), dtype=torch.float32, device=DEV)
    kw = dict(max_kv_len=c["max_kv_len"], page_table=c["page_table"], out=out, lse=lse,
              workspace=ws)
    if mode == oracle.VERIFY:
        md.md_verify_attn(c["q"], c["k"], c["v"], c["kv_lens"], **kw)
    else:
        md.md_draft_attn(c["q"], c["k"], c["v"], c["kv_lens"], n_sink, window, **kw)
    torch.cuda.synchronize()
    return out.float().cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)


def _need(mode, c, n_sink=0, window=1):
    return md.md_workspace_bytes(c["q"], c["k"], c["v"], c["kv_lens"], mode=mode, n_sink=n_sink,
                                 window=window, max_kv_len=c["max_kv_len"],
                                 page_table=c["page_table"])


@pytest.fixture(params=["fused", "launch"])
def merge(request, monkeypatch):
    monkeypatch.delenv("MD_FUSED_MERGE", raising=False)
    if request.param == "fused":
        monkeypatch.setenv("MD_FUSED_MERGE", "1")
    return request.param


@pytest.mark.parametrize("fill", ["ones", "random", "foreign_tags"])
def test_garbage_workspace(fill, merge):
    """A split verify and a split draft over a workspace that starts as
    garbage: all bits set, random bytes, or counters tagged by other calls
    with arrival counts just below the chunk count."""
    c = _case(1, 4, 8, 2, [20000], 16, 301)
    for mode, n_sink, window in ((oracle.VERIFY, 0, 1), (oracle.DRAFT, 16, 4000)):
        need = _need(mode, c, n_sink, window)
        assert need > 0, "the case must split its range"
        ws = torch.empty(need, dtype=torch.uint8, device=DEV)
        if fill == "ones":
            ws.fill_(0xFF)
        elif fill == "random":
            g = torch.Generator(device=DEV)
            g.manual_seed(5)
            ws.copy_(torch.randint(0, 256, (need,), generator=g, device=DEV, dtype=torch.uint8))
        else:
            # (tag << 16) | arrivals, with tags no call of this process uses
            words = ws[: need // 8 * 8].view(torch.int64)
            i = torch.arange(words.numel(), device=DEV, dtype=torch.int64)
            words.copy_(((0x7FFF0000 + i) << 16) + i % 7)
        say(f"[split-merge] {merge} {fill} mode {mode} workspace {need} B")
        got = _call(mode, c, ws, n_sink, window)
        compare(*got, *run_oracle(mode, c, n_sink, window), "bf16", f"{fill} mode {mode}")


def test_one_workspace_across_plans(merge):
    """One workspace, sized for the largest, serves calls whose plans differ
    in groups and chunks, in an interleaved order, twice over."""
    cases = [
        (oracle.VERIFY, _case(1, 4, 8, 2, [20000], 16, 311), 0, 1),
        (oracle.VERIFY, _case(2, 5, 16, 2, [9000, 3000], 0, 312), 0, 1),
        (oracle.DRAFT, _case(1, 4, 8, 2, [20000], 16, 311), 16, 4000),
        (oracle.DRAFT, _case(3, 1, 8, 2, [6000, 7000, 2500], 0, 313), 4, 2000),
    ]
    needs = [_need(m, c, s, w) for m, c, s, w in cases]
    assert all(n > 0 for n in needs)
    ws = torch.empty(max(needs), dtype=torch.uint8, device=DEV)
    refs = [run_oracle(m, c, s, w) for m, c, s, w in cases]
    for rep in range(2):
        for i, (m, c, s, w) in enumerate(cases):
            say(f"[split-merge] {merge} reuse pass {rep} case {i}")
            compare(*_call(m, c, ws, s, w), *refs[i], "bf16", f"reuse {rep}/{i}")


def test_fused_matches_separate_merge(monkeypatch):
    """The in-launch merge (MD_FUSED_MERGE = 1) and the separate merge launch
    agree with the oracle and with each other to within rounding."""
    c = _case(2, 5, 32, 8, [30000, 17000], 16, 321)
    ref = run_oracle(oracle.VERIFY, c)
    monkeypatch.setenv("MD_FUSED_MERGE", "1")
    fused = _call(oracle.VERIFY, c, None)
    monkeypatch.delenv("MD_FUSED_MERGE")
    sep = _call(oracle.VERIFY, c, None)
    compare(*fused, *ref, "bf16", "fused")
    compare(*sep, *ref, "bf16", "separate")
    d = float(np.max(np.abs(fused[0] - sep[0])))
    say(f"  fused vs separate: max|dO| = {d:.3e}")
    assert d <= TOL["bf16"] / 4


# Ranges at the edges of the split (512 tokens stay whole; chunks of 128) and
# merges of 2 to 126 parts: Hkv, Hq, L, lens, d, dtype.
EDGES = [(1, 4, 4, [511], 64, "f32"), (1, 4, 4, [512], 128, "bf16"), (1, 4, 4, [513], 128, "bf16"),
         (2, 8, 5, [1025, 300], 64, "bf16"), (1, 4, 1, [9 * 128], 128, "bf16"),
         (1, 8, 5, [32 * 128, 5], 128, "bf16"), (1, 4, 2, [33 * 128 - 1], 64, "f32"),
         (1, 2, 3, [16001], 128, "f32"), (1, 4, 1, [16100, 1, 700], 128, "bf16")]


@pytest.mark.parametrize("case", EDGES, ids=[f"edge{i}" for i in range(len(EDGES))])
@pytest.mark.parametrize("mode", ["verify", "draft"])
def test_split_edges(case, mode):
    """Short chunks and many-part merges against the oracle (drafts: the same
    range as 3 sinks and a window)."""
    Hkv, Hq, L, lens, d, dtype = case
    lens = [max(n, L) for n in lens]
    c = wl.make_case(B=len(lens), q_len=L, Hq=Hq, Hkv=Hkv, d=d, kv_lens=lens, dtype=dtype,
                     page_size=16, seed=700 + max(lens) % 97, device=DEV)
    m, s, w = (oracle.VERIFY, 0, 1) if mode == "verify" else \
        (oracle.DRAFT, 3, max(1, max(lens) - 3 - (L - 1)))
    say(f"[split-edge] {mode} {case}")
    compare(*_call(m, c, None, s, w), *run_oracle(m, c, s, w), dtype, f"{mode} {case}")


def test_short_ranges_without_a_workspace():
    """A range of at most 1024 tokens splits when a workspace is given and runs
    unsplit without one, or with one that is too small; both match the oracle."""
    import ctypes
    lib = md.load_library()
    c = _case(1, 4, 8, 2, [1000], 16, 731)
    need = _need(oracle.VERIFY, c)
    assert need > 0
    ref = run_oracle(oracle.VERIFY, c)
    for nbytes in (None, 256, need):
        ws = None if nbytes is None else torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        out = torch.full_like(c["q"], float("nan"))
        lse = torch.full(c["q"].shape[:3], float("nan"), dtype=torch.float32, device=DEV)
        a = md.make_args(c["q"], c["k"], c["v"], c["kv_lens"], max_kv_len=c["max_kv_len"],
                         page_table=c["page_table"], out=out, lse=lse, workspace=ws)
        st = torch.cuda.current_stream().cuda_stream
        assert lib.md_verify_attn(ctypes.byref(a), st) == md.MD_OK
        torch.cuda.synchronize()
        compare(out.float().cpu().numpy().astype(np.float64),
                lse.cpu().numpy().astype(np.float64), *ref, "bf16", f"workspace {nbytes}")


# Splits that more than cover the compute units: units that leave a second round
# nearly empty (B * Hkv = 320 of 256), and 64-channel rows of three and four row
# tiles, two workgroups per compute unit.  B, Hkv, Hq, L, lens, d, page.
PAST_SLOTS = [(40, 8, 8, 1, [3000 - 25 * i for i in range(40)], 128, 16),
              (4, 8, 64, 8, [8000, 5001, 100, 7999], 64, 16),
              (4, 8, 64, 5, [16000, 9000, 15999, 40], 64, 0)]


@pytest.mark.parametrize("case", PAST_SLOTS, ids=[f"past{i}" for i in range(len(PAST_SLOTS))])
def test_splits_past_the_compute_units(case):
    B, Hkv, Hq, L, lens, d, page = case
    c = wl.make_case(B=B, q_len=L, Hq=Hq, Hkv=Hkv, d=d, kv_lens=lens, dtype="bf16", page_size=page,
                     seed=740 + B, device=DEV, S_alloc=None if page else max(lens) + 5)
    need = _need(oracle.VERIFY, c)
    say(f"[past-slots] {case[:4]} d={d} workspace {need} B")
    assert need > B * L * Hq * (d + 1) * 4, "the case must split its range"
    compare(*_call(oracle.VERIFY, c, None), *run_oracle(oracle.VERIFY, c), "bf16", str(case[:4]))


@pytest.mark.parametrize("entry", ["bare", "noalloc"])
def test_covering_units_without_a_workspace(entry):
    """320 units cover the compute units by themselves: a split that only saves
    time asks no caller for a workspace, and the entry point that allocates
    nothing runs it unsplit too."""
    import ctypes
    lib = md.load_library()
    B, Hkv, Hq, L, lens, d, page = PAST_SLOTS[0]
    c = wl.make_case(B=B, q_len=L, Hq=Hq, Hkv=Hkv, d=d, kv_lens=lens, dtype="bf16", page_size=page,
                     seed=750, device=DEV)
    assert _need(oracle.VERIFY, c) > 0
    out = torch.full_like(c["q"], float("nan"))
    lse = torch.full(c["q"].shape[:3], float("nan"), dtype=torch.float32, device=DEV)
    kw = dict(max_kv_len=c["max_kv_len"], page_table=c["page_table"], out=out, lse=lse)
    say(f"[no workspace] {entry}")
    if entry == "noalloc":
        md.md_attn_noalloc(oracle.VERIFY, c["q"], c["k"], c["v"], c["kv_lens"], **kw)
    else:
        a = md.make_args(c["q"], c["k"], c["v"], c["kv_lens"], **kw)
        st = torch.cuda.current_stream().cuda_stream
        assert lib.md_verify_attn(ctypes.byref(a), st) == md.MD_OK
    torch.cuda.synchronize()
    compare(out.float().cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64),
            *run_oracle(oracle.VERIFY, c), "bf16", f"no workspace, {entry}")


# Hkv, lens, position of the NaN key: merges of a few parts, of nine (the last
# part alone in its wave) and of 32, and cut groups of the balanced verify.
NAN_KEYS = [(1, [600], 599), (1, [600], 0), (1, [9 * 128], 9 * 128 - 1), (1, [4001], 2000),
            (8, [4700 + 7 * i for i in range(64)], 4650)]


@pytest.mark.parametrize("case", NAN_KEYS, ids=[f"nan{i}" for i in range(len(NAN_KEYS))])
def test_nan_score_reaches_the_row(case):
    """A NaN key makes its sequence's rows NaN (lse -inf), split or not."""
    Hkv, lens, at = case
    c = _case(len(lens), 1, 4 * Hkv, Hkv, lens, 0, 760)
    assert _need(oracle.VERIFY, c) > 0
    c["k"][0, at] = float("nan")
    say(f"[nan key] {Hkv} heads, {len(lens)} sequences, at {at}")
    o, lse = _call(oracle.VERIFY, c, None)
    assert np.isnan(o[0]).all() and np.isneginf(lse[0]).all()
    assert np.isfinite(o[1:]).all() and np.isfinite(lse[1:]).all()


@pytest.mark.parametrize("share", ["sixth", "longer_cache"])
def test_workspace_between_plans(share):
    """One sequence of 16384 tokens: a workspace that holds the coarse split but
    not the finer one runs the coarse one, as does the workspace of a longer
    cache, whose own need is the smaller of the two."""
    import ctypes
    lib = md.load_library()
    c = _case(1, 1, 8, 2, [16384], 16, 770)
    need = _need(oracle.VERIFY, c)
    nbytes = need // 6 if share == "sixth" else _need(
        oracle.VERIFY, _case(1, 1, 8, 2, [24000], 16, 771))
    assert nbytes < need
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    out = torch.full_like(c["q"], float("nan"))
    lse = torch.full(c["q"].shape[:3], float("nan"), dtype=torch.float32, device=DEV)
    a = md.make_args(c["q"], c["k"], c["v"], c["kv_lens"], max_kv_len=c["max_kv_len"],
                     page_table=c["page_table"], out=out, lse=lse, workspace=ws)
    say(f"[workspace between] {nbytes} of {need} B")
    assert lib.md_verify_attn(ctypes.byref(a), torch.cuda.current_stream().cuda_stream) == md.MD_OK
    torch.cuda.synchronize()
    compare(out.float().cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64),
            *run_oracle(oracle.VERIFY, c), "bf16", f"{nbytes} of {need} B")
