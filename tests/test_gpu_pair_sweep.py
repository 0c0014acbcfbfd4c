"""The pair sweep (every unordered pair once, reduced into both tokens) at the edges of its tiling:
row blocks of 128 or 256 slots, 128-slot group alignment, 32-slot chunks, column segments (few row
blocks) and the XCD-affine order (>= 8
heads).  Scores and counts against the oracle; the S0-only sweep against the pair sweep.  Many short problems,
which take the full rectangle, against the same problems a few at a time."""
import numpy as np
import pytest

from gpu_util import host, mask_to_device, to_device
from paper_2608_27128_amd import binding, synth
from test_gpu_parity import masks_for, run_and_check, small_spec
from test_gpu_scorer import check_counts

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 127, 128, 129, 255, 256, 257, 385, 641]
CASES = [
    # (heads, lens, w, mask)
    (1, EDGES, 0, "policy"),
    (9, EDGES, 40, "policy"),
    (2, [513, 2049 + 64], 7, "policy"),     # (windows of chunks are crossed in test_gpu_long_sweeps.py)
    (1, [2500], 1200, "policy"),            # the window reaches over most row blocks
    (2, [300, 640], 3, "one"),
    (2, [300, 640], 3, "all"),
]


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "f32"), (128, "f32")])
@pytest.mark.parametrize("H,lens,w,kind", CASES)
def test_edges(H, lens, w, kind, d, dtype):
    batch = synth.make_batch(small_spec(H, lens, d, dtype, w, 71 + len(lens), dup_frac=0.3))
    gpu, _ = run_and_check(batch, w, kind, seed=5)
    kt = to_device(batch.keys, dtype)
    counts = host(binding.twin_counts(kt, 0.9, w, batch.cu_seqlens)["counts"])
    check_counts(batch, counts, 0.9, w)
    # the S0 columns alone give the same bits
    rt = mask_to_device(masks_for(kind, batch, 5))
    lean = binding.repair(kt, rt, batch.budget, 0.9, w, 2, 3, batch.cu_seqlens, want_all=False)
    for k in ("best_ret", "arg_ret"):
        assert np.array_equal(host(lean[k]), gpu[k]), k


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "f32"), (128, "f32")])
@pytest.mark.parametrize("with_s0", [False, True])
def test_infinite_element_names_only_tokens(d, dtype, with_s0):
    """With positive keys, an infinite element gives +Inf against every token and NaN against the
    zeros that fill the last tile past the list's end.  The scores of that problem are unspecified, but
    a reported position is one of its tokens, whatever the workspace holds past its column list."""
    import torch
    lens = [40, 300, 33]
    cu = np.concatenate([[0], np.cumsum(lens)])
    g = np.random.default_rng(d + with_s0)
    keys = (0.5 + g.random((2, cu[-1], d))).astype(np.float32)
    for h, s in ((0, 0), (1, 1), (1, 2)):
        keys[h, cu[s] + 5, 7] = np.inf
    kt = torch.from_numpy(keys).cuda()
    kt = kt.to(torch.bfloat16) if dtype == "bf16" else kt
    ret = torch.from_numpy((g.random((2, cu[-1])) < 0.5).astype(np.uint8)).cuda() if with_s0 else None
    nb = binding.workspace_bytes(binding.OP_NN_SCORES, 0 if dtype == "bf16" else 1, d, 2, cu)
    ws = torch.full((nb,), 0x7F, dtype=torch.uint8, device="cuda")
    out = {k: host(v) for k, v in binding.nn_scores(kt, ret, 3, cu, workspace=ws).items()}
    assert list(out["status"]) == [2, 0, 0, 0, 2, 2]
    for k in ("arg_all", "arg_ret") if with_s0 else ("arg_all",):
        for s, n in enumerate(lens):
            a = out[k][:, cu[s]:cu[s + 1]]
            assert a.min() >= -1 and a.max() < n, (k, s)


# (heads, lengths) of many problems, in the range that the rectangle sweeps: its row blocks hold 384 (512,
# 128) tokens, its tiles 128 (64) columns
MANY = {(128, "bf16"): (20, [1, 31, 33, 97, 255, 383, 384, 385, 641, 129]),
        (64, "bf16"): (40, [1, 31, 33, 97, 255, 511, 512, 513, 641, 129]),
        (128, "f32"): (20, [1, 31, 33, 40, 127, 128, 129, 64, 50, 60]),
        (64, "f32"): (20, [1, 31, 33, 97, 127, 128, 129, 60, 40, 64])}


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "f32"), (128, "f32")])
@pytest.mark.parametrize("kind,w", [("policy", 0), ("policy", 20), ("one", 3), ("all", 7), (None, 200)])
def test_many_short_problems_equal_few(d, dtype, kind, w):
    """A batch of many short problems goes over the full rectangle, the same problems a few at a time
    over the pairs: the same bits, and the oracle's values."""
    H, lens = MANY[d, dtype]
    batch = synth.make_batch(small_spec(H, lens, d, dtype, w, 91 + len(lens), dup_frac=0.3))
    kt = to_device(batch.keys, dtype)
    ret = None if kind is None else masks_for(kind, batch, 5)
    rt = None if ret is None else mask_to_device(ret)
    many = {k: host(v) for k, v in binding.nn_scores(kt, rt, w, batch.cu_seqlens).items()}
    for h in (0, 7, H - 1):
        few = binding.nn_scores(kt[h:h + 1], None if rt is None else rt[h:h + 1], w, batch.cu_seqlens)
        for k, v in few.items():
            if k != "status":
                assert np.array_equal(host(v)[0].view(np.int32), many[k][h].view(np.int32)), (k, h)
    run_and_check(batch, w, kind, seed=5)


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "f32"), (128, "f32")])
@pytest.mark.parametrize("tau,w", [(0.9, 0), (0.3, 20), (-0.1, 5)])
def test_many_short_problems_counts(d, dtype, tau, w):
    """(bf16: over the rectangle)"""
    lens = [1, 31, 33, 64, 200, 129]
    batch = synth.make_batch(small_spec(32, lens, d, dtype, w, 95 + len(lens), dup_frac=0.3))
    counts = host(binding.twin_counts(to_device(batch.keys, dtype), tau, w, batch.cu_seqlens)["counts"])
    check_counts(batch, counts, tau, w)


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "f32")])
@pytest.mark.parametrize("lens", [(1024, 0, 257, 1), (1023, 255, 256), (1025, 3), (512,), (40,)])
def test_repair_from_candidates(d, dtype, lens):
    """Up to 1024 tokens the repair kernel itself turns the pair sweep's candidates into results: the
    scores' bits, and the repair of those scores, whichever outputs are asked for."""
    batch = synth.make_batch(small_spec(3, list(lens), d, dtype, 5, 400 + len(lens), dup_frac=0.3))
    cu = batch.cu_seqlens
    kt, rt = to_device(batch.keys, dtype), mask_to_device(batch.retained)
    sc = binding.nn_scores(kt, rt, 5, cu)
    want = binding.repair_from_scores(sc["best_ret"], rt, batch.budget, 0.9, 2, 3, cu)
    out = binding.repair(kt, rt, batch.budget, 0.9, 5, 2, 3, cu)
    some = {k: v.clone().fill_(0) for k, v in out.items() if k in ("s1", "stats", "best_all")}
    some = binding.repair(kt, rt, batch.budget, 0.9, 5, 2, 3, cu, outputs=some)
    assert sorted(some) == ["best_all", "s1", "stats"]
    for k in ("best_ret", "arg_ret", "best_all", "arg_all"):
        assert np.array_equal(host(out[k]).view(np.int32), host(sc[k]).view(np.int32)), k
    for k in ("s1", "stats"):
        assert np.array_equal(host(out[k]), host(want[k])), k
        assert np.array_equal(host(some[k]), host(want[k])), k
    assert np.array_equal(host(some["best_all"]), host(sc["best_all"]))
    inplace = rt.clone()
    binding.repair(kt, inplace, batch.budget, 0.9, 5, 2, 3, cu, out_mask=inplace)
    assert np.array_equal(host(inplace), host(want["s1"]))
