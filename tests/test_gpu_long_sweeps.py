"""The pair sweep where one workgroup goes through many column tiles: batches with at least 1024 row blocks,
whose columns are not cut into segments.  There the row direction closes windows of 64 (bf16, d = 128) or
16 chunks inside a group, the three buffers of column candidates come round again and again, counts are
written out every 192 chunks, and with a wide window the pass after the sweep ends windows of its own and
writes its counts out after 32 and after 224 chunks more.  The same problems alone are cut into up to 16
segments, where none of that happens: both must give the same bits, and the oracle's values on sampled
rows."""
import numpy as np
import pytest

import oracle
from gpu_util import check_scores, host, mask_to_device, to_device
from paper_2608_27128_amd import binding, synth
from test_gpu_debug_build import _debug_lib, _run
from test_gpu_scorer import COUNT_MARGIN

pytestmark = pytest.mark.gpu

# (d, dtype, heads): heads * ceil(tokens / 256 or 128) >= 1024, fewer than 96 problems
CONFIGS = [(128, "bf16", 56), (64, "bf16", 56), (128, "f32", 28), (64, "f32", 28)]


def batch_of(d, dtype, H, n, w, frac=0.3):
    sp = synth.Spec(name="long", config_id=600 + d + H, n_heads=H, lens=(n,), d=d, dtype=dtype,
                    key_recipe="offset", dup_recipe="uniform", dup_frac=0.2, dup_sigma=0.02, budget_frac=frac,
                    policy_sinks=2, policy_recent=3, tau=0.9, w=w, n_sink=2, n_recent=3, seed=9)
    return synth.make_batch(sp, threads=8)


def rows_of(n, seed):
    g = np.random.default_rng(seed)
    return np.unique(np.concatenate([[0, 1, n // 2, n - 1], g.integers(0, n, 40)]))


@pytest.mark.parametrize("d,dtype,H", CONFIGS)
@pytest.mark.parametrize("w", [7, 2500])
def test_scores(d, dtype, H, w):
    n = 4800
    batch = batch_of(d, dtype, H, n, w)
    kt, rt = to_device(batch.keys, dtype), mask_to_device(batch.retained)
    many = {k: host(v) for k, v in binding.nn_scores(kt, rt, w).items()}
    for h in (0, 13, H - 1):
        alone = binding.nn_scores(kt[h:h + 1], rt[h:h + 1], w)
        for k, v in alone.items():
            if k != "status":
                assert np.array_equal(host(v)[0].view(np.int32), many[k][h].view(np.int32)), (k, h)
    for h in (0, H - 1):
        rows = rows_of(n, h)
        orc = oracle.nn_scores(batch.keys[h], dtype, batch.retained[h], w, rows=rows)
        check_scores({k: v[h] for k, v in many.items() if k != "status"}, orc, rows, batch.keys[h], dtype,
                     batch.retained[h], w)


@pytest.mark.parametrize("d,dtype,H", [(128, "bf16", 40), (64, "bf16", 40), (128, "f32", 20), (64, "f32", 20)])
@pytest.mark.parametrize("n,w", [(8000, 7), (10000, 8500)])
def test_counts(d, dtype, H, n, w):
    batch = batch_of(d, dtype, H, n, w)
    kt = to_device(batch.keys, dtype)
    many = host(binding.twin_counts(kt, 0.9, w)["counts"])
    for h in (0, H - 1):
        assert np.array_equal(host(binding.twin_counts(kt[h:h + 1], 0.9, w)["counts"])[0], many[h]), h
    for h in (0, H - 1):
        rows = rows_of(n, h)
        o = oracle.twin_counts(batch.keys[h], dtype, 0.9, w, rows=rows, margin=COUNT_MARGIN)
        assert np.all(many[h][rows] >= o["counts_lo"]) and np.all(many[h][rows] <= o["counts_hi"]), h


@pytest.mark.parametrize("d,dtype,H", CONFIGS)
def test_debug_build_matches(d, dtype, H):
    """As in the debug build's own tests, with column buffers that are used again many times."""
    batch = batch_of(d, dtype, H, 4800, 32)
    kt, rt = to_device(batch.keys, dtype), mask_to_device(batch.retained)
    dt = 0 if dtype == "bf16" else 1
    a = _run(binding.lib(), kt, rt, batch, dt)
    b = _run(_debug_lib(), kt, rt, batch, dt)
    for k in a:
        assert np.array_equal(a[k], b[k]), k
