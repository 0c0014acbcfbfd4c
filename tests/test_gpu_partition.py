"""The partition into S0 and evicted column lists at the edges of its kernels: rounds of 256 tokens,
4 rounds (no sequence over 1024 tokens), 16 rounds (4096) and the slab-by-slab kernel beyond."""
import pytest

from test_gpu_parity import run_and_check, small_spec
from paper_2608_27128_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [(1, 255, 256, 257), (1023, 1024, 0), (1025, 64), (4096, 3), (4097, 256)])
@pytest.mark.parametrize("kind", ["policy", "one"])
def test_partition_edges(lens, kind):
    batch = synth.make_batch(small_spec(2, list(lens), 64, "bf16", 4, 300 + len(lens) + lens[0] % 7))
    run_and_check(batch, 4, kind, seed=3)


@pytest.mark.parametrize("n_seqs", [15, 16, 17])
def test_table_edges(n_seqs):
    """Up to 16 sequences the table goes with the partition, beyond that it is uploaded first."""
    lens = [37 * (s + 1) % 101 for s in range(n_seqs - 1)] + [700]
    batch = synth.make_batch(small_spec(9, lens, 64, "bf16", 4, 320 + n_seqs))
    run_and_check(batch, 4, "policy", seed=3)
