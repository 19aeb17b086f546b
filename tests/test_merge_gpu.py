"""Merging split partials: one range count below, at and above each step of
the merge kernel (parts of a wavefront, loads in flight, 64 ranges at a time)."""
import pytest

from helpers import check_chunks, run_gpu, say
from paper_2606_22968_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_q,h_kv,d", [(4, 1, 128), (3, 3, 64)])
@pytest.mark.parametrize("splits", [2, 3, 5, 9, 17, 63, 64, 65, 129, 1000])
def test_merge_any_range_count(gpu, oracle_lib, splits, h_q, h_kv, d):
    lengths = [8300, 5]  # 130 prefix tiles behind the second chunk
    say(f"[case] merge splits={splits} h_q={h_q} h_kv={h_kv} d={d}")
    q, k, v = synth.make_qkv(90, sum(lengths), h_q, h_kv, d)
    scale = d ** -0.5
    runner = run_gpu(q, k, v, lengths, scale, block_size=64, num_splits=splits)
    assert runner.splits[1] == min(splits, 131)
    check_chunks(oracle_lib, runner, q, k, v, scale, rows_of=lambda c, n: [0, 1, 4], label=f"splits={splits}")


@pytest.mark.parametrize("length", [128, 129])
def test_merge_few_and_many_rows(gpu, oracle_lib, length):
    """512 and 516 (token, head) rows: both sides of the loads-ahead rule."""
    q, k, v = synth.make_qkv(92, 2048 + length, 4, 2, 64)
    runner = run_gpu(q, k, v, [2048, length], 0.125, block_size=64, num_splits=21)
    check_chunks(oracle_lib, runner, q, k, v, 0.125, rows_of=lambda c, n: [0, 1, 63, n - 1], label=f"rows={4 * length}")


@pytest.mark.parametrize("h_q,h_kv,d", [(4, 1, 128), (4, 4, 64)])
@pytest.mark.parametrize("splits", [63, 64, 65, 129])
def test_merge_many_rows_of_many_ranges(gpu, oracle_lib, splits, h_q, h_kv, d):
    """520 rows: the loads of many rows, below, at and above 64 ranges at a time."""
    q, k, v = synth.make_qkv(93, 8300 + 130, h_q, h_kv, d)
    runner = run_gpu(q, k, v, [8300, 130], d ** -0.5, block_size=64, num_splits=splits)
    assert runner.splits[1] == splits
    check_chunks(oracle_lib, runner, q, k, v, d ** -0.5, rows_of=lambda c, n: [0, 1, 63, 64, n - 1],
                 label=f"rows=520 splits={splits}")
