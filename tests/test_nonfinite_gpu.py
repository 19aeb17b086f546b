"""NaN and infinite inputs: every placement of a chunk's rows, unsplit and
split, gives NaN (O and LSE) on exactly the rows on which the oracle does, and
the values of finite inputs on all others."""
import numpy as np
import pytest
import torch

from helpers import LSE_MAX_ABS, O_MAX_ABS, oracle_chunk, run_gpu, say
from paper_2606_22968_amd import synth

pytestmark = pytest.mark.gpu

H_Q, H_KV = 8, 2
LENGTHS = [300, 45]


def _plant(what, q, k, v):
    """Changes the inputs; returns the first chunk whose O is compared (a hidden V
    shares tiles with visible ones, and 0 * NaN is NaN there)."""
    nan, inf = float("nan"), float("inf")
    if what == "query_row":
        q[7, 3] = nan
        q[299, 0] = nan
        q[320, 7] = nan
    elif what == "only_visible_key":
        k[0, 0] = nan
    elif what == "a_wavefronts_keys":
        k[64:96, 1] = nan
    elif what == "last_key":
        k[344, 0, 5] = nan
    elif what == "infinite_key":  # a score of +inf where Q is positive, of -inf where it is negative
        k[100, 1, 9] = inf
    elif what == "value":
        v[100, 0, 6] = nan
        v[210, 1, 2] = inf
        return 1
    return 0


@pytest.mark.parametrize("placement", ["mirrored", "adjacent", "single", "short"])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("what", ["query_row", "only_visible_key", "a_wavefronts_keys", "last_key", "infinite_key",
                                  "value"])
def test_nonfinite_inputs_reach_the_rows_that_see_them(gpu, oracle_lib, monkeypatch, placement, splits, d, what):
    monkeypatch.setenv("MOCAP_PAIRING", placement)
    say(f"[case] {what} placement={placement} splits={splits} d={d}")
    q, k, v = synth.make_qkv(110, sum(LENGTHS), H_Q, H_KV, d)
    first = _plant(what, q, k, v)
    scale = d ** -0.5
    runner = run_gpu(q, k, v, LENGTHS, scale, block_size=64, num_splits=splits)
    assert runner.splits[1] == splits
    for c in range(first, len(LENGTHS)):
        p, n = runner.prefixes[c], LENGTHS[c]
        ref_o, ref_lse = oracle_chunk(oracle_lib, q, k, v, p, n, scale)
        for got, want, bar in ((runner.o[p:p + n].cpu(), ref_o, O_MAX_ABS), (runner.lse(c).cpu(), ref_lse, LSE_MAX_ABS)):
            got = got.double().numpy()
            assert np.array_equal(np.isnan(got), np.isnan(want)), f"chunk {c}: {np.isnan(got).sum()} NaN, " \
                f"{np.isnan(want).sum()} expected"
            assert np.array_equal(np.isinf(got), np.isinf(want))
            finite = np.isfinite(want)
            assert np.abs(got[finite] - want[finite]).max(initial=0.0) <= bar


def test_a_short_first_chunk_planned_by_the_library(gpu):
    """256 tokens (always unsplit, the short kernel): one NaN query row, no zeros."""
    q, k, v = synth.make_qkv(111, 256, 8, 8, 64)
    q[100, 2] = float("nan")
    runner = run_gpu(q, k, v, [256], 0.125)
    bad = torch.zeros(256, 8, dtype=torch.bool)
    bad[100, 2] = True
    assert torch.equal(torch.isnan(runner.o.cpu()).all(-1), bad) and torch.equal(torch.isnan(runner.o.cpu()).any(-1), bad)
    assert torch.equal(torch.isnan(runner.lse(0).cpu()), bad.t())


@pytest.mark.parametrize("splits", [2, 70])
def test_merge_of_nan_partials(gpu, splits):
    """NaN keys in one range only: NaN, whatever the other ranges hold."""
    q, k, v = synth.make_qkv(112, 4500, 4, 1, 128)
    k[1000:1064] = float("nan")
    runner = run_gpu(q, k, v, [4490, 10], 128 ** -0.5, block_size=64, num_splits=splits)
    assert runner.splits[1] == splits
    assert torch.isnan(runner.o[4490:]).all() and torch.isnan(runner.lse(1)).all()
