"""Every placement of a chunk's rows in workgroups (row groups in mirrored or
adjacent pairs, one group per workgroup, or the short kernel's 32-row slots
whose wavefronts share the keys), forced through MOCAP_PAIRING, against the
oracle: rows at and around 32 and 128 for several group sizes, keys at and
around the steps of 32 and the tiles of 64, ranges that end inside a chunk,
unwritten store memory full of NaN, and the overflow rescale."""
import pytest
import torch

from helpers import check_chunks, run_gpu, say
from paper_2606_22968_amd import synth
from paper_2606_22968_amd.prefill import ChunkedPrefill

pytestmark = pytest.mark.gpu

PLACEMENTS = ["mirrored", "adjacent", "single", "short"]


@pytest.mark.parametrize("placement", PLACEMENTS)
@pytest.mark.parametrize("h_q,h_kv,d,lengths", [
    (4, 1, 128, [8, 1, 7, 9, 33, 31, 32, 65]),   # 32, 4, 28, 36, 132, 124, 128, 260 rows
    (3, 1, 64, [11, 10, 43, 22, 64, 86, 1]),     # rows off every multiple of 32
    (5, 5, 128, [1, 31, 32, 33, 127, 32, 129]),  # one head per KV head
    (64, 1, 64, [1, 2, 3, 40]),                  # a token's heads over two slots
    (40, 1, 128, [1, 3, 70]),                    # groups that share a slot with the next token's
])
@pytest.mark.parametrize("splits", [1, 3, 0])
def test_rows_and_keys_at_edges(gpu, oracle_lib, monkeypatch, placement, h_q, h_kv, d, lengths, splits):
    monkeypatch.setenv("MOCAP_PAIRING", placement)
    say(f"[case] placement={placement} h_q={h_q} h_kv={h_kv} d={d} splits={splits}")
    q, k, v = synth.make_qkv(70 + h_q, sum(lengths), h_q, h_kv, d)
    scale = d ** -0.5
    runner = run_gpu(q, k, v, lengths, scale, block_size=64, num_splits=splits, pool_fill=float("nan"))
    check_chunks(oracle_lib, runner, q, k, v, scale, label=f"{placement} splits={splits}")


@pytest.mark.parametrize("placement", PLACEMENTS)
@pytest.mark.parametrize("h_q,h_kv,d,lengths", [
    (4, 2, 128, [1100, 5, 17, 700]),
    (16, 2, 64, [1000, 13, 130]),
])
def test_even_ranges_two_stores(gpu, oracle_lib, monkeypatch, placement, h_q, h_kv, d, lengths):
    """Automatic plans, with and without a second store: the same bits."""
    monkeypatch.setenv("MOCAP_PAIRING", placement)
    q, k, v = synth.make_qkv(80 + h_q, sum(lengths), h_q, h_kv, d)
    scale = d ** -0.5
    one = run_gpu(q, k, v, lengths, scale, block_size=128, pool_fill=float("nan"))
    say(f"[case] placement={placement} splits={one.splits}")
    check_chunks(oracle_lib, one, q, k, v, scale, label=f"{placement} {one.splits}")
    two = run_gpu(q, k, v, lengths, scale, runner=ChunkedPrefill(
        h_q, h_kv, d, lengths, block_size=128, pool_fill=float("nan"), remote=(128, 960)))
    assert two.splits == one.splits
    assert torch.equal(one.o.view(torch.int16), two.o.view(torch.int16))


@pytest.mark.parametrize("d", [64, 128])
def test_short_kernel_overflow_rescale(gpu, oracle_lib, monkeypatch, d):
    """Scores that grow by more than 60 binary orders from step to step."""
    monkeypatch.setenv("MOCAP_PAIRING", "short")
    lengths = [600, 40]
    q, k, v = synth.make_qkv(91, sum(lengths), 4, 1, d)
    q[:, :, 0] = 8.0
    for at, grow in ((10, 8.0), (45, 80.0), (300, 160.0), (310, 240.0), (630, 320.0)):
        k[at, :, 0] = grow
    scale = d ** -0.5 if d == 64 else 0.125
    for splits in (1, 0):
        runner = run_gpu(q, k, v, lengths, scale, block_size=64, num_splits=splits)
        check_chunks(oracle_lib, runner, q, k, v, scale, label=f"rescale d={d} splits={splits}")
