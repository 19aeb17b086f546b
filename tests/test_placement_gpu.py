"""Every placement of a chunk's rows in workgroups (row groups in mirrored or
adjacent pairs, one group per workgroup, or the short kernel's 32-row slots
whose wavefronts share the keys), forced through MOCAP_PAIRING, against the
oracle: rows at and around 32 and 128 for several group sizes, keys at and
around the steps of 32 and the tiles of 64, ranges that end inside a chunk,
unwritten store memory full of NaN, and the overflow rescale."""
import pytest
import torch

from helpers import check_chunks, run_gpu, say
from paper_2606_22968_amd import binding, synth
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
@pytest.mark.parametrize("splits", [1, 2, 3, 0])
def test_rows_and_keys_at_edges(gpu, oracle_lib, monkeypatch, placement, h_q, h_kv, d, lengths, splits):
    monkeypatch.setenv("MOCAP_PAIRING", placement)
    say(f"[case] placement={placement} h_q={h_q} h_kv={h_kv} d={d} splits={splits}")
    q, k, v = synth.make_qkv(70 + h_q, sum(lengths), h_q, h_kv, d)
    scale = d ** -0.5
    runner = run_gpu(q, k, v, lengths, scale, block_size=64, num_splits=splits, pool_fill=float("nan"))
    assert splits == 0 or runner.splits[-1] == min(splits, (sum(lengths[:-1]) + 63) // 64 + 1)
    check_chunks(oracle_lib, runner, q, k, v, scale, label=f"{placement} splits={splits}")


def _first_chunk_sampled(c, n):
    return [0, 1, 63, 64, n // 2, n - 1] if c == 0 else None


@pytest.mark.parametrize("placement", PLACEMENTS)
@pytest.mark.parametrize("h_q,h_kv,d,lengths", [
    (4, 2, 128, [5000, 5, 17, 33]),
    (16, 2, 64, [9001, 13, 130, 40]),
    (32, 8, 128, [9001, 7]),
    (8, 8, 64, [4000, 64, 3]),
])
def test_even_ranges_two_stores(gpu, oracle_lib, monkeypatch, placement, h_q, h_kv, d, lengths):
    """Automatic plans that are split, with one store, with two, and through the no-allocation call: the same bits."""
    monkeypatch.setenv("MOCAP_PAIRING", placement)
    S = sum(lengths)
    q, k, v = synth.make_qkv(80 + h_q, S, h_q, h_kv, d)
    scale = d ** -0.5
    one = run_gpu(q, k, v, lengths, scale, block_size=128, pool_fill=float("nan"))
    say(f"[case] placement={placement} splits={one.splits}")
    assert min(one.splits[1:]) > 2
    check_chunks(oracle_lib, one, q, k, v, scale, rows_of=_first_chunk_sampled, label=f"{placement} {one.splits}")
    two = run_gpu(q, k, v, lengths, scale, runner=ChunkedPrefill(
        h_q, h_kv, d, lengths, block_size=128, pool_fill=float("nan"), remote=(128, 960)))
    assert two.splits == one.splits
    for c, p in enumerate(one.prefixes):
        n = lengths[c]
        o, lse = torch.empty_like(one.o[p:p + n]), torch.empty_like(one.lse(c))
        binding.mocap_chunk_attn_noalloc(one.store, one.table, q[p:p + n].cuda(), p, scale, o, lse)
        torch.cuda.synchronize()
        for got_o, got_lse in ((two.o[p:p + n], two.lse(c)), (o, lse)):
            assert torch.equal(got_o.view(torch.int16), one.o[p:p + n].view(torch.int16))
            assert torch.equal(got_lse, one.lse(c))


@pytest.mark.parametrize("splits", [1, 4, 0])
@pytest.mark.parametrize("d", [64, 128])
def test_short_kernel_overflow_rescale(gpu, oracle_lib, monkeypatch, d, splits):
    """Scores that grow by more than 60 binary orders from step to step."""
    monkeypatch.setenv("MOCAP_PAIRING", "short")
    lengths = [5000, 40]
    q, k, v = synth.make_qkv(91, sum(lengths), 4, 1, d)
    q[:, :, 0] = 8.0
    for at, grow in ((10, 8.0), (45, 80.0), (300, 160.0), (310, 240.0), (3100, 280.0), (5030, 320.0)):
        k[at, :, 0] = grow
    scale = d ** -0.5 if d == 64 else 0.125
    runner = run_gpu(q, k, v, lengths, scale, block_size=64, num_splits=splits)
    assert runner.splits[1] == splits or (splits == 0 and runner.splits[1] > 1)
    check_chunks(oracle_lib, runner, q, k, v, scale, rows_of=lambda c, n: [0, 9, 10, 11, 45, 46, 309, 310, 3099, 4999]
                 if c == 0 else None, label=f"rescale d={d} splits={runner.splits}")
