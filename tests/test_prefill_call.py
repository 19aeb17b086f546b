"""mocap_chunk_prefill: a whole chunk sequence in one call gives the bits of the
calls made one by one, and ChunkedPrefill.run takes it only where the loop would
accept the same inputs."""
import ctypes

import pytest
import torch

from helpers import say
from paper_2606_22968_amd import binding, synth
from paper_2606_22968_amd.prefill import ChunkedPrefill

FAKE = 0x10000  # aligned, never dereferenced
INVALID, UNSUPPORTED, WORKSPACE = 1, 2, 3


def _call(lib, kv="", lengths=(64, 64), n_table=64, num_chunks=None, k=FAKE, h_q=32, h_kv=8, block_size=256,
          head_dim=128, scale=0.1, o=FAKE, lse=FAKE, ws=None, ws_bytes=0, num_splits=0):
    store = binding.mocap_kv_store(FAKE, FAKE, 64, block_size, 8, 128)
    arr = (ctypes.c_int32 * len(lengths))(*lengths) if lengths is not None else None
    return lib.mocap_chunk_prefill(None if kv is None else ctypes.byref(store), FAKE, n_table, arr,
                                   len(lengths or ()) if num_chunks is None else num_chunks, FAKE, k, FAKE, h_q, h_kv,
                                   head_dim, scale, o, lse, ws, ws_bytes, num_splits, None)


REFUSED = [
    (dict(kv=None), INVALID),
    (dict(block_size=100), UNSUPPORTED),
    (dict(lengths=None, num_chunks=2), INVALID),
    (dict(num_chunks=-1), INVALID),
    (dict(lengths=(-3, 5)), INVALID),
    (dict(n_table=0), INVALID),
    (dict(k=0), INVALID),
    (dict(k=FAKE + 2), INVALID),
    (dict(h_q=0), INVALID),
    # Refused by the attention, or behind a chunk that is in order.
    (dict(scale=0.0), INVALID),
    (dict(scale=float("nan")), INVALID),
    (dict(h_q=12), INVALID),
    (dict(h_kv=4), INVALID),
    (dict(head_dim=64), INVALID),
    (dict(head_dim=256), INVALID),
    (dict(o=0), INVALID),
    (dict(lse=0), INVALID),
    (dict(lse=FAKE + 4), INVALID),
    (dict(num_splits=-1), INVALID),
    (dict(num_splits=2), WORKSPACE),
    (dict(num_splits=2, ws=FAKE, ws_bytes=1024), WORKSPACE),
    (dict(num_splits=2, ws=FAKE + 8, ws_bytes=1 << 30), WORKSPACE),
    (dict(lengths=(200, -100)), INVALID),
    (dict(lengths=(64, 0, 64, 64 * 256)), INVALID),
    (dict(lengths=(64, 2**31 - 1)), INVALID),
    (dict(lengths=(64,) * 4, n_table=1, block_size=64), INVALID),
]


@pytest.mark.parametrize("kwargs,expect", REFUSED)
def test_refused_before_anything_is_enqueued(host_lib, kwargs, expect):
    before = host_lib.record_launches()
    assert _call(host_lib, **kwargs) == expect
    assert host_lib.record_launches() == before


@pytest.mark.parametrize("kwargs,launches", [
    (dict(lengths=(), num_chunks=0), 0),
    (dict(lengths=(0, 0), k=0, o=0, lse=0), 0),
    (dict(), 4),
    (dict(lengths=(64, 0, 5)), 4),
    (dict(num_splits=2, ws=FAKE, ws_bytes=1 << 30), 5),  # the second chunk's merge
])
def test_accepted(host_lib, kwargs, launches):
    before = host_lib.record_launches()
    assert _call(host_lib, **kwargs) == 0
    assert host_lib.record_launches() - before == launches


@pytest.mark.gpu
@pytest.mark.parametrize("h_q,h_kv,d,lengths,splits", [
    (8, 8, 64, [256, 256, 1, 77], 0),
    (6, 3, 128, [5, 0, 130, 700], 0),   # LSE regions off 16 bytes, an empty chunk
    (8, 2, 128, [300, 200], 3),
])
def test_one_call_equals_the_loop(gpu, h_q, h_kv, d, lengths, splits):
    say(f"[case] one call h_q={h_q} h_kv={h_kv} d={d} lengths={lengths} splits={splits}")
    S = sum(lengths)
    q, k, v = (t.cuda() for t in synth.make_qkv(95, S + 3, h_q, h_kv, d))  # more tokens than the chunks use
    runs = []
    for events in (None, [[torch.cuda.Event() for _ in range(3)] for _ in lengths]):  # events: the loop
        r = ChunkedPrefill(h_q, h_kv, d, lengths, block_size=64, num_splits=splits, pool_fill=0.0)
        r.o.fill_(float("nan"))
        assert r._one_call(q, k, v)
        r.run(q, k, v, d ** -0.5, events=events)
        torch.cuda.synchronize()
        runs.append(r)
    one, loop = runs
    assert torch.equal(one.o.view(torch.int16), loop.o.view(torch.int16))
    assert torch.equal(one.store.k_pool, loop.store.k_pool) and torch.equal(one.store.v_pool, loop.store.v_pool)
    for c in range(len(lengths)):
        assert torch.equal(one.lse(c), loop.lse(c))


@pytest.mark.gpu
def test_inputs_the_loop_refuses_stay_refused(gpu):
    r = ChunkedPrefill(8, 2, 64, [64, 64], block_size=64)
    q, k, v = (t.cuda() for t in synth.make_qkv(96, 128, 8, 2, 64))
    with pytest.raises(ValueError):
        r.run(q[:100], k, v, 0.1)                       # too few tokens
    with pytest.raises(TypeError):
        r.run(q.float(), k, v, 0.1)
    with pytest.raises(ValueError):
        r.run(q.transpose(1, 2), k, v, 0.1)             # not contiguous
    with pytest.raises(ValueError):
        r.run(q, k.view(128, 1, 128), v.view(128, 1, 128), 0.1)  # other heads
    with pytest.raises(ValueError):
        r.run(q, k, v.cpu(), 0.1)
    before = r.store.k_pool.view(torch.int16).clone(), r.store.v_pool.view(torch.int16).clone()
    with pytest.raises(binding.MocapError) as e:
        r.run(q, k, v, 0.0)
    assert e.value.status == INVALID
    r.num_splits = 3  # a plan that needs more than the workspace
    with pytest.raises(binding.MocapError) as e:
        r.run(q, k, v, 0.1)
    assert e.value.status == WORKSPACE
    for lengths in ([90, -10, 48], [-5, 5], [64, 64, 1]):
        with pytest.raises(ValueError):
            binding.mocap_chunk_prefill(r.store, r.table, lengths, q, k, v, 0.1, r.o, r._lse_flat, r.workspace)
    assert torch.equal(r.store.k_pool.view(torch.int16), before[0])
    assert torch.equal(r.store.v_pool.view(torch.int16), before[1])


@pytest.mark.gpu
@pytest.mark.parametrize("owner,name", [
    (ChunkedPrefill, "append"), (ChunkedPrefill, "attend"), (ChunkedPrefill, "lse"),
    (binding, "mocap_kv_append"), (binding, "mocap_chunk_attn"), (None, "attend"),
])
def test_replaced_calls_are_made(gpu, monkeypatch, owner, name):
    """A wrapper around a method (of the class or of one object) or around a call of the binding sees every chunk."""
    r = ChunkedPrefill(8, 2, 64, [64, 50, 14], block_size=64)
    q, k, v = (t.cuda() for t in synth.make_qkv(97, 128, 8, 2, 64))
    calls = []
    original = getattr(owner or r, name)

    def wrapper(*args, **kwargs):
        calls.append(name)
        return original(*args, **kwargs)
    assert r._one_call(q, k, v)
    want = r.run(q, k, v, 0.1).clone()
    assert not calls
    with monkeypatch.context() as patch:
        patch.setattr(owner or r, name, wrapper)
        got = r.run(q, k, v, 0.1)
        assert calls == [name] * 3
        assert torch.equal(got, want)
    if owner is not None:
        assert r._one_call(q, k, v)


@pytest.mark.gpu
def test_an_output_only_the_loop_accepts(gpu):
    """One-token chunks of an O with a longer row stride: each slice is contiguous, the whole is not."""
    r = ChunkedPrefill(4, 2, 64, [1, 1, 1], block_size=64)
    q, k, v = (t.cuda() for t in synth.make_qkv(98, 3, 4, 2, 64))
    want = r.run(q, k, v, 0.125).clone()
    r.o = torch.zeros(3, 8, 64, dtype=torch.bfloat16, device="cuda")[:, :4]
    assert torch.equal(r.run(q, k, v, 0.125), want)


@pytest.mark.gpu
def test_current_stream_handle(gpu, monkeypatch):
    """The handle of the current stream, also in a torch without the raw accessors."""
    side = torch.cuda.Stream()
    for raw, device in ((binding._raw_stream, binding._raw_device), (binding._raw_stream, torch.cuda.current_device),
                        (None, torch.cuda.current_device)):
        monkeypatch.setattr(binding, "_raw_stream", raw)
        monkeypatch.setattr(binding, "_raw_device", device)
        assert binding._stream_handle(None) == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(side):
            assert binding._stream_handle(None) == side.cuda_stream
        assert binding._stream_handle(side) == side.cuda_stream
