"""What AttentionBlock.forward hands to the library, with the library's calls recorded instead of run (no GPU needed)."""
from types import SimpleNamespace

import pytest
import torch

from paper_2502_12574_amd import attention_block as ab
from paper_2502_12574_amd import binding as hb

HKV, G, D, CHUNK = 2, 2, 256, 64


class _Stream:
    device_index = 3

    def wait_event(self, ev):
        pass


class _Device:
    """Stands for torch.cuda.device: the device that is current, 0 outside."""
    current = 0

    def __init__(self, index):
        self.index = index

    def __enter__(self):
        self.before, _Device.current = _Device.current, self.index

    def __exit__(self, *exc):
        _Device.current = self.before


@pytest.fixture
def block(monkeypatch):
    """A block over CPU buffers, and the list of library calls its forward makes."""
    calls = []
    monkeypatch.setattr(torch.cuda, "device", _Device)
    for name in ("hi_qkv_rope", "hi_prefill_group", "hi_decode_group", "hi_out_proj"):
        monkeypatch.setattr(hb, name, lambda *a, _name=name, **kw: calls.append((_name, a, _Device.current)))
    ss = SimpleNamespace(problem=hb.make_problem(1, HKV, G, 256, CHUNK), plan=SimpleNamespace(heads_per_group=HKV),
                         device=torch.device("cpu"), out_dtype=torch.bfloat16, mode=hb.HI_MODE_RESIDENT, ctx=None,
                         s_compute=_Stream(), s_d2h=_Stream())
    hq = HKV * G
    return ab.AttentionBlock(ss, 0, torch.zeros((hq + 2 * HKV) * 128, D, dtype=torch.bfloat16),
                             torch.zeros(D, hq * 128, dtype=torch.bfloat16)), calls


def _x(n):
    return torch.zeros(n, D, dtype=torch.bfloat16)


@pytest.mark.parametrize("n", [CHUNK + 1, 4 * CHUNK])
def test_more_rows_than_the_chunk_are_refused_before_the_first_call(block, n):
    blk, calls = block
    with pytest.raises(RuntimeError):
        blk.forward(_x(n), 0, _x(n))
    assert calls == []


@pytest.mark.parametrize("n", [1, 2, CHUNK])
def test_up_to_the_chunk_every_address_range_lies_in_its_buffer(block, n):
    blk, calls = block
    blk.forward(_x(n), 0, _x(n))
    names = [c[0] for c in calls]
    assert names == ["hi_qkv_rope", "hi_decode_group" if n == 1 else "hi_prefill_group", "hi_out_proj"]
    qkv, attn = calls[0][1], calls[1][1]
    room = {blk.q.data_ptr(): blk.q.nbytes, blk.attn.data_ptr(): blk.attn.nbytes}
    for pair in blk.kv:
        room.update({t.data_ptr(): t.nbytes for t in pair})
    for addr, heads in [(qkv[10], HKV * G), (qkv[11], HKV), (qkv[12], HKV), (attn[4], HKV * G), (attn[5], HKV), (attn[6], HKV),
                        (calls[2][1][1], HKV * G)]:
        assert heads * n * 256 <= room[addr]


@pytest.mark.parametrize("n", [1, 5])
def test_the_calls_run_on_the_sessions_device(block, n):
    """The caller may have another device current; a launch into a stream of a device that is not current fails."""
    blk, calls = block
    blk.forward(_x(n), 0, _x(n))
    assert len(calls) == 3 and {c[2] for c in calls} == {_Stream.device_index} and _Device.current == 0
