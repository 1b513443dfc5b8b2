"""Which library calls the step engines make, and on what (CPU only: the calls
are recorded, nothing is computed)."""
import pytest
import torch

from paper_2607_15650_amd import api
from paper_2607_15650_amd.groups import GroupedSelectiveAttention
from paper_2607_15650_amd.step import SelectiveAttention


@pytest.fixture
def calls(monkeypatch):
    """Every call as (name, arguments), in order."""
    log = []
    for name in ("attn_partition_states", "attn_block_states", "merge_states", "contrib", "compose"):
        monkeypatch.setattr(api, name, lambda *a, _n=name, **k: log.append((_n, a)))
    for name in ("attn_workspace_bytes", "contrib_workspace_bytes"):
        monkeypatch.setattr(api, name, lambda *a, **k: 256)
    monkeypatch.setattr(api, "compose_workspace", lambda *a, **k: torch.empty(256, dtype=torch.uint8))
    return log


def run(kind, P, q, B=1):
    """One step of an engine over P partitions of 4 tokens, one head, D=64."""
    offs = [4 * j for j in range(P + 1)]
    if kind == "step":
        e = SelectiveAttention(B, 1, 64, offs, 0.125, torch.bfloat16, "cpu")
        return e.step(0, 1, q, q, q, [1] * P)
    e = GroupedSelectiveAttention(B, 1, 64, offs, 1, 1, 0.125, torch.bfloat16, "cpu")
    return e.step(0, q, q, q, e.groups)


@pytest.mark.parametrize("kind", ["step", "group"])
@pytest.mark.parametrize("P", [2, 16, 17, 64])
def test_composition_and_weights_are_one_call(calls, kind, P):
    """At every number of states: the call is faster than composition and
    weights on their own, in both engines."""
    q = torch.zeros((1, 4 * P, 1, 64), dtype=torch.bfloat16)
    run(kind, P, q)
    assert [n for n, _ in calls] == ["attn_block_states", "compose"]


@pytest.mark.parametrize("kind", ["step", "group"])
@pytest.mark.parametrize("B", [1, 2])
@pytest.mark.parametrize("shift,strided", [(0, False), (1, False), (4, False), (8, False), (0, True)])
def test_query_block_is_in_place_or_an_aligned_copy(calls, kind, B, shift, strided):
    """Read in place where the kernels' 16-byte loads can read it, otherwise a
    copy of the block's rows; the rows handed over are the block's either way."""
    P, n = 3, B * 12 * 64
    flat = torch.arange(2 * n + 8, dtype=torch.float32).to(torch.bfloat16)
    q = flat[shift:shift + 2 * n:2].view(B, 12, 1, 64) if strided else flat[shift:shift + n].view(B, 12, 1, 64)
    run(kind, P, q, B)
    name, args = calls[0]
    assert name == "attn_block_states"
    got, begin, length = args[:3]
    assert got.is_contiguous() and got.data_ptr() % 16 == 0 and length == 4
    assert torch.equal(got[:, begin:begin + length], q[:, 4:8])
    assert (got.data_ptr() == q.data_ptr()) == (not strided and q.data_ptr() % 16 == 0)
