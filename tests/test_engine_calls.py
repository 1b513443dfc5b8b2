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
