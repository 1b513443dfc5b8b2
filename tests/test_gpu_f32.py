"""GPU parity of the float32 attention kernel's forms (waves that split the
keys, workgroups of 128 and of 256 rows), which the launch picks by its
number of query tiles: ragged tiles, key counts around the 32-key tile and
the per-wave ranges, empty partitions, and operands the three-plane bf16 split
cannot represent (infinities, NaN, values beyond bf16's largest), which the
kernel hands to its float32 MFMA pass.

Reference: torch in float64 on the same float32 values.  Tolerance 1e-5 on
OUT and LSE at unit-variance inputs, as for every float32 result here: a sum
of at most 400 float32 terms is within 400 * 2^-24 = 2.4e-5 of their absolute
sum in the worst case and about sqrt(400) * 2^-24 = 1.2e-6 at random."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def reference(q, k, v, offs, scale):
    import torch
    outs, lses = [], []
    for a, e in zip(offs, offs[1:]):
        s = torch.matmul(q.double().transpose(1, 2), k[:, a:e].double().permute(0, 2, 3, 1)) * scale
        lse = torch.logsumexp(s, -1) if e > a else torch.full(s.shape[:-1], float("-inf"), dtype=torch.float64)
        p = torch.exp(s - lse[..., None]) if e > a else s
        outs.append(torch.matmul(p, v[:, a:e].double().transpose(1, 2)).transpose(1, 2))
        lses.append(lse)
    return outs, lses


def run(q, k, v, offs, scale):
    import torch
    from paper_2607_15650_amd import api
    B, L, H, D = q.shape
    P = len(offs) - 1
    out = torch.full((P, B, L, H, D), 7.0, device="cuda")
    lse = torch.full((P, B, H, L), 7.0, device="cuda")
    api.attn_partition_states(q.cuda(), k.cuda(), v.cuda(), offs, [1] * P, scale, out, lse)
    torch.cuda.synchronize()
    return out.cpu(), lse.cpu()


def inputs(B, L, S, H, D, seed):
    import torch
    g = torch.Generator().manual_seed(seed)
    return [torch.randn((B, n, H, D), generator=g) + c for n, c in ((L, 0.0), (S, 0.3), (S, 0.0))]


# (D, H, q_len, partition lengths): on 256 compute units the first two of each
# head dim run the key-splitting form (up to 512 tiles of 32 rows), the third
# the 128-row form, the last at D=128 the 256-row form
SHAPES = [
    (64, 1, 1, [1, 0, 31, 32, 33]),
    (64, 2, 65, [255, 256, 257, 400]),          # eight waves: 8 tiles of 32 keys, one more, a partial one
    (64, 20, 130, [1, 63, 64, 65, 97, 0]),
    (128, 1, 33, [1, 0, 31, 127, 128, 129]),    # four waves
    (128, 3, 31, [160, 400]),
    (128, 20, 129, [33, 64, 95, 0]),            # 400 tiles of 32 rows
    (128, 40, 129, [33, 64, 95]),               # 240 workgroups of 128 rows
    (128, 50, 257, [1, 32, 65, 96]),            # 256-row workgroups
]


@pytest.mark.parametrize("D,H,q_len,lens", SHAPES)
def test_forms_match_float64(D, H, q_len, lens):
    offs = np.concatenate([[0], np.cumsum(lens)]).tolist()
    q, k, v = inputs(1, q_len, offs[-1], H, D, q_len + D)
    out, lse = run(q, k, v, offs, 1 / math.sqrt(D))
    outs, lses = reference(q, k, v, offs, 1 / math.sqrt(D))
    for j, n in enumerate(lens):
        if n == 0:
            assert bool((out[j] == 0).all()) and bool((lse[j] == float("-inf")).all())
        else:
            assert float((out[j] - outs[j]).abs().max()) <= 1e-5, j
            assert float((lse[j] - lses[j]).abs().max()) <= 1e-5, j


@pytest.mark.parametrize("D,H,q_len", [(64, 1, 40), (64, 20, 260), (128, 1, 40), (128, 60, 129), (128, 120, 257)])
def test_operands_the_planes_cannot_hold(D, H, q_len):
    """Head 0: a key whose scores are -inf (no weight).  Other partitions: a
    value beyond bf16's range, an infinite value, a NaN key."""
    import torch
    lens = [70, 40, 40, 40]
    offs = np.concatenate([[0], np.cumsum(lens)]).tolist()
    q, k, v = inputs(1, q_len, offs[-1], H, D, 3)
    q[:, :, 0, 5] = q[:, :, 0, 5].abs() + 0.1
    k[0, 50, 0, 5] = float("-inf")
    big = 3.3999e38                                  # rounds to infinity in bf16
    v[0, 80, 0, 7] = big
    v[0, 120, 0, 9] = float("inf")
    k[0, 160, 0, 3] = float("nan")
    out, lse = run(q, k, v, offs, 1 / math.sqrt(D))
    kk, vv = k.clone(), v.clone()
    vv[0, 120, 0, 9] = 0.0
    outs, lses = reference(q, kk, vv, offs, 1 / math.sqrt(D))
    # the masked key has no weight: torch agrees (exp(-inf) = 0)
    assert float((out[0] - outs[0]).abs().max()) <= 1e-5 and float((lse[0] - lses[0]).abs().max()) <= 1e-5
    # relative where the large value enters
    rel = (out[1] - outs[1]).abs() / outs[1].abs().clamp_min(1.0)
    assert float(rel.max()) <= 1e-5 and float((lse[1] - lses[1]).abs().max()) <= 1e-5
    assert bool((out[2][0, :, 0, 9] == float("inf")).all())
    o2, r2 = out[2].clone(), outs[2].clone()
    o2[0, :, 0, 9] = r2[0, :, 0, 9] = 0.0
    assert float((o2 - r2).abs().max()) <= 1e-5 and float((lse[2] - lses[2]).abs().max()) <= 1e-5
    assert bool(torch.isnan(out[3][0, :, 0]).all())
    if H > 1:
        assert float((out[3][0, :, 1:] - outs[3][0, :, 1:]).abs().max()) <= 1e-5


@pytest.mark.parametrize("D,H,q_len", [(64, 1, 40), (64, 20, 260), (128, 1, 40), (128, 60, 129), (128, 120, 257)])
def test_values_below_the_range_of_the_planes(D, H, q_len):
    """Nonzero operands under 2^-110 have fewer bits in the planes than in
    float32: V columns of ever smaller values, down to float32's subnormal
    ones, beside a column of zeros, and queries so small that only large keys
    make scores of them.

    Tolerance: 1e-5 of the column's largest output, and where products are
    subnormal half a spacing (2^-150) for each of the n terms, the sum and its
    normalisation."""
    import torch
    lens = [70, 33]
    offs = [0, 70, 103]
    scale = 1 / math.sqrt(D)
    q, k, v = inputs(1, q_len, offs[-1], H, D, 5)
    for i, e in enumerate((0, 100, 109, 111, 113, 116, 120, 124, 126, 128, 132, 136, 140)):
        v[:, :, 0, i] *= 2.0 ** -e
    v[:, :, 0, 20] = 0.0
    v[:, :70, 0, 21] = 0.0
    v[0, 50, 0, 21] = 2.0 ** -140
    if H > 1:                                    # a head of zeros, and one of ordinary values
        v[:, :, 1] = 0.0
    out, lse = run(q, k, v, offs, scale)
    outs, lses = reference(q, k, v, offs, scale)
    for j, n in enumerate(lens):
        tol = 1e-5 * outs[j].abs().amax(1, keepdim=True) + (n + 2) * 2.0 ** -150
        bad = ((out[j] - outs[j]).abs() > tol).nonzero()
        assert len(bad) == 0, (j, bad[0].tolist(), len(bad))
        assert float((lse[j] - lses[j]).abs().max()) <= 1e-5, j
    for e in (115, 125):
        ks, qs = k * 2.0 ** e, q * 2.0 ** -e     # the same scores, but for subnormal queries
        out, lse = run(qs, ks, v, offs, scale)
        outs, lses = reference(qs, ks, v, offs, scale)
        for j in range(2):
            assert float((out[j] - outs[j]).abs().max()) <= 1e-5, (e, j)
            assert float((lse[j] - lses[j]).abs().max()) <= 1e-5, (e, j)
