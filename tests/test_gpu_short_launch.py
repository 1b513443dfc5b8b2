"""Launches of few rounds at both head dims: static over the XCDs' lists with
a split tail (lists of unequal length among them), the hand-scheduled D=64
kernel in launches of less than a round, and balanced launches of more than
eight rounds, against the static launch without a workspace (bit for bit when
unsplit) and against float64.

Tolerances: bf16 states 1e-2 (unit-variance inputs, P V in bf16), LSE 2e-3."""
import pytest

pytestmark = pytest.mark.gpu

# (D, H, q_len, partition lengths)
CASES = [
    (64, 1, 1, [1]),
    (64, 3, 257, [65, 64, 63]),                    # 18 tasks: lists of 3 and 2
    (64, 5, 700, [130, 129, 128, 127, 126]),       # 75 tasks
    (64, 10, 4096, [520, 519]),                    # 320 tasks of 9 tiles: a round and a quarter, split or not
    (64, 11, 3000, [1100, 1050]),                  # 264 tasks of 18 tiles: 8 more than a round
    (128, 11, 3000, [1100, 1050]),
    (128, 3, 257, [65, 64, 63]),
    (64, 12, 3800, [70, 64, 66, 65, 64, 63, 64, 64, 70, 68, 64, 66]),   # 2,160 tasks: claimed
    (128, 12, 3800, [70, 64, 66, 65, 64, 63, 64, 64, 70, 68, 64, 66]),
    # D=64 around one round of 384-row tasks on 256 compute units
    (64, 9, 4096, [1024, 1000]),                   # 198 of them, 288 of 256 rows, short partitions: compiled kernel
    (64, 12, 2048, [2048, 2000, 2048]),            # 216, 288, long: compiled, or split with the workspace for it
    (64, 9, 4096, [300, 2100]),                    # the same of unequal lengths
    (64, 8, 6244, [700, 1234]),                    # 272: hand-scheduled
    (64, 8, 6244, [700, 2500]),                    # its last round split
    (64, 12, 2048, [2048, 700]),                   # 192 of 256 rows: hand-scheduled
]


@pytest.mark.parametrize("D,H,q_len,lens", CASES)
def test_launches_match_static_and_float64(D, H, q_len, lens):
    import torch
    from paper_2607_15650_amd import api
    P = len(lens)
    offs = [sum(lens[:j]) for j in range(P + 1)]
    g = torch.Generator(device="cuda").manual_seed(q_len)
    q, k, v = (torch.randn((1, n, H, D), generator=g, device="cuda").to(torch.bfloat16)
               for n in (q_len, offs[-1], offs[-1]))
    sel = [1] * P
    need = api.attn_workspace_bytes(torch.bfloat16, 1, H, D, q_len, offs, sel)

    def launch(n):
        ws = None if n is None else torch.full((n,), 0x5A, dtype=torch.uint8, device="cuda")
        out = torch.full((P, 1, q_len, H, D), 9.0, dtype=torch.bfloat16, device="cuda")
        lse = torch.full((P, 1, H, q_len), 9.0, device="cuda")
        api.attn_partition_states(q, k, v, offs, sel, D ** -0.5, out, lse, ws)
        return out, lse

    static = launch(None)
    unsplit = launch(256)
    assert torch.equal(static[0], unsplit[0]) and torch.equal(static[1], unsplit[1])
    full = launch(need)
    for j in range(P):
        for h in range(0, H, 5):
            s = torch.mm(q[0, :, h].double(), k[0, offs[j]:offs[j + 1], h].double().t().contiguous()) * D ** -0.5
            lse = torch.logsumexp(s, 1)
            ref = torch.mm((s - lse[:, None]).exp(), v[0, offs[j]:offs[j + 1], h].double())
            # few keys: a row is within 2^-8 max|v| of the exact one for the
            # probabilities, and 2^-9 of itself for the store
            tol = 1e-2 if lens[j] > 100 else 2.0 ** -7 * float(v.abs().max())
            for out, l in (static, full):
                assert float((out[j, 0, :, h].double() - ref).abs().max()) <= tol, (j, h)
                assert float((l[j, 0, h].double() - lse).abs().max()) <= 2e-3, (j, h)


def split_bytes(n, f):
    """Workspace of a split of n tasks of 256 rows at D=64 over f key ranges."""
    up = lambda x: -(-x // 256) * 256
    return 256 + up(n * f * 256 * 64 * 4) + up(n * f * 256 * 4)


@pytest.mark.parametrize("H,q_len,lens,split", [
    (9, 4096, [1024, 1024], None),                 # one round of 384-row tasks, short partitions
    (9, 4096, [300, 1984], None),                  # 31 tiles
    (9, 4096, [300, 1985], (32, 8)),               # 32: 256-row tasks, 288 of them
    (12, 2048, [2048, 2048, 2048], (32, 8)),
    (8, 6144, [2048, 2048], None),                 # 384 of them: a round and a half
    (8, 6244, [700, 2500], (144, 3)),              # 272 of 384 rows
    (12, 2048, [2048, 700], None),                 # 192 of 256 rows: nothing to split
])
def test_plan_of_short_head_dim_64_launches(H, q_len, lens, split):
    """The workspace tells which kernel's tasks a launch runs."""
    import torch
    from paper_2607_15650_amd import api
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("shapes are for 256 compute units")
    offs = [sum(lens[:j]) for j in range(len(lens) + 1)]
    need = api.attn_workspace_bytes(torch.bfloat16, 1, H, 64, q_len, offs, [1] * len(lens))
    assert need == (256 if split is None else split_bytes(*split))


def test_compiled_kernel_splits_its_last_round():
    """K of 2 GiB a partition, which the hand-scheduled kernel cannot address:
    272 tasks of 384 rows, the last 16 split."""
    import torch
    from paper_2607_15650_amd import api
    H, D, q_len, n = 272, 64, 100, 61700
    g = torch.Generator(device="cuda").manual_seed(0)
    q, k, v = (torch.randn((1, m, H, D), generator=g, device="cuda", dtype=torch.bfloat16) for m in (q_len, n, n))
    need = api.attn_workspace_bytes(torch.bfloat16, 1, H, D, q_len, [0, n], [1])
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert need > 256
    for size in (None, need):
        out = torch.full((1, 1, q_len, H, D), 9.0, dtype=torch.bfloat16, device="cuda")
        lse = torch.full((1, 1, H, q_len), 9.0, device="cuda")
        ws = None if size is None else torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda")
        api.attn_partition_states(q, k, v, [0, n], [1], D ** -0.5, out, lse, ws)
        for h in (0, 131, 255, 256, 271):
            s = torch.mm(q[0, :, h].double(), k[0, :, h].double().t().contiguous()) * D ** -0.5
            l = torch.logsumexp(s, 1)
            ref = torch.mm((s - l[:, None]).exp(), v[0, :, h].double())
            assert float((out[0, 0, :, h].double() - ref).abs().max()) <= 1e-2, h
            assert float((lse[0, 0, h].double() - l).abs().max()) <= 2e-3, h


@pytest.mark.parametrize("dtype,D,H", [("bf16", 64, 3), ("bf16", 128, 3), ("f32", 64, 3), ("f32", 128, 60)])
@pytest.mark.parametrize("q_begin,q_len", [(0, 257), (300, 257), (443, 257), (699, 1)])
def test_query_block_read_in_place(dtype, D, H, q_begin, q_len):
    """The block of a longer query tensor, batch of 2: bit for bit the launch
    on a copy of its rows; blocks outside the rows are refused."""
    import torch
    from paper_2607_15650_amd import _lib, api
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    offs = [0, 200, 430]
    g = torch.Generator(device="cuda").manual_seed(D)
    q, k, v = (torch.randn((2, n, H, D), generator=g, device="cuda").to(dt) for n in (700, 430, 430))
    got, ref = ([torch.full((2, 2, q_len, H, D), 9.0, dtype=dt, device="cuda"),
                 torch.full((2, 2, H, q_len), 9.0, device="cuda")] for _ in range(2))
    n = api.attn_workspace_bytes(dt, 2, H, D, q_len, offs, [1, 1])
    ws = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
    api.attn_block_states(q, q_begin, q_len, k, v, offs, [1, 1], D ** -0.5, *got, ws)
    api.attn_partition_states(q[:, q_begin:q_begin + q_len].contiguous(), k, v, offs, [1, 1], D ** -0.5, *ref, ws)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    for bad in (-1, 700 - q_len + 1):
        with pytest.raises(ValueError):
            api.attn_block_states(q, bad, q_len, k, v, offs, [1, 1], D ** -0.5, *got, ws)


def test_step_takes_a_strided_query_tensor():
    """Query tensors that are not contiguous are copied, as before."""
    import torch
    from paper_2607_15650_amd.step import SelectiveAttention
    g = torch.Generator(device="cuda").manual_seed(0)
    q, k, v = (torch.randn((2, 600, 2, 64), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    wide = torch.stack([q, q], dim=3)[:, :, :, 0]
    assert not wide.is_contiguous()
    res = []
    for x in (q, wide):
        sa = SelectiveAttention(2, 2, 64, [0, 200, 400, 600], 0.125)
        res.append(sa.step(0, 1, x, k, v, [1, 1, 1]))
    assert all(torch.equal(a, b) for a, b in zip(*res))


@pytest.mark.parametrize("D,H,q_len", [(64, 3, 300), (128, 3, 300), (64, 12, 2048)])
@pytest.mark.parametrize("shift", [1, 2, 4])
def test_query_tensor_at_any_even_address(D, H, q_len, shift):
    """bf16 queries 2, 4 or 8 bytes past a 16-byte boundary: the launch on an
    aligned copy, bit for bit, through the call and through an engine."""
    import torch
    from paper_2607_15650_amd import api
    from paper_2607_15650_amd.step import SelectiveAttention
    offs = [0, q_len, 2 * q_len]
    g = torch.Generator(device="cuda").manual_seed(shift)
    flat = torch.randn(2 * 2 * q_len * H * D + 8, generator=g, device="cuda").to(torch.bfloat16)
    q = flat[shift:shift + 4 * q_len * H * D].view(2, 2 * q_len, H, D)
    k, v = (torch.randn((2, 2 * q_len, H, D), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    assert q.data_ptr() % 16 != 0
    res = []
    for x in (q.clone(), q):
        out = torch.full((2, 2, 2 * q_len, H, D), 9.0, dtype=torch.bfloat16, device="cuda")
        lse = torch.full((2, 2, H, 2 * q_len), 9.0, device="cuda")
        api.attn_partition_states(x, k, v, offs, [1, 1], D ** -0.5, out, lse)
        sa = SelectiveAttention(2, H, D, offs, D ** -0.5)
        res.append((out, lse) + sa.step(0, 1, x, k, v, [1, 1]))
    assert all(torch.equal(a, b) for a, b in zip(*res))
