"""GPU tests of the streaming kernels at the edges of their instances: the
composition of float32 states over lists of 1 .. 17 slots, per-row weights
written through LDS for partition counts around the 16 staged at a time, and
state norms with a reference shared by up to four slots; the composition with
weights in one launch against the composition and the weights on their own.

Reference: torch in float64.  A float32 result here is a handful of products
and a short sum (at most 64 terms, or a fixed tree over the rows): 1e-6 on
weights, 1e-5 on composed outputs, 1e-5 relative on norms."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 9, 16, 17])
def test_merge_float32_lists(D, n):
    import torch
    from paper_2607_15650_amd import api
    P, B, L, H = 18, 2, 13, 3                     # 78 rows: a partial last workgroup
    g = torch.Generator(device="cuda").manual_seed(n)
    st = torch.randn((P, B, L, H, D), generator=g, device="cuda")
    lse = torch.randn((P, B, H, L), generator=g, device="cuda")
    lse[:, 1, 2, 5] = float("-inf")               # a row without any state
    slots = [(5 * i + 2) % P for i in range(n)]
    for out_dt in (torch.float32, torch.bfloat16):
        out = torch.full((B, L, H, D), 3.0, dtype=out_dt, device="cuda")
        lo = torch.full((B, H, L), 3.0, device="cuda")
        api.merge_states(st, lse, out, lo, slots=slots)
        ll = lse[slots].double()
        tot = torch.logsumexp(ll, 0)
        w = torch.exp(ll - tot).nan_to_num(0.0)
        ref = (st[slots].double() * w.permute(0, 1, 3, 2)[..., None]).sum(0)
        tol = 1e-5 if out_dt == torch.float32 else 2.0 ** -8 * float(ref.abs().max())
        assert float((out.double() - ref).abs().max()) <= tol
        dead = torch.isneginf(tot)
        assert bool(torch.isneginf(lo[dead]).all()) and float((lo.double() - tot)[~dead].abs().max()) <= 1e-5
    # in place into the first listed slot
    keep = ref
    api.merge_states(st, lse, st[slots[0]], lse[slots[0]], slots=slots)
    assert float((st[slots[0]].double() - keep).abs().max()) <= 1e-5


@pytest.mark.parametrize("P", [1, 3, 8, 9, 15, 16, 17, 20, 33, 64])
def test_weight_rows(P):
    import torch
    from paper_2607_15650_amd import api
    for B, H, L in ((1, 1, 1), (1, 3, 171), (2, 5, 103)):     # 1, 513 and 1,030 rows of 512 per workgroup
        g = torch.Generator(device="cuda").manual_seed(P)
        lse = torch.randn((P, B, H, L), generator=g, device="cuda")
        lse[P // 2, 0, 0, 0] = float("-inf")
        lo = torch.logsumexp(lse.double(), 0).float()
        w = torch.empty(P, device="cuda")
        pad = torch.full((B * H * L * P + 64,), 9.0, device="cuda")
        rows = pad[:B * H * L * P].view(B, H, L, P)
        ws = torch.empty(api.contrib_workspace_bytes(B, H, L, P), dtype=torch.uint8, device="cuda")
        api.contrib(lse, lo, w, ws, rows)
        ref = torch.exp(lse.double() - lo.double()).nan_to_num(0.0).permute(1, 2, 3, 0)
        assert float((rows.double() - ref).abs().max()) <= 1e-6
        assert float((w.double() - ref.mean((0, 1, 2))).abs().max()) <= 1e-6
        assert bool((pad[B * H * L * P:] == 9.0).all())
        w2 = torch.empty(P, device="cuda")
        api.contrib(lse, lo, w2, ws)
        assert torch.equal(w, w2)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8])
def test_norms_of_slots_sharing_a_reference(dtype, n):
    import torch
    from paper_2607_15650_amd import api
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    for B, L, H, D in ((1, 1, 1, 64), (1, 129, 4, 64), (2, 67, 3, 128)):   # 8, 4,128 and 6,432 chunks of 4,096
        g = torch.Generator(device="cuda").manual_seed(n)
        st = torch.randn((9, B, L, H, D), generator=g, device="cuda").to(dt)
        ref = torch.randn((B, L, H, D), generator=g, device="cuda").to(dt)
        slots = [(4 * i + 1) % 9 for i in range(n)]
        ws = torch.empty(api.norms_workspace_bytes(B, H, D, L, n), dtype=torch.uint8, device="cuda")
        for r in (ref, None):
            got = torch.empty(n, device="cuda")
            api.state_norms(st, got, ws, slots=slots, ref=r)
            exp = torch.stack([(st[j].double() - (0.0 if r is None else r.double())).norm() for j in slots])
            assert float(((got.double() - exp) / exp).abs().max()) <= 1e-5


@pytest.mark.parametrize("dtype,D,B,L,H,P,slots", [
    ("bf16", 128, 1, 1, 1, 1, None),                      # one row, one weight workgroup
    ("bf16", 64, 2, 43, 3, 8, [6, 1, 3]),                 # 258 rows: part of a row block of 512
    ("f32", 64, 1, 1025, 16, 4, None),                    # 16,400 rows: 33 row blocks
    ("bf16", 64, 1, 4150, 16, 2, None),                   # 66,400 rows: 130 blocks, two per workgroup
    ("bf16", 64, 1, 9000, 16, 9, None),                   # 282 blocks: more than one round of final sums
    ("bf16", 128, 2, 900, 10, 9, [8, 0, 2, 4, 1, 7, 3, 5, 6]),
    ("f32", 128, 1, 130, 2, 20, None),
    ("bf16", 64, 1, 70, 2, 64, None),
])
def test_compose_is_merge_and_weights(dtype, D, B, L, H, P, slots):
    import torch
    from paper_2607_15650_amd import api
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(L)
    st = torch.randn((P, B, L, H, D), generator=g, device="cuda").to(dt)
    lse = torch.randn((P, B, H, L), generator=g, device="cuda")
    lse[:, 0, 0, 0] = float("-inf")                       # a row without any state
    lse[P - 1, 0, H - 1, L // 2] = float("-inf")
    listed = list(range(P)) if slots is None else slots
    out, ref = (torch.full((B, L, H, D), 3.0, dtype=dt, device="cuda") for _ in range(2))
    lo, lref = (torch.full((B, H, L), 3.0, device="cuda") for _ in range(2))
    api.merge_states(st, lse, ref, lref, slots=slots)
    ll = lse[listed].double()
    w64 = torch.exp(ll - torch.logsumexp(ll, 0)).nan_to_num(0.0).mean((1, 2, 3))
    ws = api.compose_workspace(B, H, L, len(listed))
    # the weights kernels on the listed log-sum-exps, bit for bit
    cw = torch.empty(api.contrib_workspace_bytes(B, H, L, len(listed)), dtype=torch.uint8, device="cuda")
    first = torch.empty(len(listed), device="cuda")
    api.contrib(lse[listed].contiguous(), lref, first, cw)
    for _ in range(3):                                    # one workspace, left as it was found
        w = torch.full((len(listed),), 7.0, device="cuda")
        out.fill_(3.0)
        lo.fill_(3.0)
        api.compose(st, lse, out, lo, w, ws, slots=slots)
        assert torch.equal(out, ref) and torch.equal(lo.view(torch.int32), lref.view(torch.int32))
        assert float((w.double() - w64).abs().max()) <= 1e-6
        assert int(ws[:256].to(torch.int32).sum()) == 0
        assert torch.equal(w, first)
    api.compose(st, lse, out, None, w, ws, slots=slots)   # without the composed log-sum-exps
    assert torch.equal(w, first) and torch.equal(out, ref)


def test_compose_captured_in_a_graph():
    import torch
    from paper_2607_15650_amd import api
    P, B, L, H, D = 5, 1, 300, 4, 128
    g = torch.Generator(device="cuda").manual_seed(1)
    st = torch.randn((P, B, L, H, D), generator=g, device="cuda").to(torch.bfloat16)
    lse = torch.randn((P, B, H, L), generator=g, device="cuda")
    out = torch.empty((B, L, H, D), dtype=torch.bfloat16, device="cuda")
    lo, w, ws = torch.empty((B, H, L), device="cuda"), torch.empty(P, device="cuda"), api.compose_workspace(B, H, L, P)
    api.compose(st, lse, out, lo, w, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        api.compose(st, lse, out, lo, w, ws)
    for i in range(4):
        lse.add_(torch.randn((P, B, H, L), generator=g, device="cuda"))
        w.fill_(9.0)
        graph.replay()
        torch.cuda.synchronize()
        replayed = (out.clone(), lo.clone(), w.clone())
        api.compose(st, lse, out, lo, w, ws)              # eager work on the same workspace between
        assert all(torch.equal(a, b) for a, b in zip(replayed, (out, lo, w))), i


@pytest.mark.parametrize("n", [1, 8, 16, 20, 40])
def test_compose_needs_nothing_of_its_workspace(n):
    """Whatever the workspace holds (memory that was never written, what an
    interrupted or overlapping call left), the weights are those of the weight
    kernels."""
    import torch
    from paper_2607_15650_amd import api
    B, L, H, D = 1, 700, 5, 64
    g = torch.Generator(device="cuda").manual_seed(n)
    st = torch.randn((n, B, L, H, D), generator=g, device="cuda").to(torch.bfloat16)
    lse = torch.randn((n, B, H, L), generator=g, device="cuda")
    out = torch.empty((B, L, H, D), dtype=torch.bfloat16, device="cuda")
    lo, first = torch.empty((B, H, L), device="cuda"), torch.empty(n, device="cuda")
    api.merge_states(st, lse, out, lo)
    cw = torch.empty(api.contrib_workspace_bytes(B, H, L, n), dtype=torch.uint8, device="cuda")
    api.contrib(lse, lo, first, cw)
    ws = api.compose_workspace(B, H, L, n)
    for fill in (0xFF, 0x01, 0x7F, 0x00):
        ws.fill_(fill)
        w = torch.full((n,), 7.0, device="cuda")
        api.compose(st, lse, out, lo, w, ws)
        assert torch.equal(w, first), fill


@pytest.mark.parametrize("grouped", [False, True])
def test_first_composition_inside_a_capture(grouped):
    """An engine whose first step is captured: an eager step before any replay,
    and every replay, give the weights of an engine that never captured."""
    import torch
    from paper_2607_15650_amd.groups import GroupedSelectiveAttention
    from paper_2607_15650_amd.step import SelectiveAttention
    H, D, offs = 3, 64, [0, 130, 260, 390, 520]
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((1, 520, H, D), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))

    def engine():
        if grouped:
            e = GroupedSelectiveAttention(1, H, D, offs, 1, 1, D ** -0.5)
            return lambda t: e.step(t, q, k, v, e.groups)[2]
        e = SelectiveAttention(1, H, D, offs, D ** -0.5)
        e.cache(1)
        return lambda t: e.step(t, 1, q, k, v, [1, 1, 1, 1])[2]

    ref = engine()(0).clone()
    step = engine()
    torch.cuda.synchronize()
    # memory the captured step may be given holds anything
    junk = torch.full((1 << 22,), 0x5A, dtype=torch.uint8, device="cuda")
    del junk
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        w = step(0)
    assert torch.equal(step(1), ref)
    for i in range(3):
        w.fill_(9.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(w, ref), i
        assert torch.equal(step(2 + i), ref), i


def test_calls_go_to_the_current_stream():
    import torch
    from paper_2607_15650_amd import api
    assert api._stream() == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert api._stream() == s.cuda_stream
    assert api._stream() == torch.cuda.current_stream().cuda_stream != s.cuda_stream
