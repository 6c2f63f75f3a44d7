"""Several Sinkhorn steps in one launch, whose workgroups hand their column sums to each other, against the same steps launch by
launch: a forward whose workspace has room for the column sums of launched steps and no more takes the latter.  The same kernel on
the same numbers, so the same bits; and the answer where a wait for a neighbour runs out.  Which route a call took is asked
(query_chains), in every case."""
import pytest

pytestmark = pytest.mark.gpu

CASES = [  # kind, dtype, d, N, L, W, T, R: one block and many, one tile of band and as many as single blocks take, ragged ends
    ("plain", "bf16", 64, 1, 31, 7, 3, 2), ("plain", "bf16", 64, 2, 65, 0, 2, 1), ("plain", "bf16", 64, 8, 701, 64, 16, 2),
    ("plain", "bf16", 64, 5, 3001, 100, 9, 2), ("plain", "bf16", 64, 30, 1999, 128, 4, 3), ("plain", "bf16", 64, 3, 1023, 256, 5, 2),
    ("plain", "bf16", 64, 2, 1100, 300, 4, 3), ("plain", "bf16", 64, 1, 700, 33, 0, 4), ("plain", "bf16", 64, 1, 700, 33, 1, 2),
    ("plain", "bf16", 32, 7, 1333, 40, 5, 2), ("plain", "bf16", 128, 4, 1777, 127, 5, 2), ("plain", "bf16", 128, 2, 900, 256, 3, 2),
    ("plain", "bf16", 64, 300, 130, 60, 3, 2), ("plain", "f32", 32, 1, 256, 16, 8, 2), ("plain", "f32", 64, 8, 2000, 128, 5, 2),
    ("plain", "f32", 64, 2, 700, 255, 3, 6), ("plain", "f32", 128, 2, 500, 60, 3, 2), ("plain", "bf16", 64, 2, 400, 5000, 4, 6),
    # fp32 keeps its scores over the steps: beside the plan entries or with those evaluated twice, few tiles and many
    ("plain", "f32", 64, 4, 2000, 256, 4, 6), ("plain", "f32", 64, 8, 8000, 128, 3, 2), ("plain", "f32", 32, 8, 2000, 128, 4, 2),
    ("plain", "f32", 64, 2, 3000, 60, 4, 2), ("plain", "f32", 128, 4, 700, 33, 4, 2), ("varlen", "f32", 64, 4, 8000, 120, 3, 2),
    ("varlen", "bf16", 64, 6, 2048, 128, 6, 2), ("varlen", "f32", 64, 4, 500, 100, 4, 2), ("varlen", "bf16", 64, 4, 900, 200, 2, 3),
    ("varlen", "bf16", 64, 4, 611, 20, 1, 3),
    ("dustbin", "bf16", 64, 2, 701, 30, 6, 2), ("dustbin", "bf16", 64, 8, 4000, 128, 5, 2), ("dustbin", "f32", 64, 2, 900, 100, 4, 2),
    ("dustbin", "bf16", 128, 2, 600, 222, 3, 2), ("dustbin", "bf16", 32, 1, 20000, 60, 0, 4), ("dustbin", "f32", 32, 1, 40, 16, 3, 2),
    ("marginals", "bf16", 64, 3, 900, 100, 5, 2), ("marginals", "f32", 64, 2, 700, 50, 4, 2), ("small targets", "bf16", 64, 2, 900, 64, 4, 2),
    ("masked", "bf16", 64, 4, 700, 40, 5, 2), ("masked", "f32", 64, 2, 600, 128, 4, 3), ("masked", "bf16", 64, 2, 500, 1, 0, 3)]
LAUNCHED = [   # with as large a workspace: a dustbin's 632 blocks, which are more than a chain takes; 2000 blocks, more than fit the device;
    # windows whose words are more than the workspace of as few tail steps has room for
    ("dustbin", "bf16", 64, 8, 5000, 128, 5, 2), ("plain", "f32", 64, 16, 16000, 60, 3, 2), ("plain", "bf16", 64, 2, 1100, 300, 4, 2),
    ("plain", "f32", 64, 2, 700, 255, 3, 1), ("plain", "bf16", 64, 2, 400, 5000, 4, 2), ("plain", "f32", 64, 4, 2000, 256, 4, 2)]


def _setup(case):
    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    kind, dtype, d, N, L, W, T, R = case
    td, code = (torch.float32, 0) if dtype == "f32" else (torch.bfloat16, 1)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(31)
    Q, K, V = (torch.randn((N, 1, L, d), generator=gen, device="cuda").to(td) for _ in range(3))
    lq = lk = None
    if kind == "varlen":   # an item without queries, one with a single key, rows that end before and after the columns
        lq, lk = (torch.randint(1, L + 1, (N,), generator=gen, device="cuda").int() for _ in range(2))
        lq[0], lk[1] = 0, 1
        lq[2], lk[2] = L // 3, L
        lq[3], lk[3] = L, L // 4
    db = kind == "dustbin"
    la = lb = None
    if kind in ("marginals", "small targets"):
        a, b = (torch.rand((N, 1, L), generator=gen, device="cuda") + 0.5 for _ in range(2))
        la, lb = a.log(), (b * a.sum(-1, keepdim=True) / b.sum(-1, keepdim=True)).log()
    if kind == "small targets":
        la[..., ::16], lb[..., 5::16] = -100.0, float("-inf")
    if kind == "masked":   # (a window of one: many tokens without an active partner)
        mq, mk = ((torch.rand((N, L), generator=gen, device="cuda") > 0.3).to(torch.uint8) for _ in range(2))
    plan = binding.query_step_plan(N, 1, L, d, W, T, R, db, code, lengths=kind == "varlen")
    assert plan.whole_steps and plan.segment_blocks == 1
    few = plan.sums_offset[1] + N * plan.sums_bytes   # launches: room for two buffers of column sums
    assert few < ska.sinkhorn_attn_workspace_bytes(N, 1, L, d, W, T, R, db, code)

    def forward(nbytes=None):
        """O, UV, and whether the steps ran as a chain"""
        before = binding.query_chains().launched
        ws = None if nbytes is None else torch.full((nbytes,), 255, device="cuda", dtype=torch.uint8)
        if kind == "masked":
            out = ska.sinkhorn_attn_fwd_masked(Q, K, V, mq, mk, W, T, R, 0.7, workspace=ws)
        else:
            out = ska.sinkhorn_attn_fwd_varlen(Q, K, V, la, lb, lq, lk, W, T, R, 0.7, db, 0.3, workspace=ws)
        torch.cuda.synchronize()
        chains = binding.query_chains()
        assert chains.started == chains.launched <= before + 1
        return *out, chains.launched > before

    return forward, few


@pytest.mark.parametrize("case", CASES + LAUNCHED, ids=lambda c: "-".join(map(str, c)))
def test_a_chain_has_the_bits_of_its_steps(case):
    import torch

    from paper_2605_08123_amd import binding
    print(f"\n[case] {case}", flush=True)
    forward, few = _setup(case)
    O0, UV0, chained = forward(few)
    assert not chained and not torch.isnan(UV0).any() and torch.isfinite(O0.float()).all()
    given_up = binding.query_chains().given_up
    for _ in range(3):   # (the words of the call before lie where the next one's will)
        O, UV, chained = forward()
        assert chained == (case not in LAUNCHED)
        assert torch.equal(UV, UV0) and torch.equal(O, O0)
    assert binding.query_chains().given_up == given_up


@pytest.mark.parametrize("case", [c for c in CASES if c[:5] in (
    ("plain", "bf16", 64, 8, 701), ("plain", "bf16", 64, 5, 3001), ("plain", "f32", 64, 8, 2000), ("varlen", "bf16", 64, 6, 2048),
    ("varlen", "bf16", 64, 4, 900), ("dustbin", "bf16", 64, 8, 4000), ("dustbin", "f32", 64, 2, 900), ("marginals", "f32", 64, 2, 700),
    ("masked", "bf16", 64, 4, 700), ("masked", "f32", 64, 2, 600), ("plain", "bf16", 128, 4, 1777), ("plain", "f32", 128, 2, 500),
    ("plain", "bf16", 32, 7, 1333), ("plain", "f32", 32, 1, 256), ("dustbin", "bf16", 32, 1, 20000), ("varlen", "f32", 64, 4, 500),
    ("varlen", "bf16", 64, 4, 611), ("plain", "f32", 64, 2, 700)) or c[3:6] == (1, 700, 33)], ids=lambda c: "-".join(map(str, c)))
def test_a_wait_that_runs_out_leaves_the_answer(case):
    """One poll and no more: some workgroup gives up (if by chance none has, once more), and the launch that follows solves the
    problem by itself.  The potentials agree to rounding: (2 W + 20 + 4 M) 2^-24 per half-step on either side (see test_gpu_steps.py), M the largest exponent."""
    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    kind, dtype, d, N, L, W, T, R = case
    print(f"\n[case] {case}", flush=True)
    forward, few = _setup(case)
    O0, UV0, _ = forward(few)
    try:
        for _ in range(20):
            ska.sinkhorn_attn_set_fused_half_steps(0, 1)
            O, UV, chained = forward()
            assert chained
            chains = binding.query_chains()
            if chains.given_up == chains.launched:
                break
        assert chains.given_up == chains.launched
    finally:
        ska.sinkhorn_attn_set_fused_half_steps(0)
    assert torch.equal(torch.isneginf(UV), torch.isneginf(UV0))
    x, y = (torch.where(torch.isneginf(z), 0.0, z.double()) for z in (UV, UV0))
    M = 1.4427 * max(float(y.abs().max()), 6.0 * d ** 0.5 / 0.7)
    # (a dustbin's row and column are sums over all tokens)
    bound = 2 * 2 * (T + R) * ((L if kind == "dustbin" else 2 * min(W, L)) + 21 + 4 * M) * 2.0 ** -24
    err = float((x - y).abs().max())
    print(f"   |UV - UV0| {err:.1e} (bound {bound:.1e})", flush=True)
    assert err <= bound
    rel = float((O.double() - O0.double()).norm() / O0.double().norm())
    assert rel <= 2 * bound + (2.0 ** -8 if dtype == "bf16" else 0.0), rel


@pytest.mark.parametrize("B,H,L,d,W,T,R,room", [(2, 2, 2500, 64, 100, 6, 2, True), (3, 3, 446, 32, 255, 2, 1, False),
                                                (3, 3, 446, 32, 255, 2, 2, True), (1, 2, 446, 64, 255, 3, 2, True)])
def test_a_chain_with_learned_dustbin_tokens_is_replayed_by_launches(B, H, L, d, W, T, R, room):
    """Captured steps are launches: the same bits as the eager chain, tokens' spokes and gradients included.  (Wide bands over few
    rows take most room in the workspace, which the spokes follow.)"""
    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    eps = 0.5
    Q, K, V, G = (torch.randn((B, H, L, d), generator=gen, device="cuda").bfloat16() for _ in range(4))
    tok = [torch.randn((B, H, d), generator=gen, device="cuda") for _ in range(3)]
    ws = torch.empty(ska.sinkhorn_attn_workspace_bytes(B, H, L, d, W, T, R, True, 1), device="cuda", dtype=torch.uint8)

    def run():
        O, UV = ska.sinkhorn_attn_fwd_dustbin_token(Q, K, V, *tok, W, T, R, eps, workspace=ws)
        return [O, UV, *ska.sinkhorn_attn_bwd_dustbin_token(Q, K, V, *tok, O, G, UV, W, T, R, eps, workspace=ws)]

    before = binding.query_chains().launched
    eager = [x.clone() for x in run()]
    torch.cuda.synchronize()
    assert binding.query_chains().launched == before + room
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        out = run()
    assert binding.query_chains().launched == before + room
    for _ in range(3):
        for x in out:
            x.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for x, y in zip(out, eager):
            assert torch.isfinite(y.float()).all() and torch.equal(x, y)


@pytest.mark.parametrize("N,dtype,R,T", [(1, "bf16", 16, 2), (16, "bf16", 13, 3), (1, "f32", 20, 0), (1, "f32", 16, 1)])
def test_no_chain_where_launched_steps_have_no_room(N, dtype, R, T):
    """A few rows with many tail steps: room for a chain's words and none for two buffers of launched sums.  The steps are half-steps
    then, queued or not, and none of them is lost."""
    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    td, code = (torch.float32, 0) if dtype == "f32" else (torch.bfloat16, 1)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    L, W, d = 4, 3, 64
    Q, K, V = (torch.randn((N, 1, L, d), generator=gen, device="cuda").to(td) for _ in range(3))
    assert not binding.query_step_plan(N, 1, L, d, W, T, R, False, code).whole_steps
    before = binding.query_chains().launched
    S = (Q.double() @ K.double().transpose(-1, -2).contiguous())[:, 0] / (0.7 * d ** 0.5)
    v, uv = torch.zeros((N, L), device="cuda", dtype=torch.float64), []
    for t in range(T + R):
        u = -torch.logsumexp(S + v[:, None], 2)
        v1 = -torch.logsumexp(S + u[:, :, None], 1)
        if t >= T:
            uv += [u, v1]
        v = v1
    try:
        for mode in (0, 1, 2):
            ska.sinkhorn_attn_set_fused_half_steps(mode)
            O, UV = ska.sinkhorn_attn_fwd(Q, K, V, W, T, R, 0.7)
            torch.cuda.synchronize()
            if mode == 0:
                O0, UV0 = O.clone(), UV.clone()
                assert binding.query_chains().launched == before
            assert torch.equal(O, O0) and torch.equal(UV, UV0), mode
    finally:
        ska.sinkhorn_attn_set_fused_half_steps(0)
    # per half-step (2 W + 20 + 4 M) 2^-24 (see above), M the largest exponent; bf16: and the scaled operand's rounding, 2^-9 of |Q| |K|^T
    big = float((Q.double().abs() @ K.double().abs().transpose(-1, -2).contiguous()).max()) / (0.7 * d ** 0.5)
    M = 1.4427 * (big + float(UV0.abs().max()))
    bound = 2 * (T + R) * ((2 * W + 20 + 4 * M) * 2.0 ** -24 + (2.0 ** -9 * big if dtype == "bf16" else 0.0))
    err = float((UV0[:, 0, 2:].double() - torch.stack(uv, 1)).abs().max())
    print(f"[case] {N, dtype, R, T} |UV - UV64| {err:.1e} (bound {bound:.1e})", flush=True)
    assert err <= bound


@pytest.mark.parametrize("first,second", [(a, b) for a in ("steps", "half-steps") for b in ("steps", "half-steps")])
def test_no_chain_beside_one_that_has_not_started(first, second):
    """A call whose chain stands behind other work on its stream: another stream's call runs as launches, the same stream's next one as a
    chain.  All of them have the bits of launches."""
    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    sizes = {"steps": (4, 700, 64, 6), "half-steps": (2, 9000, 500, 3)}
    data = {k: [torch.randn((N, 1, L, 64), generator=gen, device="cuda").bfloat16() for _ in range(3)] for k, (N, L, _, _) in sizes.items()}

    def ws(kind):
        N, L, W, T = sizes[kind]
        return torch.empty(ska.sinkhorn_attn_workspace_bytes(N, 1, L, 64, W, T, 2, False, 1), device="cuda", dtype=torch.uint8)

    def call(kind, w):
        N, L, W, T = sizes[kind]
        before = binding.query_chains().launched
        return *ska.sinkhorn_attn_fwd(*data[kind], W, T, 2, 0.6, workspace=w), binding.query_chains().launched - before

    few = binding.query_step_plan(4, 1, 700, 64, 64, 6)
    few = few.sums_offset[1] + 4 * few.sums_bytes
    ref = {"steps": call("steps", ws("steps")[:few]), "half-steps": call("half-steps", ws("half-steps"))}
    assert ref["steps"][2] == ref["half-steps"][2] == 0
    A, B = torch.cuda.Stream(), torch.cuda.Stream()
    room = [ws(first), ws(second), ws(second)]
    try:
        ska.sinkhorn_attn_set_fused_half_steps(2)
        for k in sizes:
            assert call(k, ws(k))[2] == 1   # (both kinds are chains here)
        torch.cuda.synchronize()
        with torch.cuda.stream(A):
            torch.cuda._sleep(300_000_000)   # (some tenths of a second; ends by itself)
            one = call(first, room[0])
        chains = binding.query_chains()
        waiting = chains.started != chains.launched
        with torch.cuda.stream(B):
            two = call(second, room[1])
        with torch.cuda.stream(A):
            three = call(second, room[2])
        torch.cuda.synchronize()
    finally:
        ska.sinkhorn_attn_set_fused_half_steps(0)
    assert waiting and (one[2], two[2], three[2]) == (1, 0, 1)
    for kind, got in ((first, one), (second, two), (second, three)):
        assert torch.equal(got[0], ref[kind][0]) and torch.equal(got[1], ref[kind][1])
    chains = binding.query_chains()
    assert chains.started == chains.launched


@pytest.mark.parametrize("kind,split", [("steps", False), ("half-steps", False), ("half-steps", True)])
def test_after_a_wait_that_ran_out_calls_are_launched(kind, split):
    """(split: half-steps that were queued for one launch run on the two streams after all)"""
    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    gen = torch.Generator(device="cuda")
    gen.manual_seed(12)
    N, L, W, mode = (8, 700, 64, 0) if kind == "steps" else (3, 9000, 500, 2)
    Q, K, V = (torch.randn((N, 1, L, 64), generator=gen, device="cuda").bfloat16() for _ in range(3))

    def call():
        before = binding.query_chains().launched
        out = ska.sinkhorn_attn_fwd(Q, K, V, W, 6, 2, 0.6)
        torch.cuda.synchronize()
        return *out, binding.query_chains().launched - before

    try:
        ska.sinkhorn_attn_set_split_min_edges(0.0 if split else 5e7)
        ska.sinkhorn_attn_set_fused_half_steps(mode)
        ref = call()
        assert ref[2] == 1
        for _ in range(20):   # (until a wait has run out)
            ska.sinkhorn_attn_set_fused_half_steps(mode, 1)
            call()
            chains = binding.query_chains()
            if chains.given_up == chains.launched:
                break
        assert chains.given_up == chains.launched
        for _ in range(3):
            O, UV, chained = call()
            assert not chained and torch.equal(O, ref[0]) and torch.equal(UV, ref[1])
        ska.sinkhorn_attn_set_fused_half_steps(mode)
        O, UV, chained = call()
        assert chained and torch.equal(O, ref[0]) and torch.equal(UV, ref[1])
    finally:
        ska.sinkhorn_attn_set_split_min_edges(5e7)
        ska.sinkhorn_attn_set_fused_half_steps(0)


def test_a_chain_behind_one_that_gave_up():
    """In the queue when the one before gives up: it waits less long, and runs to its end where nothing keeps its workgroups out."""
    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    gen = torch.Generator(device="cuda")
    gen.manual_seed(13)
    Q, K, V = (torch.randn((8, 1, 700, 64), generator=gen, device="cuda").bfloat16() for _ in range(3))
    ws = [torch.empty(ska.sinkhorn_attn_workspace_bytes(8, 1, 700, 64, 64, 6, 2, False, 1), device="cuda", dtype=torch.uint8) for _ in range(2)]
    call = lambda i: ska.sinkhorn_attn_fwd(Q, K, V, 64, 6, 2, 0.6, workspace=ws[i])
    try:
        ska.sinkhorn_attn_set_fused_half_steps(0)
        O0, UV0 = call(0)
        for _ in range(20):   # (until a wait has run out)
            torch.cuda._sleep(100_000_000)
            ska.sinkhorn_attn_set_fused_half_steps(0, 1)
            first, before = call(0), binding.query_chains()
            ska.sinkhorn_attn_set_fused_half_steps(0)
            second = call(1)
            torch.cuda.synchronize()
            chains = binding.query_chains()
            assert chains.launched == before.launched + 1 and before.started < before.launched
            if chains.given_up == before.launched:
                break
        assert chains.given_up == before.launched
    finally:
        ska.sinkhorn_attn_set_fused_half_steps(0)
    assert torch.equal(second[0], O0) and torch.equal(second[1], UV0)
    # (the first one's bound is that of the test of waits that run out: 2 * 2 * 8 half-steps of (2 W + 21 + 4 M) 2^-24 each)
    M = 1.4427 * max(float(UV0.abs().max()), 6.0 * 8 / 0.6)
    assert float((first[1] - UV0).abs().max()) <= 2 * 2 * 8 * (2 * 64 + 21 + 4 * M) * 2.0 ** -24


@pytest.mark.parametrize("kind", ["steps", "half-steps"])
def test_no_chain_on_a_stream_with_some_of_the_cus(kind):
    """What the device holds at once may not fit the CUs of such a stream: its calls are launched, with the same bits."""
    import ctypes

    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    torch.cuda.init()
    hip = ctypes.CDLL("libamdhip64.so")
    hip.hipExtStreamCreateWithCUMask.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_uint32, ctypes.POINTER(ctypes.c_uint32)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(14)
    N, L, W, mode = (8, 700, 64, 0) if kind == "steps" else (2, 9000, 500, 2)
    Q, K, V = (torch.randn((N, 1, L, 64), generator=gen, device="cuda").bfloat16() for _ in range(3))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    words = (cus + 31) // 32
    masks = {"all": [0xffffffff] * words, "half": [0xffffffff if i < words // 2 else 0 for i in range(words)]}
    results = {}
    try:
        ska.sinkhorn_attn_set_fused_half_steps(mode)
        for name, mask in masks.items():
            st = ctypes.c_void_p()
            assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(st), words, (ctypes.c_uint32 * words)(*mask)) == 0
            with torch.cuda.stream(torch.cuda.ExternalStream(st.value)):
                before = binding.query_chains().launched
                O, UV = ska.sinkhorn_attn_fwd(Q, K, V, W, 6, 2, 0.6)
                torch.cuda.synchronize()
                assert binding.query_chains().launched - before == (name == "all")
            results[name] = O, UV
    finally:
        ska.sinkhorn_attn_set_fused_half_steps(0)
    assert all(torch.equal(x, y) for x, y in zip(results["all"], results["half"]))


@pytest.mark.parametrize("what", ["NaN", "no partner"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_what_is_no_number_stays_none_where_a_wait_ran_out(what, dtype):
    """One query with a NaN, or one key whose scores are all -inf (its first column sum has no entry, which is an error then): the
    solve after a chain that gave up says NaN wherever the band carries it, as the launched steps do, and nowhere out of their reach."""
    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    gen = torch.Generator(device="cuda")
    gen.manual_seed(15)
    L, W, T, R, at = 3000, 20, 1, 2, 1500
    td, code = (torch.float32, 0) if dtype == "f32" else (torch.bfloat16, 1)
    Q, K, V = (torch.randn((1, 1, L, 64), generator=gen, device="cuda").to(td) for _ in range(3))
    if what == "NaN":
        Q[0, 0, at, 5] = float("nan")
    else:
        Q[..., 0], K[..., 0] = 64.0, 0.0
        K[0, 0, at, 0] = -3e38
    few = binding.query_step_plan(1, 1, L, 64, W, T, R, False, code)
    few = few.sums_offset[1] + few.sums_bytes
    full = ska.sinkhorn_attn_workspace_bytes(1, 1, L, 64, W, T, R, False, code)
    run = lambda n: ska.sinkhorn_attn_fwd(Q, K, V, W, T, R, 0.7, workspace=torch.empty(n, device="cuda", dtype=torch.uint8))
    results = [run(few), run(full)]
    try:
        for _ in range(20):
            ska.sinkhorn_attn_set_fused_half_steps(0, 1)
            again = run(full)
            torch.cuda.synchronize()
            chains = binding.query_chains()
            if chains.given_up == chains.launched:
                break
        assert chains.given_up == chains.launched
    finally:
        ska.sinkhorn_attn_set_fused_half_steps(0)
    results.append(again)
    away = (torch.arange(L, device="cuda") - at).abs()
    for route, (O, UV) in zip(("launched", "chain", "solved again"), results):
        # (the first half-step marks a query without a score as inactive; its scores are NaN all the same)
        # a half-step carries it W further; steps carry it to whole tiles of 32 and blocks
        for slot in range(1, 2 * (R + 1)):
            h = slot - (0 if what == "NaN" else 1)
            nan = torch.isnan(UV[0, 0, slot])
            assert nan[(away <= h * W) & ((away > 0) | (h != slot) | (slot % 2 == 1))].all(), (route, slot)
            assert not nan[away > h * (W + 160) + 160].any(), (route, slot)
        assert torch.isnan(O[0, 0, (away <= 3 * W) & (away > 0)]).all() and torch.isfinite(O[0, 0, away > 1200]).all(), route


FIRST_CHAIN = """
import threading
import torch
import paper_2605_08123_amd as ska
from paper_2605_08123_amd import binding
gen = torch.Generator(device="cuda")
gen.manual_seed(16)
N, L, W = 8, 700, 64
Q, K, V, G = (torch.randn((N, 1, L, 64), generator=gen, device="cuda").bfloat16() for _ in range(4))
ws = torch.empty(ska.sinkhorn_attn_workspace_bytes(N, 1, L, 64, W, 6, 2, False, 1), device="cuda", dtype=torch.uint8)
out = {n: torch.empty_like(Q) for n in ("O", "dQ", "dK", "dV")}
out["UV"] = torch.empty((N, 1, 6, L), device="cuda")
step = lambda T: ska.sinkhorn_attn_step(Q, K, V, G, W, T, 2, 0.6, workspace=ws, **out)
step(0)   # (whole steps, too few for a chain)
torch.cuda.synchronize()
assert binding.query_chains().launched == 0
errors, x, other = [], torch.zeros(1 << 16, device="cuda"), torch.cuda.Stream()
def call():
    try:
        with torch.cuda.stream(other):
            step(6)
    except Exception as e:
        errors.append(e)
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph, stream=torch.cuda.Stream(), capture_error_mode="global"):
    x.add_(1.0)
    thread = threading.Thread(target=call)
    thread.start()
    thread.join()
    x.mul_(2.0)
graph.replay()
torch.cuda.synchronize()
assert not errors and float(x[0]) == 2.0 and binding.query_chains().launched == 1
first = {n: t.clone() for n, t in out.items()}
step(6)
torch.cuda.synchronize()
assert binding.query_chains().launched == 2 and all(torch.equal(t, first[n]) for n, t in out.items())
print("fine")
"""


def test_a_first_chain_beside_another_threads_capture():
    """A process's first chain, in a thread while another one captures in global mode (memory for the gate is allocated then)."""
    import os
    import subprocess
    import sys
    run = subprocess.run([sys.executable, "-c", FIRST_CHAIN], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                         capture_output=True, text=True, timeout=100)
    assert run.returncode == 0 and "fine" in run.stdout, run.stderr
