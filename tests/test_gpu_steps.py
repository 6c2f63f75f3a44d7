"""Whole Sinkhorn steps from one evaluation of the scores against the half-steps they replace.  A forward whose workspace
holds the prescaled operand and nothing more runs half-step by half-step, so both routes can be compared over every form
the steps accept: lengths, marginals, masks, a dustbin, both storage types, every head dimension, the sizes at which
a block shape or a segment length changes over.

Bound: both routes compute the same potentials in fp32.  A half-step adds to a potential at most the rounding of its
exponents (three terms of size M, the largest score or potential in base 2), of a sum of 2 W + 2 terms and of one
exponential and one logarithm: (2 W + 20 + 4 M) 2^-24.  The half-steps do not enlarge a difference of potentials, so over
2 (T + R) of them two routes are at most twice the sum apart."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHORT = [  # kind, dtype, d, N, L, W, T, R
    ("plain", "bf16", 64, 1, 31, 7, 3, 2), ("plain", "bf16", 64, 2, 65, 0, 2, 1), ("plain", "bf16", 64, 3, 129, 32, 1, 2),
    ("plain", "bf16", 64, 2, 500, 33, 0, 3), ("plain", "bf16", 64, 2, 701, 64, 5, 2), ("plain", "bf16", 64, 2, 700, 65, 4, 1),
    ("plain", "bf16", 64, 1, 999, 96, 3, 2), ("plain", "bf16", 64, 1, 1000, 128, 2, 2), ("plain", "bf16", 64, 1, 1000, 129, 3, 2),
    ("plain", "bf16", 64, 1, 1025, 224, 4, 2), ("plain", "bf16", 64, 1, 1023, 256, 3, 2), ("plain", "bf16", 64, 1, 400, 5000, 3, 2),
    ("plain", "bf16", 32, 2, 333, 40, 3, 2), ("plain", "bf16", 32, 2, 777, 100, 3, 2), ("plain", "bf16", 32, 1, 900, 250, 3, 2),
    ("plain", "bf16", 128, 2, 333, 40, 3, 2), ("plain", "bf16", 128, 1, 777, 127, 3, 2), ("plain", "bf16", 128, 1, 900, 200, 3, 2),
    ("plain", "bf16", 128, 1, 900, 256, 3, 2), ("plain", "bf16", 64, 2, 1100, 300, 3, 2), ("plain", "bf16", 32, 1, 1500, 480, 3, 1),
    ("plain", "bf16", 64, 1, 1500, 481, 2, 1), ("plain", "f32", 32, 1, 1200, 400, 2, 2), ("varlen", "bf16", 64, 4, 900, 350, 3, 1),
    ("plain", "f32", 32, 1, 256, 16, 8, 2), ("plain", "f32", 32, 2, 611, 99, 3, 2),
    ("plain", "f32", 32, 1, 800, 256, 3, 2), ("plain", "f32", 64, 2, 300, 64, 3, 2), ("plain", "f32", 64, 1, 700, 111, 3, 2),
    ("plain", "f32", 64, 1, 700, 255, 3, 2), ("plain", "f32", 128, 1, 300, 50, 3, 2), ("plain", "f32", 128, 1, 500, 128, 3, 2),
    ("varlen", "bf16", 64, 4, 600, 50, 3, 2), ("varlen", "f32", 64, 4, 500, 100, 2, 2), ("varlen", "bf16", 64, 4, 900, 200, 3, 1),
    ("marginals", "bf16", 64, 2, 600, 100, 3, 2), ("marginals", "f32", 32, 2, 400, 20, 2, 2), ("masked", "bf16", 64, 2, 500, 31, 3, 2),
    ("masked", "f32", 64, 2, 700, 128, 3, 2), ("dustbin", "bf16", 64, 2, 701, 30, 3, 2), ("dustbin", "f32", 32, 2, 500, 100, 1, 2),
    ("dustbin", "bf16", 128, 2, 600, 222, 2, 2), ("dustbin", "bf16", 64, 1, 9000, 256, 2, 1),
    ("plain", "bf16", 64, 1, 1000, 160, 3, 2), ("plain", "bf16", 64, 2, 777, 161, 3, 2), ("plain", "bf16", 32, 1, 900, 192, 3, 1),
    ("plain", "bf16", 128, 1, 700, 150, 3, 2), ("dustbin", "bf16", 128, 1, 900, 180, 2, 1), ("plain", "f32", 64, 1, 700, 160, 3, 2),
    ("plain", "f32", 64, 1, 700, 161, 2, 2), ("dustbin", "f32", 64, 2, 300, 90, 2, 2), ("plain", "f32", 128, 1, 300, 32, 3, 2)]
LONG = [  # other block shapes; segments of several blocks, also ragged ones and ones that end inside a problem
    ("plain", "bf16", 64, 1, 50000, 20, 2, 1), ("plain", "bf16", 64, 1, 50001, 100, 2, 2), ("plain", "bf16", 64, 1, 66000, 97, 3, 1),
    ("plain", "bf16", 64, 3, 40001, 128, 2, 1), ("plain", "bf16", 64, 1, 17000, 130, 2, 1), ("plain", "bf16", 64, 1, 40000, 256, 3, 1),
    ("plain", "bf16", 64, 2, 70001, 200, 2, 1), ("plain", "bf16", 64, 300, 700, 130, 2, 1), ("plain", "bf16", 32, 2, 40000, 100, 2, 1),
    ("plain", "bf16", 32, 1, 60000, 256, 2, 1), ("plain", "bf16", 128, 1, 33000, 60, 2, 1), ("plain", "bf16", 128, 1, 33000, 120, 2, 1),
    ("plain", "bf16", 128, 1, 20000, 120, 2, 1), ("plain", "bf16", 128, 1, 33000, 256, 2, 1), ("plain", "bf16", 128, 3, 30001, 200, 3, 1),
    ("plain", "f32", 64, 1, 40001, 256, 2, 1), ("varlen", "bf16", 128, 4, 30000, 130, 3, 1), ("dustbin", "bf16", 128, 1, 40000, 250, 2, 1),
    ("plain", "bf16", 128, 600, 100, 130, 2, 1), ("plain", "f32", 32, 1, 60000, 100, 2, 1), ("plain", "f32", 32, 1, 60000, 256, 2, 1),
    ("plain", "f32", 64, 1, 40000, 128, 2, 1), ("plain", "f32", 128, 1, 20000, 64, 2, 1), ("varlen", "bf16", 64, 4, 40000, 256, 3, 1),
    ("varlen", "bf16", 64, 8, 20000, 70, 2, 1), ("marginals", "bf16", 64, 2, 70000, 128, 2, 1), ("masked", "bf16", 64, 2, 70000, 129, 2, 1),
    ("dustbin", "bf16", 64, 1, 70000, 128, 2, 1), ("dustbin", "f32", 32, 1, 60000, 200, 2, 1),
    ("plain", "bf16", 64, 1, 17000, 170, 2, 1), ("plain", "bf16", 64, 1, 17001, 200, 2, 1), ("plain", "bf16", 64, 1, 40000, 150, 2, 2),
    ("dustbin", "bf16", 64, 1, 40001, 190, 2, 1), ("plain", "bf16", 128, 1, 40001, 160, 2, 1), ("dustbin", "bf16", 128, 1, 20000, 90, 2, 1),
    ("plain", "bf16", 128, 1, 40000, 70, 2, 1), ("plain", "bf16", 128, 1, 34000, 170, 2, 2), ("dustbin", "bf16", 64, 1, 70000, 96, 2, 1),
    ("plain", "f32", 64, 1, 10000, 170, 2, 1), ("plain", "bf16", 128, 1, 40000, 16, 2, 1), ("dustbin", "bf16", 64, 1, 60000, 20, 2, 1),
    # padded batches whose items are all short, or one long among short ones (the segments are cut from the valid rows), with
    # targets as well
    ("short", "bf16", 64, 4, 20000, 256, 3, 1), ("short", "bf16", 64, 8, 16001, 128, 2, 2), ("short", "bf16", 128, 4, 20000, 200, 2, 1),
    ("short", "f32", 64, 3, 30000, 250, 2, 1), ("short", "f32", 32, 4, 20001, 100, 2, 1), ("short", "bf16", 32, 5, 20001, 256, 2, 1),
    ("short targets", "bf16", 64, 4, 20000, 200, 3, 1), ("short targets", "f32", 64, 3, 30000, 250, 2, 1),
    ("short", "bf16", 64, 8, 30000, 200, 2, 1), ("short", "bf16", 64, 14, 30000, 200, 2, 1), ("short", "bf16", 64, 300, 700, 256, 2, 1),
    ("uneven", "bf16", 64, 8, 30000, 200, 2, 1), ("uneven", "bf16", 64, 1, 200000, 256, 2, 1), ("uneven", "bf16", 128, 5, 30000, 150, 2, 1),
    ("uneven", "bf16", 64, 33, 12000, 256, 2, 1), ("uneven", "bf16", 64, 7, 60000, 128, 2, 1), ("uneven", "f32", 64, 5, 30000, 250, 2, 1),
    ("uneven", "bf16", 64, 16, 30000, 130, 2, 1)]


HALF_STEPS = [("plain", "bf16", 64, 1, 1500, 481, 2, 1)]   # the others run whole steps


@pytest.mark.parametrize("case", SHORT + LONG, ids=lambda c: "-".join(map(str, c)))
def test_steps_equal_half_steps(case):
    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    kind, dtype, d, N, L, W, T, R = case
    print(f"\n[case] {case}", flush=True)
    whole = binding.query_step_plan(N, 1, L, d, W, T, R, kind == "dustbin", 0 if dtype == "f32" else 1,
                                    lengths=kind[:5] in ("varle", "short", "uneve")).whole_steps
    assert bool(whole) == (case not in HALF_STEPS)   # (both sides of the rule's lines)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(17)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V = (torch.randn((N, 1, L, d), generator=gen, device="cuda").to(td) for _ in range(3))
    eps, db = 0.7, kind == "dustbin"
    la = lb = lq = lk = mq = mk = None
    if kind == "varlen":   # one item without queries, one with a single key, the others anything
        lq, lk = (torch.randint(1, L + 1, (N,), generator=gen, device="cuda").int() for _ in range(2))
        lq[0], lk[1] = 0, 1
        lq[2], lk[2] = L // 3, L   # rows end well before the columns do
    if kind.startswith("short"):
        lq, lk = (torch.randint(L // 12, L // 8, (N,), generator=gen, device="cuda").int() for _ in range(2))
        lk[-1] = 3   # (less than a block, and queries far beyond it)
    if kind == "uneven":   # half of them empty or nearly so, at both ends one of all rows
        lq, lk = (torch.randint(0, 40, (N,), generator=gen, device="cuda").int() for _ in range(2))
        lq[::3], lk[::3] = L - 5, L
        lq[N // 2:N // 2 + 2] = lk[N // 2:N // 2 + 2] = L // 2
    if kind in ("marginals", "short targets"):
        a, b = (torch.rand((N, 1, L), generator=gen, device="cuda") + 0.5 for _ in range(2))
        la, lb = a.log(), (b * a.sum(-1, keepdim=True) / b.sum(-1, keepdim=True)).log()
    if kind == "masked":
        mq, mk = ((torch.rand((N, L), generator=gen, device="cuda") > 0.3).to(torch.uint8) for _ in range(2))

    def forward(nbytes):
        ws = None if nbytes is None else torch.empty(nbytes, device="cuda", dtype=torch.uint8)
        if kind == "masked":
            return ska.sinkhorn_attn_fwd_masked(Q, K, V, mq, mk, W, T, R, eps, workspace=ws)
        return ska.sinkhorn_attn_fwd_varlen(Q, K, V, la, lb, lq, lk, W, T, R, eps, db, 0.3, workspace=ws)

    O, UV = forward(None)
    O0, UV0 = forward(max(16, Q.numel() * 2 if dtype == "bf16" else 16))   # room for the prescaled operand alone
    torch.cuda.synchronize()
    assert torch.equal(torch.isneginf(UV), torch.isneginf(UV0))
    x, y = (torch.where(torch.isneginf(z), 0.0, z.double()) for z in (UV, UV0))
    assert torch.isfinite(x).all() and torch.isfinite(y).all()
    score = float((Q.double().norm(dim=-1).max() * K.double().norm(dim=-1).max()) / (eps * d ** 0.5))
    M = 1.4427 * max(score, float(y.abs().max()))
    # a dustbin's row and column are sums over all tokens, taken in a tree: a thread's own terms (one per block of its segment,
    # L / 256 in a half-step's element), its wavefront's, its workgroup's, the segments'.  (A segment left out of
    # ("dustbin", L = 70000, W = 128) would move the dustbin's potentials by 1 / 137, more than ten times the bound.)
    terms = 2 * min(W, L) + 1 + (L // 256 + 64 if db else 0)
    bound = 2 * 2 * (T + R) * (terms + 20 + 4 * M) * 2.0 ** -24
    err = float((x - y).abs().max())
    print(f"   |UV - UV0| {err:.1e} (bound {bound:.1e}), M {M:.0f}", flush=True)
    assert err <= bound
    # a plan entry moves by at most the two potentials' differences, and (bf16) to the other neighbour
    rel = float((O.double() - O0.double()).norm() / O0.double().norm())
    assert rel <= 2 * bound + (2.0 ** -8 if dtype == "bf16" else 0.0), rel


def test_steps_take_spread_potentials():
    """Row targets of 1 and e^60 in turn, row by row, against a column target of 1: the potentials inside one block are
    60 apart, which a stabiliser per row carries in either direction (one partner per token: the plan is the identity)."""
    import torch

    import paper_2605_08123_amd as ska
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    L = 3000
    Q, K, V = (torch.randn((1, 1, L, 64), generator=gen, device="cuda").bfloat16() for _ in range(3))
    la = 60.0 * (torch.arange(L, device="cuda") % 2).float().view(1, 1, L)
    O, UV = ska.sinkhorn_attn_fwd_marginals(Q, K, V, la, torch.zeros_like(la), 0, 3, 2, 1.0)
    assert torch.isfinite(UV).all()
    u, v = UV[0, 0, 4].double(), UV[0, 0, 5].double()
    s = (Q.double() * K.double()).sum(-1)[0, 0] / 8.0
    # after a column step the column sums are one; scores from a bf16 copy of Q: 2^-9 of the terms' sizes
    assert float((u + v + s).abs().max()) <= 2.0 ** -9 * float((Q.double() * K.double()).abs().sum(-1).max() / 8.0) + 1e-4


@pytest.mark.parametrize("dtype,L", [("bf16", 1024), ("f32", 1000), ("bf16", 70000)])
def test_first_step_of_a_continuation_stage_takes_the_half_steps_range(dtype, L):
    """A stage raises the plan to the ratio of the two eps.  Every second row here spreads evenly over its 257 partners, so
    that at a ratio of 20 its entries go down to e^-111 and its sum to e^-105; the other rows match one partner each and have
    potentials e^100 larger, which the half-steps' common stabiliser takes.  Finite, and the same as by half-steps."""
    import torch

    import paper_2605_08123_amd as ska
    W, d, R, eps_s = 128, 64, 2, [10.0, 0.5, 0.5]
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    r = torch.randn((L, d), generator=gen, device="cuda")
    r[:, 0] = 0
    r /= r.norm(dim=-1, keepdim=True)
    e0 = torch.zeros(d, device="cuda")
    e0[0] = 1
    even = (torch.arange(L, device="cuda") % 2 == 0)[:, None]
    Q, K, V = (x.view(1, 1, L, d).to(td).contiguous() for x in (torch.where(even, 30.5 * e0, 31 * r), 30 * e0 + 31 * r, r))
    for T_stage in ([3, 0, 2], [3, 0, 0], [3, 2, 1]):
        O, UV = ska.sinkhorn_attn_fwd_eps_schedule(Q, K, V, W, eps_s, T_stage, R, 0.5)
        ws = torch.empty(max(16, Q.numel() * 2 if dtype == "bf16" else 16), device="cuda", dtype=torch.uint8)
        O0, UV0 = ska.sinkhorn_attn_fwd_eps_schedule(Q, K, V, W, eps_s, T_stage, R, 0.5, workspace=ws)
        assert torch.isfinite(UV0).all() and torch.isfinite(UV).all(), T_stage
        M = 1.4427 * max(31.0 * 31.0 * 1.1 / (0.5 * d ** 0.5), float(UV0.abs().max()))
        bound = 2 * 2 * (sum(T_stage) + R) * (2 * W + 21 + 4 * M) * 2.0 ** -24
        assert float((UV - UV0).abs().max()) <= bound, T_stage


@pytest.mark.parametrize("L,W,d", [(256, 16, 32), (256, 32, 32), (700, 30, 128)])
def test_fp32_steps_are_no_further_from_64_bits_than_half_steps(L, W, d):
    """The same 24 problems both ways against the oracle: the rms distance of O."""
    import torch

    import oracle
    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd.workloads import Workload, make_inputs
    w = Workload("fp32", 41, 1, 24, L, d, W, 8, 2, 1.0, "f32")
    arrays = make_inputs(w, 41)
    ref = oracle.band_batched(*arrays, w.W, w.T, w.R, w.eps)["O"]
    Q, K, V = (torch.from_numpy(x).cuda() for x in arrays[:3])
    err = []
    for ws in (None, torch.empty(16, device="cuda", dtype=torch.uint8)):
        O, _ = ska.sinkhorn_attn_fwd(Q, K, V, w.W, w.T, w.R, w.eps, workspace=ws)
        err.append(float(np.sqrt(np.mean((O.cpu().numpy().astype(np.float64) - ref) ** 2))))
    print(f"\n   steps {err[0]:.3e}, half-steps {err[1]:.3e}", flush=True)
    assert err[0] <= err[1]


LOWEST = -3.4028234663852886e38
TARGETS = [  # dtype, d, L, W, which tokens have the target e^x, x
    *[("bf16", 64, 1000, 64, k, x) for k in ("rows", "columns", "both") for x in (-80.0, -100.0, -1e4, LOWEST, float("-inf"))],
    *[("f32", 64, 1000, 64, k, x) for k in ("rows", "columns", "both") for x in (-30.0, -84.0, -1e4)],
    ("bf16", 64, 70000, 128, "both", -100.0), ("bf16", 64, 40000, 256, "both", -90.0), ("bf16", 64, 17000, 200, "both", -1e4),   # segments, blocks
    ("bf16", 128, 33000, 200, "both", -100.0), ("bf16", 128, 33000, 100, "both", -90.0), ("f32", 64, 40000, 256, "both", -100.0),
    ("f32", 32, 60000, 100, "both", -90.0), ("bf16", 64, 1000, 400, "both", -100.0),
    ("bf16", 64, 1000, 64, "all", -60.0), ("f32", 64, 1000, 100, "all", -60.0), ("bf16", 64, 1000, 64, "end", -60.0)]


@pytest.mark.parametrize("case", TARGETS, ids=lambda c: "-".join(map(str, c)))
def test_steps_take_small_targets(case):
    """Targets of e^x among unit ones: every sixteenth row and / or column, all of them, or rows and columns from some token on.
    Against the half-steps, which take the largest potential of a block as stabiliser; token by token, since a
    potential near x is known to its own rounding and the others as without small targets."""
    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    dtype, d, L, W, which, x = case
    print(f"\n[case] {case}", flush=True)
    td, code = (torch.float32, 0) if dtype == "f32" else (torch.bfloat16, 1)
    T, R, eps = 3, 2, 1.0
    assert binding.query_step_plan(1, 1, L, d, W, T, R, False, code).whole_steps
    gen = torch.Generator(device="cuda")
    gen.manual_seed(29)
    Q, K, V = (torch.randn((1, 1, L, d), generator=gen, device="cuda").to(td) for _ in range(3))
    i = torch.arange(L, device="cuda")
    hit = {"all": i >= 0, "end": i >= 700}.get(which)
    la, lb = torch.zeros((2, 1, 1, L), device="cuda")
    la[..., hit if hit is not None else i % 16 == 0] = x if which != "columns" else 0.0
    lb[..., hit if hit is not None else i % 16 == 5] = x if which != "rows" else 0.0

    def forward(nbytes):
        ws = None if nbytes is None else torch.empty(nbytes, device="cuda", dtype=torch.uint8)
        return ska.sinkhorn_attn_fwd_marginals(Q, K, V, la, lb, W, T, R, eps, workspace=ws)

    O, UV = forward(None)
    O0, UV0 = forward(max(16, Q.numel() * 2 if dtype == "bf16" else 16))   # half-steps
    assert torch.equal(torch.isneginf(UV), torch.isneginf(UV0))
    a, b = (torch.where(torch.isneginf(z), 0.0, z.double()) for z in (UV, UV0))
    assert torch.isfinite(a).all() and torch.isfinite(b).all() and torch.isfinite(O.float()).all()
    score = float((Q.double().norm(dim=-1).max() * K.double().norm(dim=-1).max()) / (eps * d ** 0.5))
    M = 1.4427 * torch.clamp(b.abs(), min=score + (abs(x) if which in ("all", "end") else 0.0))
    # (the bound of test_steps_equal_half_steps; a potential as large as its target has one rounding of its own per update more)
    bound = 2 * 2 * (T + R) * (2 * W + 1 + 20 + 4 * M) * 2.0 ** -24
    worst = float(((a - b).abs() / bound).max())
    print(f"   |UV - UV0| at most {worst:.2f} of the bound", flush=True)
    assert worst <= 1.0
    rel = float((O.double() - O0.double()).norm() / O0.double().norm())
    assert rel <= 2 * 2 * 2 * (T + R) * (2 * W + 21 + 4 * 1.4427 * (score + 64)) * 2.0 ** -24 + (2.0 ** -8 if dtype == "bf16" else 0.0), rel


SPLIT = [  # dtype, d, N, L, W, R, lengths of the first and of the second half of the problems (0: a padded item without tokens)
    ("bf16", 64, 5, 20000, 128, 2, 40, 20000), ("bf16", 64, 5, 20000, 128, 1, 20000, 0), ("bf16", 64, 2, 60001, 256, 2, 0, 60001),
    ("bf16", 64, 3, 9000, 60, 3, 9000, 300), ("bf16", 128, 3, 17000, 256, 2, 17000, 1), ("f32", 64, 3, 5001, 100, 2, 5001, 17),
    ("bf16", 64, 3, 4001, 400, 2, 33, 4001), ("bf16", 64, 5, 4001, 470, 1, 4001, 0)]   # (these two: sums over the backward's vectors)


@pytest.mark.parametrize("case", SPLIT, ids=lambda c: "-".join(map(str, c)))
def test_split_step_with_unequal_halves_equals_one_stream(case):
    """Without a dustbin the two halves of a one-call step run forward and backward without waiting for each other: the
    half that is done first must not write over what the other one still reads.  The same bits as on one stream."""
    import torch

    import paper_2605_08123_amd as ska
    from paper_2605_08123_amd import binding
    dtype, d, N, L, W, R, len0, len1 = case
    print(f"\n[case] {case}", flush=True)
    td, code = (torch.float32, 0) if dtype == "f32" else (torch.bfloat16, 1)
    plan = binding.query_step_plan(N, 1, L, d, W, 6, R, False, code, one_call=True, lengths=True)
    assert plan.whole_steps and bool(plan.sums_apart) == (W <= 256)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(23)
    Q, K, V, G = (torch.randn((N, 1, L, d), generator=gen, device="cuda").to(td) for _ in range(4))
    lens = torch.tensor([len0] * (N // 2) + [len1] * (N - N // 2), dtype=torch.int32, device="cuda")
    ws = torch.empty(ska.sinkhorn_attn_workspace_bytes(N, 1, L, d, W, 6, R, False, code), device="cuda", dtype=torch.uint8)

    def step(streams):
        ska.sinkhorn_attn_set_streams(streams)
        ws.fill_(255)   # (NaN wherever a float is read that was not written)
        out = ska.sinkhorn_attn_step(Q, K, V, G, W, 6, R, 0.7, False, 0.0, None, None, lens, lens, workspace=ws)
        torch.cuda.synchronize()
        return out

    try:
        ska.sinkhorn_attn_set_split_min_edges(0.0)
        one = step(1)
        for _ in range(3):
            for x, y in zip(step(2), one):
                assert torch.isfinite(y.float()).all() and torch.equal(x, y)
    finally:
        ska.sinkhorn_attn_set_streams(2)
        ska.sinkhorn_attn_set_split_min_edges(5e7)
