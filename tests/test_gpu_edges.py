"""Sizes at which a kernel or a dispatch rule changes over, each against the fp64 oracle (bars of tests/measures.py)."""
import numpy as np
import pytest

import oracle
from paper_2605_08123_amd.workloads import Workload, make_inputs
from tests.measures import TOL, assert_per_tensor, floors
from tests.test_gpu_parity import check, rel, run_gpu

pytestmark = pytest.mark.gpu


def work(name, L, d, W, T, dtype, H=1, R=2, **kw):
    return Workload(name, 0, B=1, H=H, L=L, d=d, W=W, T=T, R=R, eps=0.8, dtype=dtype, **kw)


def base_cotangent_terms(q, k, v, g, W, R, eps, score, UV):
    """fp64: the terms whose sum is the dustbin element of the base cotangent (eta0[L]) of one problem with a scalar
    dustbin, by the reverse recurrences of Prop. 1 written out over the 2 W + 1 diagonals of the band."""
    L, c = q.shape[0], 1.0 / (eps * np.sqrt(q.shape[1]))
    diag = [(slice(max(0, -o), L - max(0, o)), slice(max(0, o), L - max(0, -o))) for o in range(-W, W + 1)]   # (rows, columns)
    S = [c * np.einsum("ld,ld->l", q[i], k[j]) for i, j in diag]
    us, vs = UV[0::2], UV[1::2]

    def rows(u, x, y):   # sum over the band of exp(S + u_i + x_j) y_j
        out = np.zeros(L)
        for s, (i, j) in zip(S, diag):
            out[i] += np.exp(s + u[i] + x[j]) * y[j]
        return out

    def cols(u, x, y):   # sum over the band of exp(S + u_i + x_j) y_i
        out = np.zeros(L)
        for s, (i, j) in zip(S, diag):
            out[j] += np.exp(s + u[i] + x[j]) * y[i]
        return out

    u, x = us[R], vs[R]
    ub, vb, ubL, vbL = np.zeros(L), np.zeros(L), 0.0, 0.0
    for s, (i, j) in zip(S, diag):
        sb = np.exp(s + u[i] + x[j]) * np.einsum("ld,ld->l", g[i], v[j])
        ub[i] += sb
        vb[j] += sb
    for t in range(R, 0, -1):
        u, x = us[t], vs[t]
        ub = ub - rows(u, x, vb) - np.exp(score + u[:L] + x[L]) * vbL
        ubL -= np.sum(np.exp(score + u[L] + x[:L]) * vb) + np.exp(score + u[L] + x[L]) * vbL
        x = vs[t - 1]
        vb = -cols(u, x, ub) - np.exp(score + u[L] + x[:L]) * ubL
        terms = -np.exp(score + u + x[L]) * np.append(ub, ubL)
        vbL, ub, ubL = terms.sum(), np.zeros(L), 0.0
    return terms


@pytest.mark.parametrize("dtype,d,L", [(t, d, L) for t, d in (("f32", 32), ("bf16", 32), ("bf16", 64))
                                       for L in (4094, 4095, 4096, 8190, 8191, 8192, 9000)]
                         + [("bf16", 32, L) for L in (65536, 65537, 73727)])
def test_dustbin_element_batches(dtype, d, L):
    """L + 1 values in batches of 4096 (mat-vecs, bf16 d = 32) or 8192 (half-steps), then single ones.  The half-steps'
    element is in the potentials.  The mat-vecs' reaches dQ and dK only through spokes of plan mass 1/L, so
    it is compared by itself, as eta0[L]: a sum of terms known to the tensors' tolerance each, whose errors are
    independent, hence within four times tol times the root of the sum of their squares.  In fp32 that bar sees a
    single value left out; in bf16, the same loop over the same fp32 vectors, a batch in most cases."""
    w = work("dustbin_edge", L, d, 5, 2, dtype, dustbin=True, dustbin_score=0.3)
    got, ref = check(w, want_eta0=True)
    q, k, v, g = (x[0, 0].astype(np.float64) for x in make_inputs(w))
    terms = base_cotangent_terms(q, k, v, g, w.W, w.R, w.eps, w.dustbin_score, ref["UV"][0, 0])
    bar = 4 * TOL[dtype] * np.sqrt(np.sum(terms ** 2))
    err = abs(got["eta0"][0, 0, L] - terms.sum())
    print(f"   eta0[L] {terms.sum():.4e} off {err:.1e} (bar {bar:.1e}; a term {np.median(np.abs(terms)):.1e})", flush=True)
    assert err <= bar
    assert dtype != "f32" or np.median(np.abs(terms)) > 2 * bar


@pytest.mark.parametrize("dtype,d,L", [("f32", 32, 1024), ("bf16", 64, 1025), ("bf16", 128, 2047), ("bf16", 32, 65),
                                       ("f32", 128, 130), ("f32", 64, 8200)])
def test_token_sums_chunks(dtype, d, L):
    """Weighted row sums in chunks of 1024 rows: whole, one row over, one short, less than a pass."""
    import torch

    import paper_2605_08123_amd as ska
    w = work("token_edge", L, d, 9, 3, dtype, dustbin=True)
    print(f"\n[case] {w} learned tokens", flush=True)
    arrays = make_inputs(w, 5)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, G = (torch.from_numpy(x).cuda().to(td) for x in arrays)
    toks = [np.random.default_rng(7 + i).standard_normal((1, 1, d)).astype(np.float32) for i in range(3)]
    tq, tk, tv = (torch.from_numpy(t).cuda() for t in toks)
    O, UV = ska.sinkhorn_attn_fwd_dustbin_token(Q, K, V, tq, tk, tv, w.W, w.T, w.R, w.eps)
    res = ska.sinkhorn_attn_bwd_dustbin_token(Q, K, V, tq, tk, tv, O, G, UV, w.W, w.T, w.R, w.eps)
    q, k, v, g = (t[0, 0].float().cpu().numpy().astype(np.float64) for t in (Q, K, V, G))
    ref = oracle.band_dustbin_token(q, k, v, g, *(t[0, 0] for t in toks), w.W, w.T, w.R, w.eps)
    for name, t in zip(("O", "dQ", "dK", "dV", "dq_db", "dk_db", "dv_db"), (O, *res)):
        e = rel(t[0, 0].float().cpu().numpy().astype(np.float64), ref[name])
        print(f"   {name} {e:.2e}", flush=True)
        assert e <= TOL[dtype], (name, e)


@pytest.mark.parametrize("d,H,L", [(64, 3, 22000), (32, 2, 32769), (64, 1, 65536)])
def test_output_map_block_sizes(d, H, L):
    """128-row blocks up to 65536 rows in a launch, 256-row blocks above."""
    w = work("apply_edge", L, d, 21, 2, "bf16", H=H)
    print(f"\n[case] {w}", flush=True)
    arrays = make_inputs(w, 3)
    got = run_gpu(w, arrays, one_call=True)
    ref = oracle.band_batched(*arrays, w.W, w.T, w.R, w.eps)
    assert_per_tensor(got, ref, w.dtype, floors(w.dtype, *arrays, ref["O"], w.eps), where=w.name)


@pytest.mark.parametrize("L,W,R", [(31, 7, 2), (33, 40, 1), (127, 31, 2), (129, 32, 3), (161, 64, 2), (1000, 95, 5)])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64), ("f32", 128)])
def test_double_buffered_matrix_sweeps(dtype, d, L, W, R):
    """Ragged last tiles and band edges; modifier terms as pack columns (bf16, R <= 2), in one group of four or in two."""
    check(work("generic_edge", L, d, W, 3, dtype, H=2, R=R))


@pytest.mark.parametrize("H,L,W", [(1, 65536, 9), (1, 65537, 200), (1, 98304, 9), (1, 98305, 9), (400, 300, 9), (1, 131072, 192),
                                   (2, 65600, 9)])
def test_vector_sweep_block_sizes_wide_heads(H, L, W):
    """d = 128: 128-row blocks while 512 of them hold a launch (768 with a narrow band), 256-row ones while 512 of those do."""
    w = work("block_edge", L, 128, W, 2, "bf16", H=H)
    print(f"\n[case] {w}", flush=True)
    arrays = make_inputs(w, 3)
    got = run_gpu(w, arrays, one_call=True)
    ref = oracle.band_batched(*arrays, w.W, w.T, w.R, w.eps)
    assert_per_tensor(got, ref, w.dtype, floors(w.dtype, *arrays, ref["O"], w.eps), where=w.name)


@pytest.mark.parametrize("L", [65536, 100000])
def test_potentials_that_jump_between_blocks_of_128_rows(L):
    """One partner per token and row targets of 1 and e^50 in turn, 128 rows each, against column targets of 1: after two
    steps the potentials of neighbouring groups are 100 apart, more than one stabiliser for both could carry, and
    the plan is the identity all the same.  256-row blocks (L = 100000) have to take one per 128 rows."""
    import torch

    import paper_2605_08123_amd as ska
    print(f"\n[case] stabiliser range L={L}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    Q, K, V = (torch.randn((1, 1, L, 128), generator=gen, device="cuda").bfloat16() for _ in range(3))
    log_a = 50.0 * ((torch.arange(L, device="cuda") // 128) % 2).float().view(1, 1, L)
    O, UV = ska.sinkhorn_attn_fwd_marginals(Q, K, V, log_a, torch.zeros_like(log_a), 0, 1, 1, 1.0)
    assert torch.isfinite(UV).all()
    assert float((O.float() - V.float()).norm() / V.float().norm()) < TOL["bf16"]


@pytest.mark.parametrize("R", [1, 2])
def test_wide_heads_keep_modifier_terms_in_fp32(R):
    """One partner per token, all queries and all keys alike: the plan is the identity with entries that bf16 holds
    exactly, Z and the modifier terms are equal, and dQ = dK = 0.  What is left is the rounding of Z minus the
    terms: sums of 128 products of order one in fp32, below 2^-20 of Z with room to spare (2^-23 each); terms kept
    to 16 bits leave 2^-18.8 (with fp32 terms 2^-22.7)."""
    import torch

    import paper_2605_08123_amd as ska
    L, d, eps = 300, 128, 0.8
    print(f"\n[case] modifier terms d={d} R={R}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    q, k = (torch.randn((1, 1, 1, d), generator=gen, device="cuda").bfloat16() for _ in range(2))
    Q, K = (x.expand(1, 1, L, d).contiguous() for x in (q, k))
    V, G = (torch.randn((1, 1, L, d), generator=gen, device="cuda").bfloat16() for _ in range(2))
    O, UV, dQ, dK, dV = ska.sinkhorn_attn_step(Q, K, V, G, 0, 3, R, eps)
    assert torch.equal(O, V) and torch.equal(dV, G)
    z = (G.double() * V.double()).sum(-1, keepdim=True) / (eps * d ** 0.5)
    for got, other in ((dQ, K), (dK, Q)):
        left = float(got.double().norm() / (z * other.double()).norm())
        print(f"   left of Z: 2^{np.log2(max(left, 1e-30)):.1f}", flush=True)
        assert left <= 2.0 ** -20


@pytest.mark.parametrize("N,L", [(1, 70), (2, 33), (1000, 70)])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_an_infinity_in_the_last_row_stays_in_its_column(d, N, L):
    """Rows past the end of a ragged last tile are stand-ins for the last row, times a plan entry of zero: an infinite
    value of V there may not reach any other column of O, nor one of dO any other column of dV (both block sizes)."""
    import torch

    import paper_2605_08123_amd as ska
    print(f"\n[case] infinite payload N={N} L={L} d={d}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    Q, K, V, G = (torch.randn((1, N, L, d), generator=gen, device="cuda").bfloat16() for _ in range(4))
    V[..., L - 1, d - 2] = float("inf")
    O, UV = ska.sinkhorn_attn_fwd(Q, K, V, 5, 3, 2, 0.8)
    V[..., L - 1, d - 2] = 1.0
    G[..., L - 1, d - 3] = float("inf")
    dQ, dK, dV = ska.sinkhorn_attn_bwd(Q, K, V, O, G, UV, 5, 3, 2, 0.8)
    for got, at in ((O, d - 2), (dV, d - 3)):
        cols = (~torch.isfinite(got)).flatten(0, 2).any(0).nonzero().flatten().tolist()
        assert cols == [at], cols
