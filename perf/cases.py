"""The work this library is used for, as cases that can be timed and compared.

A case is one call pattern of the public entry points (`paper_2605_08123_amd.binding`) at one size: a
forward for inference, a forward and a backward as two calls (an autograd function around the
library), or the one-call step for a cotangent known beforehand.  `listed()` names the cases that are
quoted, `draw(rng)` gives another one of the same ranges, `prepare(case, seed)` makes what a program
holds before the call, `run(state)` is one pass, `work(case)` what the pass cannot do without and
`tolerance(case)` what another implementation of the same precision may differ by.

Fields of a case:
  call   "step" (one call, caller's buffers), "fwd" or "fwd_bwd" (results allocated per call)
  kind   "plain"; "varlen" (padded batch, a length per item and side); "marginals" (row and column
         targets); "masked" (inactive tokens); "dustbin" (scalar score); "token" (learned dustbin)
  B, H, L, d, W, T, R, eps, dtype ("bf16" or "f32")
  dist   "normal" (unit normal), "mid" (Q, K of variance 1/sqrt(d)), "alphabet" (20 embedded symbols)
"""
import math

import torch

import paper_2605_08123_amd as ska


def _case(name, call, kind, B, H, L, d, W, T, R, eps, dtype, dist="normal"):
    return {"name": name, "call": call, "kind": kind, "B": B, "H": H, "L": L, "d": d, "W": W, "T": T, "R": R,
            "eps": eps, "dtype": dtype, "dist": dist}


def listed():
    return [
        # the smallest configuration of the benchmark: one short fp32 sequence; launches and latency
        _case("tiny_f32", "step", "plain", 1, 1, 256, 32, 16, 8, 2, 1.0, "f32"),
        # inference on a short batch of a length that fits no tile
        _case("short_fwd", "fwd", "plain", 1, 8, 701, 64, 64, 16, 2, 0.5, "bf16"),
        # a training step of a small model: 32 problems of ordinary length (benchmark configuration)
        _case("mid", "step", "plain", 4, 8, 4096, 64, 128, 16, 2, 0.5, "bf16", "mid"),
        # the same through an autograd function (two calls, results allocated), ragged sizes
        _case("ragged_train", "fwd_bwd", "plain", 2, 8, 3001, 64, 100, 16, 2, 0.5, "bf16"),
        # a padded batch of sequences of different lengths
        _case("varlen", "step", "varlen", 8, 4, 2048, 64, 128, 16, 2, 0.5, "bf16"),
        # protein-like pairs with one dustbin token per side (benchmark configuration)
        _case("dustbin", "step", "dustbin", 2, 4, 16384, 64, 256, 20, 2, 0.5, "bf16", "alphabet"),
        # learned dustbin tokens trained through autograd
        _case("token_train", "fwd_bwd", "token", 2, 4, 5000, 64, 128, 16, 2, 0.5, "bf16"),
        # fp32 storage at an ordinary size (reference runs, gradient checks at scale)
        _case("f32_train", "fwd_bwd", "plain", 1, 8, 4096, 64, 128, 16, 2, 1.0, "f32"),
        # wide heads
        _case("wide_head", "step", "plain", 1, 8, 16384, 128, 256, 20, 2, 0.5, "bf16"),
        # long context (benchmark configuration)
        _case("long", "step", "plain", 1, 4, 65536, 64, 256, 20, 2, 0.5, "bf16"),
        # the benchmark's headline configuration: one device's share of the data-parallel run
        _case("paper", "step", "plain", 1, 2, 262144, 64, 256, 20, 2, 0.5, "bf16"),
        # its long-context shape with a half-band of 1024
        _case("paper_w1024", "step", "plain", 1, 1, 262144, 64, 1024, 15, 2, 0.5, "bf16"),
    ]


def _cost(c):
    """Band edges times sweeps, weighted by the head dimension and the storage type."""
    w = min(c["W"], c["L"] - 1)
    e = float(c["B"] * c["H"]) * c["L"] * (2 * w + 1)
    return e * (c["T"] + c["R"] + 4) * (1.0 + c["d"] / 64.0) * (8.0 if c["dtype"] == "f32" else 1.0)


def draw(rng):
    kind = rng.choices(["plain", "varlen", "marginals", "dustbin", "masked", "token"], [10, 3, 2, 3, 1, 1])[0]
    call = rng.choice(["fwd", "fwd_bwd"] if kind in ("masked", "token") else ["step", "step", "fwd", "fwd_bwd"])
    dtype = rng.choices(["bf16", "f32"], [4, 1])[0]
    c = {"call": call, "kind": kind, "B": rng.choice([1, 1, 2, 4, 8]), "H": rng.choice([1, 2, 4, 8]),
         "L": int(round(math.exp(rng.uniform(math.log(200.0), math.log(262144.0))))),
         "d": rng.choices([32, 64, 128], [1, 4, 1])[0],
         "W": int(round(math.exp(rng.uniform(math.log(16.0), math.log(1024.0))))),
         "T": rng.randint(8, 20), "R": rng.choices([1, 2, 3], [1, 6, 1])[0],
         "eps": rng.choice([0.5, 0.7, 1.0]), "dtype": dtype, "dist": rng.choices(["normal", "mid"], [3, 1])[0]}
    cap = _cost(_case("", "step", "plain", 1, 1, 262144, 64, 1024, 15, 2, 0.5, "bf16"))
    while _cost(c) > cap or c["B"] * c["H"] * c["L"] > 1 << 20:   # fewer problems first, then shorter ones
        if c["B"] > 1:
            c["B"] //= 2
        elif c["H"] > 1:
            c["H"] //= 2
        else:
            c["L"] = int(c["L"] / 1.3)
    c["W"] = min(c["W"], c["L"] - 1)
    return c


def _inputs(c, gen, td):
    shape = (c["B"], c["H"], c["L"], c["d"])
    new = lambda s=shape: torch.randn(s, generator=gen, device="cuda", dtype=torch.float32)
    if c["dist"] == "alphabet":   # token ids over 20 symbols, looked up in per-head random tables
        x, y = (torch.randint(20, shape[:3], generator=gen, device="cuda") for _ in range(2))
        out = []
        for ids in (x, y, y, x):
            tab = new(shape[:2] + (20, shape[3]))
            out.append(torch.gather(tab, 2, ids[..., None].expand(shape)))
    else:
        s = c["d"] ** -0.25 if c["dist"] == "mid" else 1.0
        out = [new() * s, new() * s, new(), new()]
    return [t.to(td).contiguous() for t in out]


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    td = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    Q, K, V, G = _inputs(c, gen, td)
    B, H, L, d = Q.shape
    db = c["kind"] in ("dustbin", "token")
    st = {"case": c, "Q": Q, "K": K, "V": V, "dO": G,
          # scratch a program keeps between calls
          "ws": torch.empty(ska.sinkhorn_attn_workspace_bytes(B, H, L, d, c["W"], c["T"], c["R"], db,
                                                              0 if td == torch.float32 else 1),
                            device="cuda", dtype=torch.uint8)}
    if c["call"] == "step":
        st["out"] = {n: torch.empty_like(Q) for n in ("O", "dQ", "dK", "dV")}
        st["out"]["UV"] = torch.empty((B, H, 2 * (c["R"] + 1), L + int(db)), device="cuda", dtype=torch.float32)
    if c["kind"] == "varlen":
        st["len_q"], st["len_k"] = (torch.randint((L + 1) // 2, L + 1, (B,), generator=gen, device="cuda").int()
                                    for _ in range(2))
    if c["kind"] == "marginals":
        a, b = (torch.rand((B, H, L), generator=gen, device="cuda") + 0.5 for _ in range(2))
        b *= a.sum(-1, keepdim=True) / b.sum(-1, keepdim=True)   # compatible totals
        st["log_a"], st["log_b"] = a.log(), b.log()
    if c["kind"] == "masked":
        st["mask_q"], st["mask_k"] = ((torch.rand((B, L), generator=gen, device="cuda") > 0.1).to(torch.uint8)
                                      for _ in range(2))
    if c["kind"] == "token":
        st["tok"] = [torch.randn((B, H, d), generator=gen, device="cuda") for _ in range(3)]
    return st


def run(state):
    s, c = state, state["case"]
    Q, K, V, G, ws = s["Q"], s["K"], s["V"], s["dO"], s["ws"]
    W, T, R, eps, kind = c["W"], c["T"], c["R"], c["eps"], c["kind"]
    db = kind == "dustbin"
    la, lb, lq, lk = (s.get(n) for n in ("log_a", "log_b", "len_q", "len_k"))
    if c["call"] == "step":
        O, UV, dQ, dK, dV = ska.sinkhorn_attn_step(Q, K, V, G, W, T, R, eps, db, 0.0, la, lb, lq, lk, workspace=ws,
                                                   **s["out"])
        return {"O": O, "UV": UV, "dQ": dQ, "dK": dK, "dV": dV}
    if kind == "token":
        O, UV = ska.sinkhorn_attn_fwd_dustbin_token(Q, K, V, *s["tok"], W, T, R, eps, workspace=ws)
        out = {"O": O, "UV": UV}
        if c["call"] == "fwd_bwd":
            res = ska.sinkhorn_attn_bwd_dustbin_token(Q, K, V, *s["tok"], O, G, UV, W, T, R, eps, workspace=ws)
            out.update(zip(("dQ", "dK", "dV", "dq_db", "dk_db", "dv_db"), res))
        return out
    if kind == "masked":
        O, UV = ska.sinkhorn_attn_fwd_masked(Q, K, V, s["mask_q"], s["mask_k"], W, T, R, eps, workspace=ws)
        out = {"O": O}   # (the potentials of inactive tokens are -inf, which has no relative error)
    else:
        O, UV = ska.sinkhorn_attn_fwd_varlen(Q, K, V, la, lb, lq, lk, W, T, R, eps, db, 0.0, workspace=ws)
        out = {"O": O, "UV": UV}
    if c["call"] == "fwd_bwd":
        res = ska.sinkhorn_attn_bwd_varlen(Q, K, V, la, lb, lq, lk, O, G, UV, W, T, R, eps, db, 0.0, workspace=ws)
        out.update(zip(("dQ", "dK", "dV"), res))
    return out


def work(case):
    """Every input read once and every output written once; on the matrix cores one score evaluation
    per Sinkhorn step (the state is O(L), so no step can keep the scores of the one before), the
    products of the output map, and in the backward one more score evaluation, dO V^T and the three
    products that give dQ, dK and dV; an exponential and two additions per edge and step."""
    c = case
    N, L, d, be = c["B"] * c["H"], c["L"], c["d"], 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "varlen":
        L = int(0.75 * L)   # lengths are uniform over the upper half of the range
    w = min(c["W"], L - 1)
    edges = float(N) * (L * (2 * w + 1) - w * (w + 1))
    bwd = c["call"] != "fwd"
    mats = 4 + (4 if bwd else 0) + (1 if c["call"] == "fwd_bwd" else 0)   # (two calls: O is read back)
    return {"bytes": float(N) * L * (mats * d * be + 8 * (c["R"] + 1)),
            "flops": edges * ((2 * d + 3) * (c["T"] + c["R"]) + 2 * d + (10 * d if bwd else 0))}


def tolerance(case):
    """Measured against the fp64 oracle over 50 drawn cases: at most 4.1e-3 on any output in bf16 (rounding of
    the scaled operand, of the plan as a matrix operand and of the stored results), 1.1e-6 in fp32 at L = 6000.
    The gradients of the learned tokens are sums over all L spokes that nearly cancel: 2e-2 in bf16."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 2e-2 if case["kind"] == "token" else 1e-2}
