"""The work a user of this engine has it do, as cases that can be timed.

Every case goes through the package's entry points (`paper_2508_19525_amd`, the binding of
include/blb.h) the way bench.py, the tests and a server program use them: contexts are made once
per parameter set, keys, plans, executors and encrypted inputs are in hand before the call, and a
pass is one operator (or one short chain of them) on ciphertexts resident in HBM.  Knobs stay at
their defaults except the plan format, which a caller chooses.

    listed()             the named cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs, keys, plans and executors of a case, from the seed alone
    run(state)           one pass; returns every output word
    work(case)           bytes and operations one pass cannot do without
    exact(case, seed)    None: outputs are residues (whole numbers), not rounded values
"""
import ctypes
import math

import numpy as np
import torch

import paper_2508_19525_amd as B
from paper_2508_19525_amd import workloads as wl

# (log2 N, ciphertext primes, special primes, digits, log2 scale): the parameter sets of the
# workloads -- the small operator, the BERT-base linear operators, the served operators, the
# attention product and the attention output
SMALL = (12, 2, 1, 2, 30)
BASE = (13, 3, 1, 3, 40)
SERVED = (14, 4, 2, 2, 40)
ATT_OUT = (14, 5, 2, 3, 40)


def _params(p):
    return {"log_n": p[0], "n_q": p[1], "n_special": p[2], "dnum": p[3], "log_scale": p[4]}


def listed():
    return [
        # one rotation of one ciphertext, at the smallest ring: the unit every other operator is
        # built from, called alone where a program applies its own schedule (latency)
        dict(name="rotate_one", kind="rotate", **_params(SMALL), count=1),
        # the smallest fused linear operator (32 x 32 times 32 x 32), called eagerly, with the mask
        dict(name="linear_32", kind="linear", **_params(SMALL), L=32, d_in=32, d_out=32, cplx=False, packed=False, graph=False),
        # the BERT-base 128 x 768 x 768 projection as one recorded executor: the serving step of a
        # program that runs one operator over and over
        dict(name="linear_bert_base", kind="linear", **_params(BASE), L=128, d_in=768, d_out=768, cplx=False, packed=False, graph=True),
        # ragged sizes, complex-slot outputs and 50-bit plan words, called eagerly
        dict(name="linear_ragged", kind="linear", **_params(BASE), L=100, d_in=700, d_out=1130, cplx=True, packed=True, graph=False),
        # a BERT-large feed-forward projection (1024 -> 4096) at the served ring: the largest
        # plan, streamed once per pass
        dict(name="linear_bert_large", kind="linear", **_params(SERVED), L=64, d_in=1024, d_out=4096, cplx=False, packed=True, graph=False),
        # new weights, or a new sequence length: plan generation, one product with it, plan dropped
        dict(name="plan_and_linear", kind="plan", **_params(BASE), L=128, d_in=768, d_out=768, cplx=False, packed=False),
        # 12-head Q K^T of 128 tokens as a recorded executor
        dict(name="qk_bert_base", kind="qk", **_params(SERVED), heads=12, L=128, d_head=64, graph=True),
        # 12-head Softmax V and Concat(Att) W_O, called eagerly
        dict(name="attention_out", kind="attention_out", **_params(ATT_OUT), heads=12, L=128, d_v=64, d_out=768),
        # row sums over the columns of each ciphertext and the product of each row with a per-row
        # scalar, for the 24 ciphertexts of a 128 x 768 activation: the steps around a normalisation
        dict(name="row_statistics", kind="rows", **_params(BASE), L=128, n_ct=24),
        # independent clients in one call: own keys, uneven lengths, shared weights
        dict(name="batch_uneven", kind="batch", **_params(BASE), lengths="200,33,128,90,256,64,16,150,250,120,40,230", hidden=768),
        # the transform by itself, both directions, 0.5 GiB each
        dict(name="ntt_large", kind="ntt", log_n=14, n_q=4, n_special=2, dnum=2, log_scale=40, n_polys=1024, n_limbs=4),
        # requests of mixed operators and lengths into the serving runtime, whose plan cache does
        # not hold every plan: plans are generated while batches run
        dict(name="serve_mixed", kind="serve", **_params(SERVED), requests=12, L_max=128, cache_gb=4.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _plan_words(c, L=None, d_in=None, d_out=None):
    """plaintext words of a ct-pt plan: [(b, j)][(a, i)][limb][N]"""
    g = _cp_geom(c["log_n"], L or c["L"], d_in or c["d_in"], d_out or c["d_out"], c.get("cplx", False))
    return g["n_out"] * g["G"] * g["n_in"] * g["B"] * c["n_q"] * (1 << c["log_n"])


def draw(rng):
    kind = rng.choice(["rotate", "linear", "linear", "linear", "plan", "qk", "rows", "batch", "ntt", "serve"])
    if kind == "rotate":
        p = rng.choice([SMALL, BASE, SERVED, ATT_OUT])
        return dict(kind="rotate", **_params(p), count=rng.randint(1, 12))
    if kind in ("linear", "plan"):
        p = rng.choice([SMALL, BASE, BASE, SERVED])
        c = dict(kind=kind, **_params(p), L=_log_int(rng, 16, 512), d_in=_log_int(rng, 24, 4096), d_out=_log_int(rng, 24, 4096),
                 cplx=rng.random() < 0.4, packed=rng.random() < 0.4)
        while _plan_words(c) > 6e8:
            if c["d_in"] >= c["d_out"]:
                c["d_in"] = max(24, c["d_in"] * 2 // 3)
            else:
                c["d_out"] = max(24, c["d_out"] * 2 // 3)
        if kind == "linear":
            c["graph"] = rng.random() < 0.5
        return c
    if kind == "qk":
        return dict(kind="qk", **_params(SERVED), heads=rng.choice([2, 3, 4, 6, 8, 12]), L=rng.randint(33, 128),
                    d_head=rng.choice([32, 64]), graph=rng.random() < 0.5)
    if kind == "rows":
        return dict(kind="rows", **_params(BASE), L=_log_int(rng, 16, 512), n_ct=rng.randint(1, 32))
    if kind == "batch":
        k = rng.randint(3, 10)
        return dict(kind="batch", **_params(BASE), lengths=",".join(str(rng.randint(16, 256)) for _ in range(k)),
                    hidden=rng.choice([256, 500, 768]))
    if kind == "ntt":
        log_n, n_limbs = rng.choice([12, 13, 14]), rng.randint(1, 4)
        words = _log_int(rng, 1 << 20, 1 << 26)
        return dict(kind="ntt", log_n=log_n, n_q=4, n_special=2, dnum=2, log_scale=40, n_polys=max(1, words // ((1 << log_n) * n_limbs)),
                    n_limbs=n_limbs)
    return dict(kind="serve", **_params(SERVED), requests=rng.randint(3, 12), L_max=rng.randint(32, 128), cache_gb=4.0)


# ---------------------------------------------------------------------------------------
# what a program has in hand before the call
# ---------------------------------------------------------------------------------------
_CONTEXTS = {}


def _new_context(c):
    return B.blb_ctx_create(c["log_n"], c["n_q"], c["n_special"], c["dnum"], 0, torch.cuda.current_stream().cuda_stream)


def _context(c):
    """one context per parameter set, kept for the life of the program"""
    key = tuple(c[k] for k in ("log_n", "n_q", "n_special", "dnum"))
    if key not in _CONTEXTS:
        _CONTEXTS[key] = _new_context(c)
    return _CONTEXTS[key]


class State:
    """Handles and buffers of one prepared case; the library's handles are given back with it."""

    def __init__(self, case):
        self.case, self.undo = case, []

    def own(self, destroy, handle):
        self.undo.append((destroy, handle))
        return handle

    def __del__(self):
        torch.cuda.synchronize()
        for destroy, handle in reversed(self.undo):
            destroy(handle)


def _cp_geom(log_n, L, d_in, d_out, cplx=False):
    """Geometry of a ct-pt product as blb_plan_info reports it (for work() and the rotation steps)."""
    slots = 1 << (log_n - 1)
    lp = wl.lp_of(L)
    c = slots // lp
    ce = min(c, 1 << max(0, math.ceil(math.log2(d_in))))
    b = 1 << ((int(math.log2(ce)) + 1) // 2)
    n_out = -(-d_out // c)
    return {"Lp": lp, "n_in": -(-d_in // c), "n_out": (n_out + 1) // 2 if cplx else n_out, "B": b, "G": ce // b}


def _cp_steps(g):
    return [i * g["Lp"] for i in range(1, g["B"])] + [j * g["B"] * g["Lp"] for j in range(1, g["G"])]


def _cts(n, level, count):
    """`count` ciphertexts over one buffer, and the buffer"""
    words = 2 * (level + 1) * n
    t = torch.zeros(count * words, dtype=torch.int64, device="cuda")
    return [B.blb_ct(t.data_ptr() + 8 * words * k, level, 1, 0.0) for k in range(count)], t


def _encrypt(s, ctx, keys, vectors, level, seed):
    """encrypted slot vectors, at the case's scale"""
    n, scale = 1 << s.case["log_n"], 2.0 ** s.case["log_scale"]
    cts, buf = _cts(n, level, len(vectors))
    pt = torch.empty((level + 1) * n, dtype=torch.int64, device="cuda")
    for k, v in enumerate(vectors):
        B.blb_encode(ctx, v, scale, level, pt)
        B.blb_encrypt(ctx, keys, pt, level, scale, seed, k, cts[k])
    torch.cuda.synchronize()
    s.undo.append((lambda t: None, buf))
    return cts


def _spatial(X, log_n):
    slots = 1 << (log_n - 1)
    c = slots // wl.lp_of(X.shape[0])
    return [wl.pack_spatial(X, slots, a) for a in range(-(-X.shape[1] // c))]


def _plan(ctx, case, W, L, level):
    B.blb_ctx_set_knob(ctx, B.BLB_KNOB_PLAN_FORMAT, 1 if case["packed"] else 0)
    try:
        return (B.blb_plan_matmul_cp_cplx if case["cplx"] else B.blb_plan_matmul_cp)(ctx, W, L, level)
    finally:
        B.blb_ctx_set_knob(ctx, B.BLB_KNOB_PLAN_FORMAT, 0)


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    s = State(case)
    kind, n, level = case["kind"], 1 << case["log_n"], case["n_q"] - 1
    s.level, s.n, s.seed = level, n, seed
    if kind == "serve":
        _prepare_serve(s, rng)
        return s
    ctx = s.ctx = _context(case)

    def keygen(steps, more=0):
        return s.own(B.blb_keys_destroy, B.blb_keygen(ctx, seed + more, sorted(set(steps))))

    if kind == "rotate":
        s.steps = [int(x) for x in rng.choice(np.arange(1, n // 2), case["count"], replace=False)]
        s.keys = keygen(s.steps)
        s.X = _encrypt(s, ctx, s.keys, [rng.normal(0, 1, n // 2)], level, seed)
        s.Y, s.y = _cts(n, level, case["count"])
    elif kind in ("linear", "plan"):
        L = case["L"]
        s.W = rng.normal(0, 0.02, (case["d_in"], case["d_out"]))
        g = _cp_geom(case["log_n"], L, case["d_in"], case["d_out"], case["cplx"])
        s.keys = keygen(_cp_steps(g))
        s.X = _encrypt(s, ctx, s.keys, _spatial(rng.normal(0, 1, (L, case["d_in"])), case["log_n"]), level, seed)
        s.Y, s.y = _cts(n, level - 1, g["n_out"])
        s.share = torch.zeros(g["n_out"] * level * n, dtype=torch.int64, device="cuda")
        if kind == "linear":
            s.plan = s.own(B.blb_plan_destroy, _plan(ctx, case, s.W, L, level))
            if case["graph"]:
                s.ex = s.own(B.blb_exec_destroy, B.blb_exec_create_cp(ctx, s.keys, s.plan, s.X, s.Y, level - 1, s.share))
    elif kind == "qk":
        heads, L, d = case["heads"], case["L"], case["d_head"]
        s.keys = keygen(B.blb_cc_rotations(ctx, heads, L, 1))
        s.plan = s.own(B.blb_plan_destroy, B.blb_plan_matmul_cc(ctx, heads, L, d, level, schedule=1))
        Q = [rng.normal(0, 1, (L, d)) for _ in range(heads)]
        Kt = [rng.normal(0, 1, (d, L)) for _ in range(heads)]
        s.A, s.Bp = _head_operands(s, Q, Kt, L, d)
        n_out = B.blb_plan_cc_info(s.plan)["n_out"]
        s.Y, s.y = _cts(n, level - 3, n_out)
        s.share = torch.zeros(n_out * (level - 2) * n, dtype=torch.int64, device="cuda")
        if case["graph"]:
            s.ex = s.own(B.blb_exec_destroy, B.blb_exec_create_cc(ctx, s.keys, s.plan, s.A, s.Bp, s.Y, level - 3, s.share))
    elif kind == "attention_out":
        heads, L, d = case["heads"], case["L"], case["d_v"]
        W = rng.normal(0, 0.02, (heads * d, case["d_out"]))
        s.plan2 = s.own(B.blb_plan_destroy, B.blb_plan_matmul_cp_diag(ctx, W, heads, d, L, level - 3))
        s.plan = s.own(B.blb_plan_destroy, B.blb_plan_matmul_cc_sv(ctx, heads, L, d, level, schedule=1))
        g = B.blb_plan_info(s.plan2)
        s.keys = keygen(list(B.blb_cc_rotations(ctx, heads, L, 1)) + _cp_steps(g))
        z = np.exp(rng.normal(0, 1, (heads, L, L)))
        z /= z.sum(axis=2, keepdims=True)
        s.A, s.Bp = _head_operands(s, list(z), [rng.normal(0, 1, (L, d)) for _ in range(heads)], L, L)
        s.M, s.m = _cts(n, level - 3, B.blb_plan_cc_info(s.plan)["n_out"])
        s.Y, s.y = _cts(n, level - 4, g["n_out"])
        s.share = torch.zeros(g["n_out"] * (level - 3) * n, dtype=torch.int64, device="cuda")
    elif kind == "rows":
        s.lp = wl.lp_of(case["L"])
        s.nb = (n // 2) // s.lp
        steps, st = [], s.lp
        while st < n // 2:
            steps += [st, -st]
            st *= 2
        s.keys = keygen(steps)
        c = s.nb
        X = rng.normal(0, 1, (case["L"], c * case["n_ct"]))
        s.X = _encrypt(s, ctx, s.keys, _spatial(X, case["log_n"]), level, seed)
        first = np.zeros((case["n_ct"], n // 2))
        first[:, : case["L"]] = rng.uniform(0.5, 1.5, (case["n_ct"], case["L"]))
        s.S = _encrypt(s, ctx, s.keys, list(first), level, seed + 1)
        s.Y, s.y = _cts(n, level - 1, case["n_ct"])
        s.Z, s.z = _cts(n, level, case["n_ct"])
    elif kind == "batch":
        _prepare_batch(s, rng, keygen)
    elif kind == "ntt":
        q = [int(x) for x in B.blb_ctx_moduli(ctx, case["n_q"] + case["n_special"])][: case["n_limbs"]]
        gen = torch.Generator(device="cuda").manual_seed(seed)

        def residues():
            return torch.stack([torch.randint(0, m, (case["n_polys"], n), generator=gen, dtype=torch.int64, device="cuda") for m in q], dim=1)

        s.fwd, s.inv = residues(), residues()
    else:
        raise ValueError(kind)
    return s


def _head_operands(s, left, right, L, d):
    """both operands of a multi-head product, packed and encrypted per head group"""
    A, Bp, h0 = [], [], 0
    slots = s.n // 2
    for grp in B.blb_plan_cc_info(s.plan)["groups"]:
        H = grp["H"]
        for out, mats, op in ((A, left, "A"), (Bp, right, "Bp")):
            out += [wl.pack_mhp(mats[h0:h0 + H], H, L, d, a, op, slots) for a in range(grp["n_ct"])]
        h0 += H
    return _encrypt(s, s.ctx, s.keys, A, s.level, s.seed), _encrypt(s, s.ctx, s.keys, Bp, s.level, s.seed + 1)


def _prepare_batch(s, rng, keygen):
    case, ctx, n, level = s.case, s.ctx, s.n, s.level
    D, lengths = case["hidden"], [int(x) for x in case["lengths"].split(",")]
    W = rng.normal(0, 0.02, (D, D))
    plans = {}
    s.inst = (B.blb_cp_instance * len(lengths))()
    s.hold, s.y = [], []
    for i, L in enumerate(lengths):
        lp = wl.lp_of(L)
        if lp not in plans:
            plans[lp] = s.own(B.blb_plan_destroy, B.blb_plan_matmul_cp(ctx, W, lp, level))
        g = B.blb_plan_info(plans[lp])
        keys = keygen(_cp_steps(g), 100 + i)
        X = _encrypt(s, ctx, keys, _spatial(rng.normal(0, 1, (L, D)), case["log_n"]), level, s.seed + i)
        Y, y = _cts(n, level - 1, g["n_out"])
        xa, ya = (B.blb_ct * len(X))(*X), (B.blb_ct * len(Y))(*Y)
        s.hold += [xa, ya]
        s.y.append(y)
        s.inst[i] = B.blb_cp_instance(keys, plans[lp], ctypes.cast(xa, ctypes.c_void_p), len(X), ctypes.cast(ya, ctypes.c_void_p), len(Y))


SERVE_SHAPES = ((768, 768), (768, 1500), (1024, 1024))  # the operators the server holds


def _serve_requests(case):
    """[(weight, L, client)], spread over the operators, the lengths and two clients"""
    k = case["requests"]
    return [(i % 3, max(16, round(16 * (case["L_max"] / 16) ** (((i * 7) % k) / max(1, k - 1)))), (i // 2) % 2) for i in range(k)]


def _prepare_serve(s, rng):
    case, n, level = s.case, s.n, s.level
    ctx = s.ctx = s.own(B.blb_ctx_destroy, _new_context(case))  # a server's worker owns its context
    reqs = _serve_requests(case)
    steps = set()
    for w, L, _ in reqs:
        steps |= set(_cp_steps(_cp_geom(case["log_n"], L, *SERVE_SHAPES[w])))
    keys = [s.own(B.blb_keys_destroy, B.blb_keygen(ctx, s.seed + k, sorted(steps))) for k in range(2)]
    s.reqs, s.y = [], []
    for i, (w, L, client) in enumerate(reqs):
        d_in, d_out = SERVE_SHAPES[w]
        X = _encrypt(s, ctx, keys[client], _spatial(rng.normal(0, 1, (L, d_in)), case["log_n"]), level, s.seed + i)
        Y, y = _cts(n, level - 1, _cp_geom(case["log_n"], L, d_in, d_out, True)["n_out"])
        share = torch.zeros(len(Y) * level * n, dtype=torch.int64, device="cuda")
        s.y += [y, share]
        s.reqs.append((keys[client], w, L, (B.blb_ct * len(X))(*X), (B.blb_ct * len(Y))(*Y), share))
    torch.cuda.synchronize()
    B.blb_ctx_set_knob(ctx, B.BLB_KNOB_PLAN_FORMAT, 1)  # the plans of a server, whose cache is what it runs short of
    s.server = s.own(B.blb_server_destroy, B.blb_server_create(ctx, int(case["cache_gb"] * 1e9), max_batch=8, n_streams=2))
    for w, (d_in, d_out) in enumerate(SERVE_SHAPES):
        B.blb_server_add_weights(s.server, w, rng.normal(0, 0.02, (d_in, d_out)), level, cplx=True)


# ---------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------
def run(s):
    kind, ctx = s.case["kind"], s.ctx
    if kind == "rotate":
        for k, steps in enumerate(s.steps):
            B.blb_rotate(ctx, s.keys, s.X[0], steps, s.Y[k])
        return s.y
    if kind == "linear":
        if s.case["graph"]:
            B.blb_exec_run(s.ex, s.seed)
        else:
            B.blb_matmul_cp(ctx, s.keys, s.plan, s.X, s.Y)
            B.blb_mask_to_share(ctx, s.Y, s.seed, s.level - 1, s.share)
        return s.y, s.share
    if kind == "plan":
        plan = _plan(ctx, s.case, s.W, s.case["L"], s.level)
        B.blb_matmul_cp(ctx, s.keys, plan, s.X, s.Y)
        B.blb_mask_to_share(ctx, s.Y, s.seed, s.level - 1, s.share)
        torch.cuda.synchronize()  # a plan is given back only after the work that reads it
        B.blb_plan_destroy(plan)
        return s.y, s.share
    if kind == "qk":
        if s.case["graph"]:
            B.blb_exec_run(s.ex, s.seed)
        else:
            B.blb_matmul_cc(ctx, s.keys, s.plan, s.A, s.Bp, s.Y)
            B.blb_mask_to_share(ctx, s.Y, s.seed, s.level - 3, s.share)
        return s.y, s.share
    if kind == "attention_out":
        B.blb_matmul_cc(ctx, s.keys, s.plan, s.A, s.Bp, s.M)
        B.blb_matmul_cp(ctx, s.keys, s.plan2, s.M, s.Y)
        B.blb_mask_to_share(ctx, s.Y, s.seed, s.level - 4, s.share)
        return s.m, s.y, s.share
    if kind == "rows":
        B.blb_rotate_sum(ctx, s.keys, s.X, s.Y, s.lp, s.nb, 0)
        B.blb_scalar_op(ctx, s.keys, s.X, s.S, s.lp, s.nb, 1, False, s.Z)
        return s.y, s.z
    if kind == "batch":
        B.blb_batch_matmul_cp(ctx, s.inst)
        return s.y
    if kind == "ntt":
        B.blb_ntt(ctx, s.fwd, s.case["n_polys"], s.case["n_limbs"])
        B.blb_ntt(ctx, s.inv, s.case["n_polys"], s.case["n_limbs"], True)
        return s.fwd, s.inv
    for i, (keys, w, L, X, Y, share) in enumerate(s.reqs):
        B.blb_server_submit(s.server, keys, w, L, X, Y, s.seed + i, s.level - 1, share)
    B.blb_server_drain(s.server, 60)
    return s.y


# ---------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------
WORD = 8  # bytes of a ciphertext or key word
PT_WORD = 6.25  # bytes of a plan word: residues of 50-bit primes


def _ntt_flops(log_n, polys):
    """an addition, a subtraction and a modular product (taken as 2 operations) per butterfly"""
    return polys * (1 << (log_n - 1)) * log_n * 4


def _keyswitch(c, nl, count, sources=None):
    """(bytes, flops) of `count` key switches at nl limbs of `sources` hoisted sources: the switching
    key and the output once; the transforms, the key products"""
    n, k = 1 << c["log_n"], c["n_special"]
    alpha = -(-c["n_q"] // c["dnum"])
    nd, ext = -(-nl // alpha), nl + k
    src = count if sources is None else sources
    polys = src * (nl + nd * ext - nl) + count * 2 * (k + nl)
    return count * 2 * nl * n * WORD, _ntt_flops(c["log_n"], polys) + count * 2 * nd * ext * n * 4


def _key_bytes(c, keys):
    return keys * c["dnum"] * 2 * (c["n_q"] + c["n_special"]) * (1 << c["log_n"]) * WORD


def _linear_work(c, L, d_in, d_out, cplx, nl):
    n = 1 << c["log_n"]
    g = _cp_geom(c["log_n"], L, d_in, d_out, cplx)
    words = g["n_out"] * g["G"] * g["n_in"] * g["B"] * nl * n
    _, f1 = _keyswitch(c, nl, g["n_in"] * (g["B"] - 1), g["n_in"])
    _, f2 = _keyswitch(c, nl, g["n_out"] * (g["G"] - 1))
    cts = (g["n_in"] * 2 * nl + g["n_out"] * 2 * (nl - 1)) * n * WORD
    return {"bytes": words * PT_WORD + cts + _key_bytes(c, g["B"] + g["G"] - 2), "flops": words * 2 * 4 + f1 + f2, "words": words}


def _cc_work(c, sv):
    """a BSGS ct-ct product: operands, the tensors, the rotations of its schedule"""
    n, nl, lp = 1 << c["log_n"], c["n_q"], wl.lp_of(c["L"])
    nbytes, flops = 0.0, 0.0
    inner = 1 << ((int(math.log2(lp)) + 1) // 2)
    giant = lp // inner
    for H in wl.head_groups(c["heads"]):
        cols = (n // 2) // (lp * H)
        if cols < 1:
            cols = 1
        d = lp if sv else c["d_head"]
        n_ct, n_diag = -(-d // cols), -(-lp // cols)
        _, f = _keyswitch(c, nl, n_ct * 2 * (inner + giant - 2), 2 * n_ct)
        _, f2 = _keyswitch(c, nl - 2, lp + lp - n_diag)
        flops += f + f2 + lp * n_ct * 4 * (nl - 1) * n * 4
        n_out = n_diag if not sv else max(1, c["d_v"] // cols)
        nbytes += (2 * n_ct * 2 * nl + 2 * n_out * (nl - 3)) * n * WORD
    return {"bytes": nbytes + _key_bytes(c, 2 * (inner + giant)), "flops": flops}


def work(case):
    c, n = case, 1 << case["log_n"]
    kind, nl = c["kind"], c["n_q"]
    if kind == "rotate":
        b, f = _keyswitch(c, nl, c["count"])
        return {"bytes": 2 * nl * n * WORD + b + _key_bytes(c, c["count"]), "flops": f}
    if kind in ("linear", "plan"):
        w = _linear_work(c, c["L"], c["d_in"], c["d_out"], c["cplx"], nl)
        if kind == "plan":  # the plan is written as well as read
            w["bytes"] += w["words"] * PT_WORD
            w["flops"] += _ntt_flops(c["log_n"], w["words"] // n)
        return {"bytes": w["bytes"], "flops": w["flops"]}
    if kind == "qk":
        return _cc_work(c, False)
    if kind == "attention_out":
        w = _cc_work(c, True)
        v = _linear_work(c, c["L"], c["heads"] * c["d_v"], c["d_out"], False, nl - 3)
        return {"bytes": w["bytes"] + v["bytes"], "flops": w["flops"] + v["flops"]}
    if kind == "rows":
        rot = int(math.log2((n // 2) // wl.lp_of(c["L"])))
        b, f = _keyswitch(c, nl, c["n_ct"] * (2 * rot + 1))
        return {"bytes": c["n_ct"] * (4 * nl + 2 * (nl - 1) + 2 * nl) * n * WORD + _key_bytes(c, 2 * rot + 1), "flops": f}
    if kind == "batch":
        out = {"bytes": 0.0, "flops": 0.0}
        seen = set()
        for L in (int(x) for x in c["lengths"].split(",")):
            w = _linear_work(c, L, c["hidden"], c["hidden"], False, nl)
            again = wl.lp_of(L) in seen  # instances of one length share their plan
            seen.add(wl.lp_of(L))
            out["bytes"] += w["bytes"] - (w["words"] * PT_WORD if again else 0)
            out["flops"] += w["flops"]
        return out
    if kind == "ntt":
        polys = c["n_polys"] * c["n_limbs"]
        return {"bytes": 2 * 2 * polys * n * WORD, "flops": 2 * _ntt_flops(c["log_n"], polys)}
    out = {"bytes": 0.0, "flops": 0.0}
    for w, L, _ in _serve_requests(c):
        v = _linear_work(c, L, *SERVE_SHAPES[w], True, nl)
        out["bytes"] += v["bytes"]
        out["flops"] += v["flops"]
    return out


def exact(case, seed):
    """Every output is a residue word, equal or not: there is nothing to round."""
    return None
