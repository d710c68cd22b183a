"""GPU parity: the HIP library (through its C ABI) against the CPU oracle, word for word.

Ciphertexts are compared in canonical coefficient form (blb_export) against the oracle's
coefficient-form words.  Encryption randomness comes from the same seeds on both sides
(each side implements Philox4x32-10 itself).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def blb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_19525_amd as B
    B.lib()
    return B


class Ctx:
    """GPU context + oracle context with the same parameters"""

    def __init__(self, B, orc, log_n, n_q, n_sp, dnum):
        self.B, self.orc = B, orc
        self.n = 1 << log_n
        self.n_q, self.n_sp = n_q, n_sp
        self.h = B.blb_ctx_create(log_n, n_q, n_sp, dnum, 0, torch.cuda.current_stream().cuda_stream)
        self.o = orc.Context(log_n, n_q, n_sp, dnum)
        self.keep = []

    def close(self):
        torch.cuda.synchronize()
        self.B.blb_ctx_destroy(self.h)

    def ct(self, level, degree=1):
        c, t = self.B.new_ct(self.n, level, degree)
        self.keep.append(t)
        return c

    def pt_dev(self, level):
        t = torch.empty((level + 1) * self.n, dtype=torch.int64, device="cuda")
        self.keep.append(t)
        return t

    def upload_words(self, words):
        a = np.ascontiguousarray(words, dtype=np.uint64)
        t = torch.from_numpy(a.view(np.int64).reshape(-1).copy()).cuda()
        self.keep.append(t)
        return t

    def import_ct(self, words, level, degree=1):
        c = self.ct(level, degree)
        self.B.blb_import(self.h, words, c)
        return c

    def export(self, c):
        torch.cuda.synchronize()
        return self.B.blb_export(self.h, c, self.n)


@pytest.fixture(scope="module")
def c1(blb, orc):
    x = Ctx(blb, orc, 12, 2, 1, 2)
    yield x
    x.close()


@pytest.fixture(scope="module")
def c2s(blb, orc):
    x = Ctx(blb, orc, 13, 3, 1, 3)
    yield x
    x.close()


@pytest.fixture(scope="module")
def c3s(blb, orc):
    x = Ctx(blb, orc, 14, 4, 2, 2)
    yield x
    x.close()


def _ctxs(request, names):
    return [request.getfixturevalue(n) for n in names]


def test_moduli_match_oracle(c1, c2s, c3s):
    for c in (c1, c2s, c3s):
        m = c.B.blb_ctx_moduli(c.h, len(c.o.moduli))
        assert np.array_equal(m, c.o.moduli)


@pytest.mark.parametrize("name", ["c1", "c2s", "c3s"])
def test_encode_matches_oracle(request, name):
    c = request.getfixturevalue(name)
    rng = np.random.default_rng(1)
    top = c.n_q - 1
    for scale, dist in [(2.0 ** 40, "normal"), (2.0 ** 30, "uniform"), (float(c.o.q[top]), "weights")]:
        if dist == "normal":
            v = rng.normal(0, 1, c.n // 2)
        elif dist == "uniform":
            v = rng.uniform(-1, 1, c.n // 2 - 5)  # ragged: trailing slots zero
        else:
            v = rng.normal(0, 0.02, c.n // 2)
        pt = c.pt_dev(top)
        c.B.blb_encode(c.h, v, scale, top, pt)
        torch.cuda.synchronize()
        got = pt.cpu().numpy().view(np.uint64).reshape(top + 1, c.n)
        want = c.o.encode_rns(v, scale, top)
        mism = int((got != want).sum())
        assert mism == 0, f"{mism} encode mismatches at scale {scale}"


@pytest.mark.parametrize("name", ["c1", "c2s", "c3s"])
def test_encrypt_decrypt_match_oracle(request, name):
    c = request.getfixturevalue(name)
    keys_o = c.orc.Keys(c.o, 11)
    keys_g = c.B.blb_keygen(c.h, 11, [])
    rng = np.random.default_rng(2)
    for level in (c.n_q - 1, 0):
        want_pt = c.o.encode_rns(rng.normal(0, 1, c.n // 2), 2.0 ** 30, level)
        ct = c.ct(level)
        c.B.blb_encrypt(c.h, keys_g, c.upload_words(want_pt), level, 2.0 ** 30, 77, 5, ct)
        got = c.export(ct)
        want = keys_o.encrypt(want_pt, level, 77, 5)
        assert np.array_equal(got, want)
        dec = c.pt_dev(level)
        c.B.blb_decrypt(c.h, keys_g, ct, dec)
        torch.cuda.synchronize()
        assert np.array_equal(dec.cpu().numpy().view(np.uint64).reshape(level + 1, c.n), keys_o.decrypt(want, level))
    c.B.blb_keys_destroy(keys_g)


@pytest.mark.parametrize("name,steps", [("c1", [1, 5, -3]), ("c2s", [128, 1024, -1]), ("c3s", [128, 3, -128])])
def test_rotate_matches_oracle(request, name, steps):
    c = request.getfixturevalue(name)
    keys_o = c.orc.Keys(c.o, 21, [c.o.galois_elt(s) for s in steps])
    keys_g = c.B.blb_keygen(c.h, 21, steps)
    rng = np.random.default_rng(3)
    for level in sorted({c.n_q - 1, 1, 0}):
        if level >= c.n_q:
            continue
        m = rng.normal(0, 1, c.n // 2)
        want_ct = keys_o.encrypt(c.o.encode_rns(m, 2.0 ** 30, level), level, 9, 0)
        ct = c.import_ct(want_ct, level)
        for s in steps:
            out = c.ct(level)
            c.B.blb_rotate(c.h, keys_g, ct, s, out)
            got = c.export(out)
            want = keys_o.rotate(want_ct, level, s)
            assert np.array_equal(got, want), f"rotation {s} at level {level}"
    c.B.blb_keys_destroy(keys_g)


@pytest.mark.parametrize("name", ["c1", "c2s", "c3s"])
@pytest.mark.parametrize("off_in,off_out", [(1, 0), (0, 1), (1, 1)])
def test_rotate_at_odd_words(request, name, off_in, off_out):
    """Ciphertexts need 8-byte alignment only: a rotation whose input and / or output starts at an odd word
    gives the oracle's words and writes nothing around them."""
    c = request.getfixturevalue(name)
    keys_o = c.orc.Keys(c.o, 23, [c.o.galois_elt(5)])
    keys_g = c.B.blb_keygen(c.h, 23, [5])
    level = c.n_q - 1
    rng = np.random.default_rng(23)
    words = np.stack([np.stack([rng.integers(0, int(q), c.n, dtype=np.uint64) for q in c.o.q[: level + 1]]) for _ in range(2)])
    bufs, cts = [], []
    for off in (off_in, off_out):
        t = torch.full((words.size + 2,), 77, dtype=torch.int64, device="cuda")
        ct = c.ct(level)
        ct.data = t.data_ptr() + 8 * off
        bufs.append(t)
        cts.append(ct)
    c.B.blb_import(c.h, words, cts[0])
    c.B.blb_rotate(c.h, keys_g, cts[0], 5, cts[1])
    assert np.array_equal(c.export(cts[1]), keys_o.rotate(words, level, 5))
    out = bufs[1].cpu().numpy()
    assert (out[:off_out] == 77).all() and (out[off_out + words.size :] == 77).all()
    c.B.blb_keys_destroy(keys_g)


@pytest.mark.parametrize("name", ["c1", "c2s", "c3s"])
def test_rescale_matches_oracle(request, name):
    c = request.getfixturevalue(name)
    rng = np.random.default_rng(4)
    for level in range(c.n_q - 1, 0, -1):
        words = np.stack([np.stack([rng.integers(0, int(q), c.n, dtype=np.uint64) for q in c.o.q[: level + 1]]) for _ in range(2)])
        ct = c.import_ct(words, level)
        out = c.ct(level - 1)
        c.B.blb_rescale(c.h, ct, out)
        assert out.level == level - 1
        assert np.array_equal(c.export(out), c.o.rescale(words, level))


def _cp_case(c, L, d_in, d_out, level, seed, x_std=None):
    B, orc = c.B, c.orc
    rng = np.random.default_rng(seed)
    X = rng.uniform(-1, 1, (L, d_in)) if x_std is None else rng.normal(0, x_std, (L, d_in))
    W = rng.normal(0, 0.02, (d_in, d_out))
    g = c.o.cp_geometry(L, d_in, d_out)
    gal = c.o.cp_galois(L, d_in, d_out)
    steps = [i * g["Lp"] for i in range(1, g["B"])] + [j * g["B"] * g["Lp"] for j in range(1, g["G"])]
    keys_o = orc.Keys(c.o, 31, gal)
    keys_g = B.blb_keygen(c.h, 31, steps)
    scale = 2.0 ** 30
    X_words = np.stack([keys_o.encrypt(c.o.encode_rns(c.o.pack_spatial(X, a), scale, level), level, 100, a) for a in range(g["n_in"])])
    Xc = []
    for a in range(g["n_in"]):
        ct = c.import_ct(X_words[a], level)
        ct.scale = scale
        Xc.append(ct)
    plan = B.blb_plan_matmul_cp(c.h, W, L, level)
    info = B.blb_plan_info(plan)
    assert info == g
    Yc = [c.ct(level - 1) for _ in range(g["n_out"])]
    B.blb_matmul_cp(c.h, keys_g, plan, Xc, Yc)
    return dict(X=X, W=W, g=g, keys_o=keys_o, keys_g=keys_g, X_words=X_words, Yc=Yc, plan=plan, scale=scale)


@pytest.mark.parametrize("shape", [(32, 32, 32), (20, 40, 24), (5, 96, 70)])
def test_matmul_cp_matches_oracle_c1(c1, shape):
    L, d_in, d_out = shape
    r = _cp_case(c1, L, d_in, d_out, 1, sum(shape))
    want = r["keys_o"].matmul_cp(r["X_words"], 1, r["W"], L)
    for b in range(r["g"]["n_out"]):
        assert np.array_equal(c1.export(r["Yc"][b]), want[b]), f"output {b}"
    c1.B.blb_plan_destroy(r["plan"])
    c1.B.blb_keys_destroy(r["keys_g"])


def test_matmul_cp_matches_oracle_n8192_ragged(c2s):
    """N = 8192, three primes, ragged L and widths spanning several output ciphertexts"""
    L, d_in, d_out = 100, 96, 80
    r = _cp_case(c2s, L, d_in, d_out, 2, 7, x_std=1.0)
    want = r["keys_o"].matmul_cp(r["X_words"], 2, r["W"], L)
    for b in range(r["g"]["n_out"]):
        assert np.array_equal(c2s.export(r["Yc"][b]), want[b]), f"output {b}"
    # decoded accuracy against FP64
    vecs = []
    for b in range(r["g"]["n_out"]):
        pt = c2s.pt_dev(1)
        c2s.B.blb_decrypt(c2s.h, r["keys_g"], r["Yc"][b], pt)
        vecs.append(c2s.B.blb_decode(c2s.h, pt, 1, r["scale"], c2s.n // 2))
    from paper_2508_19525_amd.workloads import unpack_spatial
    got = unpack_spatial(vecs, L, d_out, c2s.n // 2)
    assert np.abs(got - r["X"] @ r["W"]).max() < 2.0 ** -10
    c2s.B.blb_plan_destroy(r["plan"])
    c2s.B.blb_keys_destroy(r["keys_g"])


@pytest.mark.parametrize("name", ["c1", "c2s"])
def test_mask_to_share_matches_oracle(request, name):
    c = request.getfixturevalue(name)
    rng = np.random.default_rng(5)
    keys_o = c.orc.Keys(c.o, 41)
    level = c.n_q - 1
    words = [keys_o.encrypt(c.o.encode_rns(rng.normal(0, 1, c.n // 2), 2.0 ** 30, level), level, 3, t) for t in range(3)]
    for target in (level, 0):
        cts = [c.import_ct(w, level) for w in words]
        share = torch.zeros(3 * (target + 1) * c.n, dtype=torch.int64, device="cuda")
        c.B.blb_mask_to_share(c.h, cts, 1234, target, share)
        torch.cuda.synchronize()
        sh = share.cpu().numpy().view(np.uint64).reshape(3, target + 1, c.n)
        for t in range(3):
            masked, want_share = c.o.mask_to_share(words[t], level, target, 1234, t)
            assert cts[t].level == target
            assert np.array_equal(c.export(cts[t]), masked)
            assert np.array_equal(sh[t], want_share)


@pytest.mark.parametrize("name", ["c1", "c2s", "c3s"])
def test_add_share_matches_oracle(request, name):
    """The server's step of the MPC-to-CKKS conversion word for word (shares uniform per limb),
    and mask-to-share followed by it restores the ciphertexts exactly."""
    c = request.getfixturevalue(name)
    rng = np.random.default_rng(8)
    keys_o = c.orc.Keys(c.o, 44)
    level = c.n_q - 1
    words = [keys_o.encrypt(c.o.encode_rns(rng.normal(0, 1, c.n // 2), 2.0 ** 30, level), level, 9, t) for t in range(3)]
    sh = np.stack([np.stack([c.orc.sample_uniform(77, i, t, 6, int(c.o.q[i]), c.n) for i in range(level + 1)]) for t in range(3)])
    cts = [c.import_ct(w, level) for w in words]
    c.B.blb_add_share(c.h, cts, c.upload_words(sh))
    for t in range(3):
        assert np.array_equal(c.export(cts[t]), c.o.add_share(words[t], level, sh[t])), f"ct {t}"
    cts = [c.import_ct(w, level) for w in words]
    share = torch.zeros(3 * (level + 1) * c.n, dtype=torch.int64, device="cuda")
    c.B.blb_mask_to_share(c.h, cts, 4321, level, share)
    c.B.blb_add_share(c.h, cts, share)
    for t in range(3):
        assert np.array_equal(c.export(cts[t]), words[t]), f"round trip ct {t}"


@pytest.mark.parametrize("name,block,n_blocks", [("c1", 32, 16), ("c2s", 64, 32), ("c2s", 128, 32)])
def test_rotate_sum_matches_oracle(request, name, block, n_blocks):
    """Rotate-and-sum word for word against the oracle on three ciphertexts: summation with the
    first-block mask, without it, and broadcast (block x n_blocks below and equal to N/2)."""
    c = request.getfixturevalue(name)
    rng = np.random.default_rng(block + n_blocks)
    steps, st = [], block
    while st < block * n_blocks:
        steps += [st, -st]
        st *= 2
    keys_o = c.orc.Keys(c.o, 46, sorted({c.o.galois_elt(x) for x in steps}))
    keys_g = c.B.blb_keygen(c.h, 46, steps)
    level = c.n_q - 1
    words = [keys_o.encrypt(c.o.encode_rns(rng.uniform(-1, 1, c.n // 2), 2.0 ** 30, level), level, 12, t) for t in range(3)]
    for direction, mask in ((0, True), (0, False), (1, False)):
        cts = [c.import_ct(w, level) for w in words]
        for x in cts:
            x.scale = 2.0 ** 30
        lv = level - 1 if mask else level
        outs = [c.ct(lv) for _ in range(3)]
        c.B.blb_rotate_sum(c.h, keys_g, cts, outs, block, n_blocks, direction, mask)
        for t in range(3):
            assert outs[t].level == lv
            want = keys_o.rotate_sum(words[t], level, block, n_blocks, direction, mask)
            assert np.array_equal(c.export(outs[t]), want), f"direction {direction} mask {mask} ct {t}"
    c.B.blb_keys_destroy(keys_g)


@pytest.mark.parametrize("name", ["c1", "c2s"])
def test_rerandomize_matches_oracle(request, name):
    """Public-key re-randomisation with flooding (object id = position in the list), word for
    word, at two levels and two flooding widths; then mask-to-share on the result."""
    c = request.getfixturevalue(name)
    rng = np.random.default_rng(6)
    keys_o = c.orc.Keys(c.o, 43)
    keys_g = c.B.blb_keygen(c.h, 43, [])
    level = c.n_q - 1
    for lvl, bits in ((level, 40), (0, 32)):
        words = [keys_o.encrypt(c.o.encode_rns(rng.normal(0, 1, c.n // 2), 2.0 ** 30, lvl), lvl, 7, t) for t in range(3)]
        cts = [c.import_ct(w, lvl) for w in words]
        c.B.blb_rerandomize(c.h, keys_g, cts, 555, bits)
        for t in range(3):
            assert np.array_equal(c.export(cts[t]), keys_o.rerandomize(words[t], lvl, 555, t, bits)), f"level {lvl} ct {t}"
    with pytest.raises(c.B.BlbError):
        c.B.blb_rerandomize(c.h, keys_g, cts, 1, 49)
    c.B.blb_keys_destroy(keys_g)


# --------------------------------------------------------------------------------------
# matmul_cc
# --------------------------------------------------------------------------------------
def _unrotated_b(mats, H, L, d, a, slots):
    """B operand without the client-side row rotation: slot i + L'(h + H kappa) <- B_h{a c + kappa, i}"""
    lp = 1 << int(np.ceil(np.log2(L)))
    cc = slots // (lp * H)
    v = np.zeros(slots)
    for h in range(H):
        for kap in range(cc):
            k = a * cc + kap
            if k < d:
                v[lp * (h + H * kap): lp * (h + H * kap) + L] = mats[h][k, :]
    return v


def _cc_case(c, heads, L, d, seed, outputs=None, prerot=True, schedule=0):
    from paper_2508_19525_amd import workloads as wl
    B, orc = c.B, c.orc
    rng = np.random.default_rng(seed)
    Q = [rng.normal(0, 1, (L, d)) for _ in range(heads)]
    Kt = [rng.normal(0, 1, (L, d)).T.copy() for _ in range(heads)]
    level, scale = c.n_q - 1, 2.0 ** 40
    steps = B.blb_cc_rotations(c.h, heads, L, schedule, b_prerotated=prerot)
    gal = sorted({c.o.galois_elt(s) for s in steps})
    keys_o = orc.Keys(c.o, 51, gal)
    keys_g = B.blb_keygen(c.h, 51, steps)
    plan = B.blb_plan_matmul_cc(c.h, heads, L, d, level, b_prerotated=prerot, schedule=schedule)
    info = B.blb_plan_cc_info(plan)
    A_g, B_g, want, h0 = [], [], [], 0
    for gi, grp in enumerate(info["groups"]):
        H = grp["H"]
        assert H == wl.head_groups(heads)[gi]
        og = c.o.cc_geometry(H, L, d)
        assert (og["c"], og["n_ct"], og["n_out"]) == (grp["c"], grp["n_ct"], grp["n_out"])
        Aw = np.stack([keys_o.encrypt(c.o.encode_rns(c.o.pack_mhp(Q[h0:h0 + H], H, L, d, a, "A"), scale, level), level, 60 + gi, a)
                       for a in range(og["n_ct"])])
        bvec = [c.o.pack_mhp(Kt[h0:h0 + H], H, L, d, a, "Bp") if prerot else _unrotated_b(Kt[h0:h0 + H], H, L, d, a, c.n // 2)
                for a in range(og["n_ct"])]
        Bw = np.stack([keys_o.encrypt(c.o.encode_rns(v, scale, level), level, 70 + gi, a) for a, v in enumerate(bvec)])
        # the client-side packing of the library's helper module agrees with the oracle's
        assert np.array_equal(wl.pack_mhp(Q[h0:h0 + H], H, L, d, 0, "A", c.n // 2), c.o.pack_mhp(Q[h0:h0 + H], H, L, d, 0, "A"))
        assert np.array_equal(wl.pack_mhp(Kt[h0:h0 + H], H, L, d, 0, "Bp", c.n // 2), c.o.pack_mhp(Kt[h0:h0 + H], H, L, d, 0, "Bp"))
        for a in range(og["n_ct"]):
            x = c.import_ct(Aw[a], level)
            x.scale = scale
            A_g.append(x)
            y = c.import_ct(Bw[a], level)
            y.scale = scale
            B_g.append(y)
        outs = None if outputs is None else [o for o in outputs if o < og["n_out"]]
        want.append((keys_o.matmul_cc(Aw, Bw, level, H, L, d, outputs=outs, b_prerotated=prerot, schedule=schedule), outs, grp))
        h0 += H
    Cd = [c.ct(level - (3 if prerot else 4)) for _ in range(info["n_out"])]
    B.blb_matmul_cc(c.h, keys_g, plan, A_g, B_g, Cd)
    return dict(Q=Q, Kt=Kt, keys_o=keys_o, keys_g=keys_g, plan=plan, info=info, A=A_g, B=B_g, C=Cd, want=want, level=level)


@pytest.mark.parametrize("heads,L,d", [(512, 4, 12), (128, 8, 20), (256, 8, 5), (32, 16, 44)])
def test_matmul_cc_tensor_tiles(c3s, heads, L, d):
    """BSGS products whose step counts give tiles of 2 x 2 outputs (L' = 4: 2 x 2 steps; L' = 8: 4 x 2) and
    the smallest of 4 x 4 (L' = 16), with sums of 1 to 9 ciphertexts (no multiple of the reduction's four):
    word for word against the oracle."""
    r = _cc_case(c3s, heads, L, d, 3 * heads + L, None, True, 1)
    for O_want, outs, grp in r["want"]:
        for o in range(grp["n_out"]):
            got = c3s.export(r["C"][_out_index(r["info"], grp, o)])
            assert np.array_equal(got, O_want[o]), f"group H={grp['H']} output {o}"
    c3s.B.blb_plan_destroy(r["plan"])
    c3s.B.blb_keys_destroy(r["keys_g"])


@pytest.fixture(scope="module")
def c5p(blb, orc):
    """five ciphertext primes at N = 16384 (two special, digits of two primes): room for step 1
    on the server"""
    x = Ctx(blb, orc, 14, 5, 2, 3)
    yield x
    x.close()


@pytest.mark.parametrize("heads,L,d,outputs,prerot,schedule", [
    (8, 32, 32, None, True, 0), (12, 64, 32, [0, 1], True, 0), (8, 32, 32, None, False, 0), (12, 40, 32, [0, 3], False, 0),
    (8, 32, 32, None, True, 1), (12, 64, 32, None, True, 1), (12, 100, 24, [1, 2], True, 1), (8, 32, 32, None, False, 1),
    (12, 40, 32, [0, 3], False, 1)])
def test_matmul_cc_matches_oracle(request, heads, L, d, outputs, prerot, schedule):
    """Multi-head ct-ct matmul word for word against the oracle, including the 8 + 4 head-group
    split; decoded outputs equal Q_h K_h^T.  prerot: B pre-rotated by the client (steps 2-3,
    four primes); otherwise step 1 runs on the server first (five primes).  schedule 1 is the
    BSGS schedule (baby / giant inner rotations, giant rotations postponed into step 3; step 1
    split into baby and giant rotations), with a ragged L and d among its cases."""
    from paper_2508_19525_amd import workloads as wl
    c3s = request.getfixturevalue("c3s" if prerot else "c5p")
    r = _cc_case(c3s, heads, L, d, heads + L, outputs, prerot, schedule)
    h0 = 0
    for O_want, outs, grp in r["want"]:
        sel = range(grp["n_out"]) if outs is None else outs
        for o in sel:
            got = c3s.export(r["C"][_out_index(r["info"], grp, o)])
            assert np.array_equal(got, O_want[o]), f"group H={grp['H']} output {o}"
        if outs is None:
            vecs = []
            for o in range(grp["n_out"]):
                ct = r["C"][_out_index(r["info"], grp, o)]
                pt = c3s.pt_dev(0)
                c3s.B.blb_decrypt(c3s.h, r["keys_g"], ct, pt)
                vecs.append(c3s.B.blb_decode(c3s.h, pt, 0, ct.scale, c3s.n // 2))
            Cs = wl.unpack_diag(vecs, grp["H"], L, c3s.n // 2)
            for h in range(grp["H"]):
                ref = r["Q"][h0 + h] @ r["Kt"][h0 + h]
                assert np.abs(Cs[h] - ref).max() < 2.0 ** -20
        h0 += grp["H"]
    c3s.B.blb_plan_destroy(r["plan"])
    c3s.B.blb_keys_destroy(r["keys_g"])


def _out_index(info, grp, o):
    base = 0
    for g in info["groups"]:
        if g is grp or g == grp:
            return base + o
        base += g["n_out"]
    raise AssertionError


# --------------------------------------------------------------------------------------
# graph executors: every replay equals the eager result
# --------------------------------------------------------------------------------------
@pytest.mark.parametrize("fmt", [0, 1])
def test_exec_cp_replays_match_eager(c2s, fmt):
    """Graph replays of a matmul_cp + mask-to-share executor equal eager calls with the same mask
    seeds, with the plan's plaintexts as 64-bit words (fmt 0) or in the 50-bit format (fmt 1); the
    50-bit plan's words also equal those of a 64-bit plan of the same weight."""
    B = c2s.B
    L, d_in, d_out, level = 64, 96, 64, 2
    B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_PLAN_FORMAT, fmt)
    try:
        r = _cp_case(c2s, L, d_in, d_out, level, 77, x_std=1.0)
    finally:
        B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_PLAN_FORMAT, 0)
    n_out = r["g"]["n_out"]
    if fmt:
        plan64 = B.blb_plan_matmul_cp(c2s.h, r["W"], L, level)
        Y64 = [c2s.ct(level - 1) for _ in range(n_out)]
        B.blb_matmul_cp(c2s.h, r["keys_g"], plan64, _xcts(c2s, r, level), Y64)
        for b in range(n_out):
            assert np.array_equal(c2s.export(r["Yc"][b]), c2s.export(Y64[b])), f"50-bit plan against 64-bit plan, output {b}"
        B.blb_plan_destroy(plan64)
    Ye = [c2s.ct(level - 1) for _ in range(n_out)]
    Yg = [c2s.ct(level - 1) for _ in range(n_out)]
    share_e = torch.zeros(n_out * level * c2s.n, dtype=torch.int64, device="cuda")
    share_g = torch.zeros_like(share_e)
    ex = B.blb_exec_create_cp(c2s.h, r["keys_g"], r["plan"], _xcts(c2s, r, level), Yg, level - 1, share_g)
    for rep, seed in enumerate([5, 6, 5]):
        B.blb_exec_run(ex, seed)
        torch.cuda.synchronize()
        got = [c2s.export(y) for y in Yg]
        got_share = share_g.cpu().numpy().copy()
        # eager work between replays
        B.blb_matmul_cp(c2s.h, r["keys_g"], r["plan"], _xcts(c2s, r, level), Ye)
        B.blb_mask_to_share(c2s.h, Ye, seed, level - 1, share_e)
        torch.cuda.synchronize()
        for b in range(n_out):
            assert np.array_equal(got[b], c2s.export(Ye[b])), f"replay {rep} output {b}"
        assert np.array_equal(got_share, share_e.cpu().numpy()), f"replay {rep} share"
    B.blb_exec_destroy(ex)
    B.blb_plan_destroy(r["plan"])
    B.blb_keys_destroy(r["keys_g"])


def test_exec_two_executors_on_two_streams(c2s):
    """Two executors of one plan (own scratch, own outputs) replayed alternately on two streams
    overlap on the device; every output equals an eager run with the same mask seed."""
    B = c2s.B
    L, d_in, d_out, level = 64, 96, 64, 2
    r = _cp_case(c2s, L, d_in, d_out, level, 78, x_std=1.0)
    n_out = r["g"]["n_out"]
    Ys = [[c2s.ct(level - 1) for _ in range(n_out)] for _ in range(2)]
    shares = [torch.zeros(n_out * level * c2s.n, dtype=torch.int64, device="cuda") for _ in range(2)]
    exs = [B.blb_exec_create_cp(c2s.h, r["keys_g"], r["plan"], _xcts(c2s, r, level), Ys[e], level - 1, shares[e]) for e in range(2)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    last = {}
    for k in range(7):
        last[k % 2] = 900 + k
        B.blb_exec_run_stream(exs[k % 2], last[k % 2], streams[k % 2].cuda_stream)
    torch.cuda.synchronize()
    for e in range(2):
        Ye = [c2s.ct(level - 1) for _ in range(n_out)]
        she = torch.zeros_like(shares[e])
        B.blb_matmul_cp(c2s.h, r["keys_g"], r["plan"], _xcts(c2s, r, level), Ye)
        B.blb_mask_to_share(c2s.h, Ye, last[e], level - 1, she)
        torch.cuda.synchronize()
        for b in range(n_out):
            assert np.array_equal(c2s.export(Ys[e][b]), c2s.export(Ye[b])), f"executor {e} output {b}"
        assert np.array_equal(shares[e].cpu().numpy(), she.cpu().numpy()), f"executor {e} share"
    for ex in exs:
        B.blb_exec_destroy(ex)


def _xcts(c, r, level):
    if "_xc" not in r:
        xs = []
        for a in range(r["g"]["n_in"]):
            ct = c.import_ct(r["X_words"][a], level)
            ct.scale = r["scale"]
            xs.append(ct)
        r["_xc"] = xs
    return r["_xc"]


@pytest.mark.parametrize("schedule", [0, 1])
def test_exec_cc_replays_match_eager(c3s, schedule):
    B = c3s.B
    r = _cc_case(c3s, 8, 32, 32, 3, schedule=schedule)
    n_out = r["info"]["n_out"]
    Cg = [c3s.ct(r["level"] - 3) for _ in range(n_out)]
    ex = B.blb_exec_create_cc(c3s.h, r["keys_g"], r["plan"], r["A"], r["B"], Cg)
    for rep in range(3):
        B.blb_exec_run(ex, 0)
        torch.cuda.synchronize()
        got = [c3s.export(x) for x in Cg]
        B.blb_matmul_cc(c3s.h, r["keys_g"], r["plan"], r["A"], r["B"], r["C"])
        torch.cuda.synchronize()
        for o in range(n_out):
            assert np.array_equal(got[o], c3s.export(r["C"][o])), f"replay {rep} output {o}"
    B.blb_exec_destroy(ex)


# --------------------------------------------------------------------------------------
# launch-shape knobs never change a bit
# --------------------------------------------------------------------------------------
def test_ntt_variants_bit_identical(c3s):
    """Every NTT launch shape -- one workgroup per poly or the persistent pipelined grid (knob
    NTT_VARIANT), 16 or 32 values per work-item (knob NTT_RADIX) -- gives identical words through a
    full matmul_cc (rotations, rescales and ModDowns at three levels), equal to the oracle's."""
    B = c3s.B
    r = _cc_case(c3s, 8, 32, 32, 11)
    base = [c3s.export(x) for x in r["C"]]
    default = (B.blb_ctx_get_knob(c3s.h, B.BLB_KNOB_NTT_VARIANT), B.blb_ctx_get_knob(c3s.h, B.BLB_KNOB_NTT_RADIX))
    try:
        for variant in (0, 1):
            for radix in (16, 32):
                B.blb_ctx_set_knob(c3s.h, B.BLB_KNOB_NTT_VARIANT, variant)
                B.blb_ctx_set_knob(c3s.h, B.BLB_KNOB_NTT_RADIX, radix)
                C2 = [c3s.ct(r["level"] - 3) for _ in range(len(r["C"]))]
                B.blb_matmul_cc(c3s.h, r["keys_g"], r["plan"], r["A"], r["B"], C2)
                for o in range(len(C2)):
                    assert np.array_equal(c3s.export(C2[o]), base[o]), f"variant {variant} radix {radix} output {o}"
        for o in range(len(r["want"][0][0])):
            assert np.array_equal(base[o], r["want"][0][0][o])
    finally:
        B.blb_ctx_set_knob(c3s.h, B.BLB_KNOB_NTT_VARIANT, default[0])
        B.blb_ctx_set_knob(c3s.h, B.BLB_KNOB_NTT_RADIX, default[1])
    B.blb_plan_destroy(r["plan"])
    B.blb_keys_destroy(r["keys_g"])


@pytest.mark.parametrize("ks_variant", [0, 2])
def test_ks_variants_bit_identical(c3s, c2s, ks_variant):
    """The per-output key inner product (knob 0) and the key-grouped one forced on every batch
    (knob 2: outputs sharing a key and Galois element in one thread, groups of up to 16, here with
    many outputs per group -- the BSGS ct-ct product's baby steps over several operand ciphertexts and
    its relinearisations, the cp baby steps across inputs) give the oracle's words through a full
    matmul_cc and through matmul_cp."""
    B = c3s.B
    for c, run in ((c3s, "cc"), (c2s, "cp")):
        default = B.blb_ctx_get_knob(c.h, B.BLB_KNOB_KS_VARIANT)
        B.blb_ctx_set_knob(c.h, B.BLB_KNOB_KS_VARIANT, ks_variant)
        try:
            if run == "cc":
                r = _cc_case(c, 12, 64, 32, 21, outputs=[0, 1], schedule=1)
                base = 0
                for O_want, outs, grp in r["want"]:
                    for o in outs:
                        assert np.array_equal(c.export(r["C"][base + o]), O_want[o]), f"cc group H={grp['H']} output {o}"
                    base += grp["n_out"]
                B.blb_plan_destroy(r["plan"])
            else:
                r = _cp_case(c, 100, 96, 80, 2, 7, x_std=1.0)
                want = r["keys_o"].matmul_cp(r["X_words"], 2, r["W"], 100)
                for b in range(r["g"]["n_out"]):
                    assert np.array_equal(c.export(r["Yc"][b]), want[b]), f"cp output {b}"
                B.blb_plan_destroy(r["plan"])
            B.blb_keys_destroy(r["keys_g"])
        finally:
            B.blb_ctx_set_knob(c.h, B.BLB_KNOB_KS_VARIANT, default)


@pytest.mark.parametrize("n_q,n_sp,dnum", [(2, 2, 1), (4, 2, 2), (3, 1, 3), (4, 1, 4), (5, 1, 5)])
@pytest.mark.parametrize("ks_variant", [0, 2])
@pytest.mark.parametrize("n_ct", [1, 2, 17, 33])
def test_ks_inner_by_digits(blb, orc, n_q, n_sp, dnum, ks_variant, n_ct):
    """Key inner products of one to four digits in registers and of five (one output per thread), outputs in
    runs of 1, 2, 16 + 1 and 16 + 16 + 1 of a key: the oracle's words."""
    c = Ctx(blb, orc, 12, n_q, n_sp, dnum)
    blb.blb_ctx_set_knob(c.h, blb.BLB_KNOB_KS_VARIANT, ks_variant)
    steps = [64, -64, 128, -128]
    keys_o = orc.Keys(c.o, 51, sorted({c.o.galois_elt(s) for s in steps}))
    keys_g = blb.blb_keygen(c.h, 51, steps)
    rng = np.random.default_rng(n_ct)
    level = n_q - 1
    words = [keys_o.encrypt(c.o.encode_rns(rng.uniform(-1, 1, c.n // 2), 2.0 ** 30, level), level, 12, t) for t in range(n_ct)]
    cts, outs = [c.import_ct(w, level) for w in words], [c.ct(level) for _ in words]
    blb.blb_rotate_sum(c.h, keys_g, cts, outs, 64, 4, 0, False)
    for t in sorted({0, n_ct // 2, n_ct - 1}):
        assert np.array_equal(c.export(outs[t]), keys_o.rotate_sum(words[t], level, 64, 4, 0, False)), f"ct {t}"
    blb.blb_keys_destroy(keys_g)
    c.close()


@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("shape", [(64, 96, 64), (20, 1, 24)])
def test_mac_variants_bit_identical(c2s, shape, fmt):
    """Every MAC launch shape gives the oracle's words, with the plan's plaintexts held as 64-bit
    words (fmt 0) or in the 50-bit format (fmt 1); the second shape has a single rotated input, so
    the unrolled variants run their remainder loop, and a partial last output tile.  The plan takes
    8N or 25N/4 bytes per limb-poly, and the MAC counts that many plaintext bytes."""
    B = c2s.B
    B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_PLAN_FORMAT, fmt)
    try:
        assert B.blb_ctx_get_knob(c2s.h, B.BLB_KNOB_PLAN_FORMAT) == fmt
        B.blb_ctx_counters(c2s.h, reset=True)
        r = _cp_case(c2s, *shape, 2, 5, x_std=1.0)
        plaintext_bytes = B.blb_ctx_counters(c2s.h)["plaintext_bytes"]
    finally:
        B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_PLAN_FORMAT, 0)
    g = r["g"]
    n_pt = g["n_out"] * g["G"] * g["n_in"] * g["B"]
    poly_bytes = c2s.n * 25 // 4 if fmt else c2s.n * 8
    assert plaintext_bytes == n_pt * 3 * poly_bytes
    base = [c2s.export(y) for y in r["Yc"]]
    want = r["keys_o"].matmul_cp(r["X_words"], 2, r["W"], shape[0])
    assert all(np.array_equal(base[b], want[b]) for b in range(len(base)))
    Xc = _xcts(c2s, r, 2)
    for var in range(B.BLB_MAC_VARIANTS):
        B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_MAC_VARIANT, var)
        Y = [c2s.ct(1) for _ in range(len(base))]
        B.blb_matmul_cp(c2s.h, r["keys_g"], r["plan"], Xc, Y)
        for b in range(len(Y)):
            assert np.array_equal(c2s.export(Y[b]), base[b]), f"variant {var}"
    B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_MAC_VARIANT, 0)
    torch.cuda.synchronize()
    held = B.blb_ctx_device_bytes(c2s.h)
    B.blb_plan_destroy(r["plan"])
    assert held - B.blb_ctx_device_bytes(c2s.h) == n_pt * 3 * poly_bytes  # the plan's own allocation
    B.blb_keys_destroy(r["keys_g"])


@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("d_out", [33, 128, 250, 512, 760, 1400])
def test_mac_shape_by_size(c2s, d_out, fmt):
    """The launch shape taken by size (knob 0) at sizes on each side of every bound of its rule (2 to
    44 column blocks, 8 to 176 outputs) gives the words of a fixed 8 x 2 shape, a partial last tile and
    an input count that is no multiple of the waves sharing the terms included."""
    B = c2s.B
    L, d_in, level = 100, 40, 2
    rng = np.random.default_rng(1700 + d_out)
    B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_PLAN_FORMAT, fmt)
    try:
        plan = B.blb_plan_matmul_cp(c2s.h, rng.normal(0, 0.02, (d_in, d_out)), L, level)
    finally:
        B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_PLAN_FORMAT, 0)
    g = B.blb_plan_info(plan)
    keys = B.blb_keygen(c2s.h, 1701, [i * g["Lp"] for i in range(1, g["B"])] + [j * g["B"] * g["Lp"] for j in range(1, g["G"])])
    mods = B.blb_ctx_moduli(c2s.h, c2s.n_q + c2s.n_sp)[: level + 1]
    X = [c2s.ct(level) for _ in range(g["n_in"])]
    for x in X:  # any residues do: the product is exact
        B.blb_import(c2s.h, np.stack([np.stack([rng.integers(0, int(q), c2s.n, dtype=np.uint64) for q in mods]) for _ in range(2)]), x)
        x.scale = 2.0 ** 40
    words = []
    for var in (13, 0):
        B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_MAC_VARIANT, var)
        Y = [c2s.ct(level - 1) for _ in range(g["n_out"])]
        B.blb_matmul_cp(c2s.h, keys, plan, X, Y)
        words.append([c2s.export(y) for y in Y])
    assert all(np.array_equal(a, b) for a, b in zip(*words))
    torch.cuda.synchronize()
    B.blb_plan_destroy(plan)
    B.blb_keys_destroy(keys)


def test_descriptor_ring_wraps(c1):
    """Eager calls whose tables fill the 64 MiB descriptor ring more than once (about 3 KiB a rotation):
    the last rotations equal the first, word for word."""
    B = c1.B
    rng = np.random.default_rng(1801)
    steps = [1, 5]
    keys = B.blb_keygen(c1.h, 1802, steps)
    x, level = c1.ct(1), 1
    mods = B.blb_ctx_moduli(c1.h, c1.n_q + c1.n_sp)[: level + 1]
    B.blb_import(c1.h, np.stack([np.stack([rng.integers(0, int(q), c1.n, dtype=np.uint64) for q in mods]) for _ in range(2)]), x)
    x.scale = 2.0 ** 30
    y = [c1.ct(level) for _ in steps]
    for k, st in enumerate(steps):
        B.blb_rotate(c1.h, keys, x, st, y[k])
    want = [c1.export(v) for v in y]
    for i in range(30000):
        B.blb_rotate(c1.h, keys, x, steps[i % 2], y[i % 2])
    assert all(np.array_equal(c1.export(v), w) for v, w in zip(y, want))
    B.blb_keys_destroy(keys)


@pytest.mark.parametrize("n_blocks", [1, 2, 4])
@pytest.mark.parametrize("direction,mask", [(0, False), (0, True), (1, False)])
def test_rotate_sum_overlapping_outputs(c1, n_blocks, direction, mask):
    """Sums and broadcasts of no, one and two steps whose outputs are the inputs' buffers in another
    order give the words of a call with buffers of its own."""
    B = c1.B
    rng = np.random.default_rng(1803 + n_blocks)
    block, level, n_ct = 64, 1, 3
    steps = [s * st for st in (block, 2 * block) for s in (1, -1)]
    keys = B.blb_keygen(c1.h, 1804, steps)
    mods = B.blb_ctx_moduli(c1.h, c1.n_q + c1.n_sp)[: level + 1]
    words = [np.stack([np.stack([rng.integers(0, int(q), c1.n, dtype=np.uint64) for q in mods]) for _ in range(2)]) for _ in range(n_ct)]

    def inputs():
        out = [c1.ct(level) for _ in range(n_ct)]
        for x, w in zip(out, words):
            B.blb_import(c1.h, w, x)
            x.scale = 2.0 ** 30
        return out

    own = [c1.ct(level) for _ in range(n_ct)]
    B.blb_rotate_sum(c1.h, keys, inputs(), own, block, n_blocks, direction, mask)
    x = inputs()
    over = [B.blb_ct(x[(t + 1) % n_ct].data, level, 1, 0.0) for t in range(n_ct)]
    B.blb_rotate_sum(c1.h, keys, x, over, block, n_blocks, direction, mask)
    for a, b in zip(own, over):
        assert (a.level, a.scale) == (b.level, b.scale)
        assert np.array_equal(c1.export(a), c1.export(b))
    B.blb_keys_destroy(keys)


@pytest.mark.parametrize("d_out,d_out2", [(96, 96), (96, 80), (96, 32)])
def test_plan_memory_is_reused_and_given_back(c1, d_out, d_out2):
    """A plan made in a destroyed plan's memory (the same size, a little smaller, too small to take it)
    gives the words of one in fresh memory; blb_ctx_device_bytes counts the plan's own bytes either
    way, and blb_ctx_trim returns what is kept to the device."""
    B = c1.B
    rng = np.random.default_rng(1805)
    L, d_in, level = 16, 64, 1
    W, W2 = rng.normal(0, 0.02, (d_in, d_out)), rng.normal(0, 0.02, (d_in, d_out2))
    mods = B.blb_ctx_moduli(c1.h, c1.n_q + c1.n_sp)[: level + 1]
    keys = X = None

    def product(plan):
        nonlocal keys, X
        g = B.blb_plan_info(plan)
        if keys is None:
            keys = B.blb_keygen(c1.h, 1806, [i * g["Lp"] for i in range(1, g["B"])] + [j * g["B"] * g["Lp"] for j in range(1, g["G"])])
            X = [c1.ct(level) for _ in range(g["n_in"])]
            for x in X:
                B.blb_import(c1.h, np.stack([np.stack([rng.integers(0, int(q), c1.n, dtype=np.uint64) for q in mods]) for _ in range(2)]), x)
                x.scale = 2.0 ** 30
        Y = [c1.ct(level - 1) for _ in range(g["n_out"])]
        B.blb_matmul_cp(c1.h, keys, plan, X, Y)
        return [c1.export(y) for y in Y]

    def bytes_of(plan):
        g = B.blb_plan_info(plan)
        return g["n_out"] * g["G"] * g["n_in"] * g["B"] * (level + 1) * c1.n * 8

    B.blb_ctx_trim(c1.h)
    plan = B.blb_plan_matmul_cp(c1.h, W2, L, level)  # fresh memory
    want = product(plan)
    B.blb_plan_destroy(plan)
    B.blb_ctx_trim(c1.h)
    free0 = torch.cuda.mem_get_info()[0]
    first = B.blb_plan_matmul_cp(c1.h, W, L, level)
    size = bytes_of(first)
    product(first)
    B.blb_plan_destroy(first)
    held = B.blb_ctx_device_bytes(c1.h)
    plan = B.blb_plan_matmul_cp(c1.h, W2, L, level)  # in the first plan's memory where it fits
    assert B.blb_ctx_device_bytes(c1.h) - held == bytes_of(plan)
    got = product(plan)
    assert all(np.array_equal(a, b) for a, b in zip(want, got))
    B.blb_plan_destroy(plan)
    assert B.blb_ctx_device_bytes(c1.h) == held
    B.blb_ctx_trim(c1.h)
    assert torch.cuda.mem_get_info()[0] >= free0 - (size // 2 if size > (64 << 20) else 0)
    B.blb_keys_destroy(keys)


# --------------------------------------------------------------------------------------
# the batched transform on its own
# --------------------------------------------------------------------------------------
def _brv(log_n):
    j = np.arange(1 << log_n)
    r = np.zeros_like(j)
    for b in range(log_n):
        r |= ((j >> b) & 1) << (log_n - 1 - b)
    return r


@pytest.mark.parametrize("name,n_polys", [("c1", 3), ("c2s", 5), ("c3s", 37)])
@pytest.mark.parametrize("variant,radix", [(0, 16), (1, 16), (0, 32), (1, 32)])
def test_ntt_matches_oracle(request, name, n_polys, variant, radix):
    """blb_ntt: word j of the forward transform is the evaluation at psi^(2 brv(j) + 1), which is
    entry brv(j) of the oracle's natural-order textbook transform; every prime of the chain
    (special primes included); the inverse returns the input exactly; a ragged poly count."""
    c = request.getfixturevalue(name)
    B = c.B
    mods = B.blb_ctx_moduli(c.h, c.n_q + c.n_sp)
    nl = len(mods)
    log_n = int(np.log2(c.n))
    rng = np.random.default_rng(1000 + n_polys)
    words = np.stack([np.stack([rng.integers(0, int(q), c.n, dtype=np.uint64) for q in mods]) for _ in range(n_polys)])
    dev = c.upload_words(words)
    default = (B.blb_ctx_get_knob(c.h, B.BLB_KNOB_NTT_VARIANT), B.blb_ctx_get_knob(c.h, B.BLB_KNOB_NTT_RADIX))
    B.blb_ctx_set_knob(c.h, B.BLB_KNOB_NTT_VARIANT, variant)
    B.blb_ctx_set_knob(c.h, B.BLB_KNOB_NTT_RADIX, radix)
    try:
        B.blb_ntt(c.h, dev, n_polys, nl, inverse=False)
        torch.cuda.synchronize()
        got = dev.cpu().numpy().view(np.uint64).reshape(n_polys, nl, c.n)
        perm = _brv(log_n)
        for p in sorted({0, n_polys - 1}):
            for m in range(nl):
                want = c.o.ntt_forward(m, words[p, m])
                assert np.array_equal(got[p, m], want[perm]), f"poly {p} limb {m}"
        B.blb_ntt(c.h, dev, n_polys, nl, inverse=True)
        torch.cuda.synchronize()
        back = dev.cpu().numpy().view(np.uint64).reshape(n_polys, nl, c.n)
        assert np.array_equal(back, words)
    finally:
        B.blb_ctx_set_knob(c.h, B.BLB_KNOB_NTT_VARIANT, default[0])
        B.blb_ctx_set_knob(c.h, B.BLB_KNOB_NTT_RADIX, default[1])
    with pytest.raises(B.BlbError):
        B.blb_ntt(c.h, dev, 1, nl + 1)
    B.blb_ntt(c.h, dev, 0, 1)


@pytest.mark.parametrize("n_q,n_sp,dnum", [(3, 1, 3), (4, 2, 2), (3, 2, 3), (4, 3, 2)])
@pytest.mark.parametrize("radix", [16, 32])
def test_transforms_in_halves(blb, orc, n_q, n_sp, dnum, radix):
    """N = 16384: the transforms that take half a polynomial per workgroup (base conversions from one or two
    limbs, rescale) give the oracle's words, with a permuted operand added (its halves stay apart under the
    Galois element) and, in the rotate-and-sum, with both; digits of one, of two and of
    an uneven number of limbs, special primes of one to three (three: whole polynomials)."""
    c = Ctx(blb, orc, 14, n_q, n_sp, dnum)
    blb.blb_ctx_set_knob(c.h, blb.BLB_KNOB_NTT_RADIX, radix)
    steps = [1, -7, 4096, -4096, 2048, -2048]
    keys_o = orc.Keys(c.o, 77, sorted({c.o.galois_elt(s) for s in steps}))
    keys_g = blb.blb_keygen(c.h, 77, steps)
    rng = np.random.default_rng(14 + n_q)
    for level in range(n_q - 1, -1, -1):
        words = np.stack([np.stack([rng.integers(0, int(q), c.n, dtype=np.uint64) for q in c.o.q[: level + 1]]) for _ in range(2)])
        words[0, :, :5] = (c.o.q[: level + 1] - 1)[:, None]
        words[1, :, 9000:9005] = 0
        for s in (1, -7):
            ct, out = c.import_ct(words, level), c.ct(level)
            blb.blb_rotate(c.h, keys_g, ct, s, out)
            assert np.array_equal(c.export(out), keys_o.rotate(words, level, s)), f"rotation {s} at level {level}"
        if level > 0:
            ct, out = c.import_ct(words, level), c.ct(level - 1)
            blb.blb_rescale(c.h, ct, out)
            assert np.array_equal(c.export(out), c.o.rescale(words, level)), f"rescale at level {level}"
    level = n_q - 1
    words = [keys_o.encrypt(c.o.encode_rns(rng.uniform(-1, 1, c.n // 2), 2.0 ** 30, level), level, 12, t) for t in range(5)]
    cts, outs = [c.import_ct(w, level) for w in words], [c.ct(level) for _ in words]
    blb.blb_rotate_sum(c.h, keys_g, cts, outs, 2048, 4, 0, False)
    for t, w in enumerate(words):
        assert np.array_equal(c.export(outs[t]), keys_o.rotate_sum(w, level, 2048, 4, 0, False)), f"ct {t}"
    blb.blb_keys_destroy(keys_g)
    c.close()


@pytest.mark.parametrize("name,block,n_ct", [("c1", 64, 1), ("c1", 512, 3), ("c2s", 1024, 2), ("c3s", 2048, 1), ("c3s", 4096, 3)])
@pytest.mark.parametrize("radix", [16, 32])
def test_masked_rescale_in_transforms(request, name, block, n_ct, radix):
    """The mask product formed by the rescale's transforms (whole limb-polys, and halves at N = 16384): the
    oracle's rotate-and-sum with the first-block mask, from random residues with 0 and q - 1 among them."""
    c = request.getfixturevalue(name)
    c.B.blb_ctx_set_knob(c.h, c.B.BLB_KNOB_NTT_RADIX, radix)
    keys_o = c.orc.Keys(c.o, 61, sorted({c.o.galois_elt(s) for s in (block, -block)}))
    keys_g = c.B.blb_keygen(c.h, 61, [block, -block])
    rng = np.random.default_rng(block + n_ct)
    level = c.n_q - 1
    words = []
    for t in range(n_ct):
        w = np.stack([np.stack([rng.integers(0, int(q), c.n, dtype=np.uint64) for q in c.o.q[: level + 1]]) for _ in range(2)])
        w[t % 2, :, 100:200] = (c.o.q[: level + 1] - 1)[:, None]
        w[t % 2, :, 300:400] = 0
        words.append(w)
    cts, outs = [c.import_ct(w, level) for w in words], [c.ct(level - 1) for _ in words]
    c.B.blb_rotate_sum(c.h, keys_g, cts, outs, block, 2, 0, True)
    for t in range(n_ct):
        assert np.array_equal(c.export(outs[t]), keys_o.rotate_sum(words[t], level, block, 2, 0, True)), f"ct {t}"
    c.B.blb_keys_destroy(keys_g)
    c.B.blb_ctx_set_knob(c.h, c.B.BLB_KNOB_NTT_RADIX, 16)


@pytest.mark.parametrize("n_polys", [85, 86, 130])
def test_ntt_persistent_grid(c3s, n_polys):
    """The persistent grid (N = 16384, more than two limb-polys per compute unit: 86 and 130 polys of 6 limbs
    on 256 of them; 85 is one workgroup each) gives the words of one workgroup per limb-poly in both
    directions, and the inverse returns the input; the extreme residues 0 and q - 1 are among them."""
    B = c3s.B
    mods = B.blb_ctx_moduli(c3s.h, c3s.n_q + c3s.n_sp)
    rng = np.random.default_rng(1807 + n_polys)
    one = np.stack([rng.integers(0, int(q), c3s.n, dtype=np.uint64) for q in mods])
    one[:, :64] = 0
    one[:, 64:128] = (mods - 1)[:, None]
    words = np.stack([np.roll(one, 37 * p, axis=1) for p in range(n_polys)])
    words[-1] = (mods - 1)[:, None]
    out = []
    for variant in (0, 1):
        B.blb_ctx_set_knob(c3s.h, B.BLB_KNOB_NTT_VARIANT, variant)
        t = torch.from_numpy(words.view(np.int64).reshape(-1).copy()).cuda()
        B.blb_ntt(c3s.h, t, n_polys, len(mods))
        torch.cuda.synchronize()
        fwd = t.cpu().numpy().copy()
        B.blb_ntt(c3s.h, t, n_polys, len(mods), True)
        torch.cuda.synchronize()
        assert np.array_equal(t.cpu().numpy().view(np.uint64).reshape(words.shape), words)
        out.append(fwd)
    B.blb_ctx_set_knob(c3s.h, B.BLB_KNOB_NTT_VARIANT, 1)
    assert np.array_equal(out[0], out[1])


# --------------------------------------------------------------------------------------
# digits of three and more primes, three and four special primes
# --------------------------------------------------------------------------------------
@pytest.mark.parametrize("n_q,n_sp,dnum", [(6, 1, 2), (8, 2, 1), (5, 4, 2), (5, 3, 3), (10, 1, 3)])
@pytest.mark.parametrize("log_n", [12, 13, 14])
def test_wide_digits(blb, orc, log_n, n_q, n_sp, dnum):
    """Base conversions of up to eight source primes and of three and four special primes: rotations and a
    rotate-and-sum over several sources give the oracle's words, from residues with 0 and q - 1 among them, at
    the levels where the digits are full, where the last one is shorter and where one prime is left."""
    c = Ctx(blb, orc, log_n, n_q, n_sp, dnum)
    steps = [64, 128, -3]
    keys_o = orc.Keys(c.o, 91, sorted({c.o.galois_elt(s) for s in steps}))
    keys_g = blb.blb_keygen(c.h, 91, steps)
    rng = np.random.default_rng(100 * log_n + n_q)

    def residues(level, t):
        w = np.stack([np.stack([rng.integers(0, int(q), c.n, dtype=np.uint64) for q in c.o.q[: level + 1]]) for _ in range(2)])
        w[1, :, 100 * t:100 * t + 64] = (c.o.q[: level + 1] - 1)[:, None]
        w[t % 2, :, 2000:2064] = 0
        w[1, level, 3000:] = int(c.o.q[level]) - 1
        return w

    for level in sorted({n_q - 1, n_q - 2, (n_q - 1) // 2, 0}):
        w = residues(level, 0)
        ct, out = c.import_ct(w, level), c.ct(level)
        blb.blb_rotate(c.h, keys_g, ct, -3, out)
        assert np.array_equal(c.export(out), keys_o.rotate(w, level, -3)), f"rotation at level {level}"
    level = n_q - 1
    words = [residues(level, t) for t in range(3)]
    cts, outs = [c.import_ct(w, level) for w in words], [c.ct(level) for _ in words]
    blb.blb_rotate_sum(c.h, keys_g, cts, outs, 64, 4, 0, False)
    for t, w in enumerate(words):
        assert np.array_equal(c.export(outs[t]), keys_o.rotate_sum(w, level, 64, 4, 0, False)), f"ct {t}"
    blb.blb_keys_destroy(keys_g)
    c.close()


# --------------------------------------------------------------------------------------
# terms that do not divide over the waves that share them; kept plan memory
# --------------------------------------------------------------------------------------
@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("L,d_in,n_ai", [(4096, 7, 7), (4096, 3, 3), (4096, 1, 1), (2048, 5, 6)])
@pytest.mark.parametrize("n_bj", [5, 11, 30])
def test_mac_uneven_terms(c2s, L, d_in, n_ai, n_bj, fmt):
    """The launch shapes that divide a product's terms over two and four waves (5 and 11 outputs: four, 30: two)
    with numbers of terms that are no multiple of them, or fewer than the waves, give the words of a shape
    whose waves take all terms."""
    B = c2s.B
    level, c = 2, 4096 // L
    rng = np.random.default_rng(1900 + n_bj)
    B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_PLAN_FORMAT, fmt)
    try:
        plan = B.blb_plan_matmul_cp(c2s.h, rng.normal(0, 0.02, (d_in, c * n_bj)), L, level)
    finally:
        B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_PLAN_FORMAT, 0)
    g = B.blb_plan_info(plan)
    assert (g["n_in"] * g["B"], g["n_out"] * g["G"]) == (n_ai, n_bj)
    keys = B.blb_keygen(c2s.h, 1901, [i * g["Lp"] for i in range(1, g["B"])] + [j * g["B"] * g["Lp"] for j in range(1, g["G"])])
    X = [c2s.ct(level) for _ in range(g["n_in"])]
    for x in X:
        B.blb_import(c2s.h, np.stack([np.stack([rng.integers(0, int(q), c2s.n, dtype=np.uint64) for q in c2s.o.q[: level + 1]])
                                      for _ in range(2)]), x)
        x.scale = 2.0 ** 40
    words = []
    for var in (13, 0):
        B.blb_ctx_set_knob(c2s.h, B.BLB_KNOB_MAC_VARIANT, var)
        Y = [c2s.ct(level - 1) for _ in range(g["n_out"])]
        B.blb_matmul_cp(c2s.h, keys, plan, X, Y)
        words.append([c2s.export(y) for y in Y])
    assert all(np.array_equal(a, b) for a, b in zip(*words))
    torch.cuda.synchronize()
    B.blb_plan_destroy(plan)
    B.blb_keys_destroy(keys)


@pytest.mark.parametrize("blocks,taken", [(10, True), (9, True), (7, False)])
def test_plan_in_kept_memory(c1, blocks, taken):
    """A plan of `blocks` column blocks (16 MiB each) made after one of 10 was destroyed takes its memory where
    at most a quarter of its own size is wasted, and gives the words of a plan in memory of its own either way.
    Taken or not is read from the device's free memory, which the temporaries' 35 MiB and their stack change
    too: less than half of a plan's size (112 to 160 MiB) means that it was taken."""
    B = c1.B
    rng = np.random.default_rng(1902)
    L, d_in, level = 16, 256, 1
    W = rng.normal(0, 0.02, (d_in, 1280))
    plan = B.blb_plan_matmul_cp(c1.h, W[:, : 128 * blocks], L, level)
    g = B.blb_plan_info(plan)
    assert (g["n_out"], g["G"] * g["n_in"] * g["B"]) == (blocks, 256)
    keys = B.blb_keygen(c1.h, 1903, [i * g["Lp"] for i in range(1, g["B"])] + [j * g["B"] * g["Lp"] for j in range(1, g["G"])])
    X = [c1.ct(level) for _ in range(g["n_in"])]
    for x in X:
        B.blb_import(c1.h, np.stack([np.stack([rng.integers(0, int(q), c1.n, dtype=np.uint64) for q in c1.o.q[: level + 1]])
                                     for _ in range(2)]), x)
        x.scale = 2.0 ** 30

    def product(p):
        Y = [c1.ct(level - 1) for _ in range(blocks)]
        B.blb_matmul_cp(c1.h, keys, p, X, Y)
        return [c1.export(y) for y in Y]

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    want = product(plan)
    B.blb_plan_destroy(plan)
    B.blb_ctx_trim(c1.h)
    first = B.blb_plan_matmul_cp(c1.h, W, L, level)
    before = free()
    B.blb_plan_destroy(first)
    assert free() - before < 80 << 20, "the block was not kept"
    held = B.blb_ctx_device_bytes(c1.h)
    plan = B.blb_plan_matmul_cp(c1.h, W[:, : 128 * blocks], L, level)
    size = blocks * 256 * (level + 1) * c1.n * 8
    grown = B.blb_ctx_device_bytes(c1.h) - held - size  # the temporaries
    assert (before - free() - grown < size / 2) == taken
    got = product(plan)
    assert all(np.array_equal(a, b) for a, b in zip(want, got))
    B.blb_plan_destroy(plan)
    B.blb_keys_destroy(keys)
    B.blb_ctx_trim(c1.h)


@pytest.mark.parametrize("name,L", [("c1", 16), ("c2s", 32)])
@pytest.mark.parametrize("blocks", [1, 64, 65])
def test_encoder_few_and_many_vectors(request, name, L, blocks):
    """Plans of 1, 32 and 33 complex vectors (one plaintext a column block, two a vector): the encoder's column
    pass takes narrow workgroups up to 32 of them and wide ones beyond; the product is the oracle's."""
    c = request.getfixturevalue(name)
    r = _cp_case(c, L, 1, 128 * blocks, c.n_q - 1, 1904)
    assert r["g"]["n_out"] * r["g"]["G"] * r["g"]["n_in"] * r["g"]["B"] == blocks
    want = r["keys_o"].matmul_cp(r["X_words"], c.n_q - 1, r["W"], L)
    for b in range(blocks):
        assert np.array_equal(c.export(r["Yc"][b]), want[b]), f"output {b}"
    c.B.blb_plan_destroy(r["plan"])
    c.B.blb_keys_destroy(r["keys_g"])


def test_encode_overflow_leaves_the_plaintext(c1):
    """A vector whose coefficients pass the encoder's range is refused with the plaintext buffer as it was, and
    the next vector is encoded."""
    v = np.random.default_rng(1905).normal(0, 1, c1.n // 2)
    pt = c1.pt_dev(1)
    pt.fill_(-7)
    with pytest.raises(c1.B.BlbError) as e:
        c1.B.blb_encode(c1.h, v, 2.0 ** 80, 1, pt)
    assert e.value.code == c1.B.BLB_EINVAL
    assert bool((pt == -7).all())
    c1.B.blb_encode(c1.h, v, 2.0 ** 40, 1, pt)
    torch.cuda.synchronize()
    assert np.array_equal(pt.cpu().numpy().view(np.uint64).reshape(2, c1.n), c1.o.encode_rns(v, 2.0 ** 40, 1))
