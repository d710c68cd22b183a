"""Host paths of the library on a machine without a GPU: libblb.so over a HIP runtime of host memory
(tests/host/hip_stub.cpp), where kernels do not run.  Memory accounting, failures of the runtime or of host
allocations, and what is launched in which order.

Each case runs in a process of its own (the stub has to be loaded before the library):
``python test_host_paths_cpu.py STUB CASE``.
"""
import ctypes
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
sys.path.insert(0, ROOT)
N = 4096


# ---------------------------------------------------------------------------------------
# cases (run in the child)
# ---------------------------------------------------------------------------------------
class Stub:
    def __init__(self, path):
        self.l = ctypes.CDLL(path, mode=ctypes.RTLD_GLOBAL)
        for name in ("stub_live", "stub_peak"):
            getattr(self.l, name).restype = ctypes.c_size_t
        for name in ("stub_launch_name", "stub_event"):
            getattr(self.l, name).restype = ctypes.c_char_p
        self.l.stub_launch_arg0.restype = ctypes.c_void_p
        self.l.stub_cap.argtypes = self.l.stub_total.argtypes = [ctypes.c_size_t]
        self.l.stub_fail_new.argtypes = [ctypes.c_long]

    def __getattr__(self, name):
        return getattr(self.l, "stub_" + name)

    def events(self):
        return [self.l.stub_event(i).decode() for i in range(self.l.stub_events())]


def _buf(B, words, level):
    import numpy as np
    a = np.zeros(words, np.uint64)
    c = B.blb_ct(a.ctypes.data, level, 1, 2.0 ** 30)
    return c, a


def _plan(B, h, n_out):
    """16 x 256 times 256 x 128 n_out at level 1, N = 4096: 16 MiB a column block"""
    import numpy as np
    plan = B.blb_plan_matmul_cp(h, np.zeros((256, 128 * n_out)), 16, 1)
    g = B.blb_plan_info(plan)
    assert g["n_out"] == n_out
    return plan, g["n_out"] * g["G"] * g["n_in"] * g["B"] * 2 * N * 8


def case_budget_caps_kept_plan_memory(S, B):
    """What the context holds (plans with their blocks' full size, kept blocks, grown temporaries) stays
    within hbm_budget_bytes, and a plan of a kept block's size takes that block."""
    mb = 1 << 20
    h = B.blb_ctx_create(12, 2, 1, 2, 0, None)
    K = B.blb_keygen(h, 1, [64])
    base = B.blb_ctx_device_bytes(h)
    B.blb_keys_destroy(K)
    B.blb_ctx_destroy(h)
    budget = base + 164 * mb
    h = B.blb_ctx_create(12, 2, 1, 2, 0, None, budget)
    uncounted = S.live() - B.blb_ctx_device_bytes(h)  # the descriptor ring
    K = B.blb_keygen(h, 1, [64])

    def check(what):
        assert S.live() - uncounted <= budget, f"{what}: {(S.live() - uncounted - budget) / mb:.0f} MiB over"

    plan, size = _plan(B, h, 10)
    check("one plan")
    B.blb_plan_destroy(plan)
    before = S.live()
    plan, same = _plan(B, h, 10)
    assert same == size and S.live() == before, "the kept block was not taken"
    B.blb_plan_destroy(plan)
    # a plan a tenth smaller than the kept block, and one in the bytes that are then left
    plan, smaller = _plan(B, h, 9)
    assert size * 4 / 5 <= smaller < size
    check("a smaller plan")
    other, _ = _plan(B, h, 1)
    check("another plan beside it")
    B.blb_plan_destroy(other)
    B.blb_plan_destroy(plan)
    check("kept blocks")
    # temporaries that grow by about 100 MiB beside kept blocks of 160
    k = 300
    a = _buf(B, 2 * k * 4 * N, 1)[1]
    cts = [[B.blb_ct(a.ctypes.data + (o * k + t) * 4 * N * 8, 1, 1, 2.0 ** 30) for t in range(k)] for o in range(2)]
    held = B.blb_ctx_device_bytes(h)
    for _ in range(3):
        B.blb_rotate_sum(h, K, cts[0], cts[1], 64, 2, 0, False)
        check("grown temporaries")
    assert B.blb_ctx_device_bytes(h) >= held + 64 * mb
    B.blb_keys_destroy(K)
    B.blb_ctx_destroy(h)
    assert S.live() == 0


def case_kept_plan_memory_is_given_back_to_any_allocation(S, B):
    """With the device's memory short of what a new context's descriptor ring, a server's weights or a server's
    plan arena take, and more than that in a destroyed plan's block, the allocation succeeds."""
    import numpy as np
    mb = 1 << 20

    def short_of(bytes_free):
        S.cap(0)
        plan, size = _plan(B, h, 10)
        B.blb_plan_destroy(plan)
        assert size == 160 * mb
        S.cap(S.live() + bytes_free)

    h = B.blb_ctx_create(12, 2, 1, 2, 0, None)
    short_of(32 * mb)
    h2 = B.blb_ctx_create(12, 2, 1, 2, 0, 0x5000)  # 64 MiB ring, 2 MiB of tables
    S.cap(0)
    h3 = B.blb_ctx_create(12, 2, 1, 2, 0, 0x6000)
    srv = B.blb_server_create(h2, 1 * mb)
    short_of(32 * mb)
    B.blb_server_add_weights(srv, 1, np.zeros((2048, 4096)), 1)  # 64 MiB
    short_of(32 * mb)
    srv2 = B.blb_server_create(h3, 64 * mb)
    for s in (srv, srv2):
        B.blb_server_destroy(s)
    S.cap(0)
    for x in (h, h2, h3):
        B.blb_ctx_destroy(x)
    assert S.live() == 0


def case_failed_copy_is_the_calls_result(S, B):
    """A device copy that fails is BLB_EDEVICE from the call that made it, with launches held back and with
    timing on (nothing held), in the allocation-free rotation too; the next call is not blamed for it."""
    h = B.blb_ctx_create(12, 2, 1, 2, 0, None)
    K = B.blb_keygen(h, 1, [64])
    x, xa = _buf(B, 4 * N, 1)
    y, ya = _buf(B, 4 * N, 1)
    for timing in (0, 1):
        B.blb_ctx_set_timing(h, timing)
        for call in (lambda: B.blb_rotate(h, K, x, 0, y), lambda: B.blb_rotate_noalloc(h, K, x, 0, y),
                     lambda: B.blb_rotate_sum(h, K, [x], [y], 64, 1, 0, False)):
            S.fail_copies(1)
            try:
                call()
            except B.BlbError as e:
                assert e.code == B.BLB_EDEVICE
            else:
                raise AssertionError("a failed copy was not reported")
            S.fail_copies(0)
            B.blb_rotate(h, K, x, 64, y)
            call()
    B.blb_keys_destroy(K)
    B.blb_ctx_destroy(h)


def case_failed_host_allocation_is_a_status(S, B):
    """Every host allocation of an eager call made to fail in turn: the call returns BLB_ENOMEM (no exception
    crosses the C boundary), and the same call then succeeds with the launches of a call of its own; with
    launches held back and not (timing)."""
    L = B.lib()
    ref = ctypes.byref
    h = B.blb_ctx_create(12, 2, 1, 2, 0, None)
    plan, _ = _plan(B, h, 1)
    g = B.blb_plan_info(plan)
    K = B.blb_keygen(h, 1, [64] + [i * g["Lp"] for i in range(1, g["B"])] + [j * g["B"] * g["Lp"] for j in range(1, g["G"])])
    x = [_buf(B, 4 * N, 1) for _ in range(2)]
    y = [_buf(B, 4 * N, 1) for _ in range(2)]
    xa, ya = (B.blb_ct * 2)(*[c for c, _ in x]), (B.blb_ct * 2)(*[c for c, _ in y])
    calls = {"rotate": lambda: L.blb_rotate(h, K, ref(xa[0]), 64, ref(ya[0])),
             "rotate_sum": lambda: L.blb_rotate_sum(h, K, xa, 2, 64, 2, 0, 1, ya),
             "mul_relin": lambda: L.blb_ew_mul_relin(h, K, xa, xa, 2, ya),
             "scalar_op": lambda: L.blb_scalar_op(h, K, xa, xa, 2, 64, 2, 1, 0, ya),
             "matmul_cp": lambda: L.blb_matmul_cp(h, K, plan, xa, 2, ya, 1)}
    K2 = B.blb_keygen(h, 1, [-64])
    calls["scalar_op"] = lambda: L.blb_scalar_op(h, K2, xa, xa, 2, 64, 2, 1, 0, ya)

    def launched(call):
        for t in range(2):
            xa[t].level, ya[t].level = 1, 1
        S.clear()
        rc = call()
        return rc, [S.launch_name(i) for i in range(S.launches()) if b"k_stage" not in S.launch_name(i)]

    for timing in (0, 1):
        B.blb_ctx_set_timing(h, timing)
        for name, call in calls.items():
            launched(call)
            rc, want = launched(call)
            assert rc == 0 and want, name
            failures = 0
            for k in range(1, 2000):
                S.fail_new(k)
                rc, _ = launched(call)
                S.fail_new(0)
                if rc == 0:
                    break
                assert rc == B.BLB_ENOMEM, (name, k, rc)
                failures += 1
                assert launched(call) == (0, want), (name, k)
            assert failures >= 5, (name, failures)
    B.blb_ctx_set_timing(h, 0)
    for k in (K, K2):
        B.blb_keys_destroy(k)
    plans = [plan] + [_plan(B, h, 1)[0] for _ in range(40)]
    for p in plans:  # (the list of kept blocks grows now and then)
        S.fail_new(1)
        L.blb_plan_destroy(p)
        S.fail_new(0)
    B.blb_ctx_destroy(h)
    assert S.live() == 0


def case_refused_wait_of_a_plans_destruction(S, B):
    """Where the device cannot be waited for (another thread records a graph), a destroyed plan's memory goes
    back to the device at once, and the next call is not blamed for the refused wait."""
    h = B.blb_ctx_create(12, 2, 1, 2, 0, None)
    K = B.blb_keygen(h, 1, [64])
    x, xa = _buf(B, 4 * N, 1)
    y, ya = _buf(B, 4 * N, 1)
    for _ in range(2):  # (the temporaries grow to their size)
        plan, size = _plan(B, h, 2)
        B.blb_plan_destroy(plan)
        B.blb_ctx_trim(h)
    plan, size = _plan(B, h, 2)
    B.blb_rotate(h, K, x, 64, y)
    held = S.live()
    S.fail_device_syncs(1)
    B.blb_plan_destroy(plan)
    S.fail_device_syncs(0)
    assert held - S.live() == size
    B.blb_rotate(h, K, x, 64, y)
    B.blb_keys_destroy(K)
    B.blb_ctx_destroy(h)


def case_base_conversions_in_whole_runs(S, B):
    """The descriptors of every base conversion come in runs that read the same source limbs (the runs that meet
    in one XCD's L2): the digits of a source at every level, a shorter last digit, launches cut at 16384
    descriptors, and halves at N = 16384; a launch takes whole runs only."""
    import struct

    def runs_of(i):
        """(descriptors, run length of the first `split`, split, run length of the rest) of launch i"""
        raw = ctypes.string_at(S.launch_arg0(i), 64)
        descs, _, _, _, group, split, tail, count = struct.unpack_from("<QQiiiiii", raw)
        k = 2 if b"k_ntt_half" in S.launch_name(i) else 1
        assert group % k == 0 and split % k == 0 and tail % k == 0 and count == S.launch_grid(i) // k * k
        d = ctypes.string_at(descs, count // k * 64)
        return [struct.unpack_from("<Q", d, 64 * j)[0] for j in range(count // k)], group // k, split // k, tail // k

    # uneven digits (2 + 2 + 1 primes; 3 + 2; 4 + 4 + 2), even ones, one prime each
    for log_n, n_q, n_sp, dnum, cts in ((12, 5, 2, 3, 9), (14, 5, 2, 3, 9), (12, 5, 1, 2, 3), (13, 10, 1, 3, 2), (12, 4, 2, 2, 5),
                                        (12, 3, 1, 3, 4), (12, 5, 2, 3, 1100)):
        n = 1 << log_n
        h = B.blb_ctx_create(log_n, n_q, n_sp, dnum, 0, None)
        K = B.blb_keygen(h, 1, [64])
        a = _buf(B, 2 * cts * 2 * n_q * n, 1)[1]
        for level in range(n_q) if cts < 100 else [n_q - 1]:
            x, y = [[B.blb_ct(a.ctypes.data + (o * cts + t) * 2 * n_q * n * 8, level, 1, 1.0) for t in range(cts)] for o in range(2)]
            S.clear()
            B.blb_rotate_sum(h, K, x, y, 64, 2, 0, False)
            seen = 0
            for i in range(S.launches()):
                if b"LdConv" not in S.launch_name(i):
                    continue
                seen += 1
                src, group, split, tail = runs_of(i)
                for lo, hi, run in ((0, split, group), (split, len(src), tail)):
                    assert (hi - lo) % run == 0
                    for r in range(lo, hi, run):
                        assert len(set(src[r:r + run])) == 1, (log_n, n_q, dnum, level, S.launch_name(i), r)
                runs = [src[r] for r in range(0, split, group)] + [src[r] for r in range(split, len(src), tail)]
                assert len(set(runs)) == len(runs)  # and a run is all of its source's descriptors
            assert seen >= 2
        B.blb_keys_destroy(K)
        B.blb_ctx_destroy(h)


def case_encode_waits_once(S, B):
    """blb_encode waits for the overflow flag with the residues enqueued before it, so that its caller's own
    wait has nothing left to wait for, and clears the flag without a launch of its own."""
    import numpy as np
    h = B.blb_ctx_create(12, 2, 1, 2, 0, None)
    v, pt = np.zeros(N // 2), np.zeros(2 * N, np.uint64)
    for _ in range(2):
        S.clear()
        B.blb_encode(h, v, 2.0 ** 30, 1, pt.ctypes.data)
        ev = S.events()
    kernels = [e for e in ev if e.startswith("launch")]
    assert len(kernels) == 3 and "k_coef_residues" in kernels[-1], ev
    assert ev[-2:] == ["copy", "wait stream"] and ev.count("wait stream") == 1, ev
    B.blb_ctx_destroy(h)


def case_kept_blocks_by_size(S, B):
    """Without a budget a plan takes a destroyed plan's block of its size or at most a quarter of its own size
    larger; other sizes get memory of their own, and the block waits for the next."""
    h = B.blb_ctx_create(12, 2, 1, 2, 0, None)
    for _ in range(3):  # (the temporaries grow to their size)
        B.blb_plan_destroy(_plan(B, h, 10)[0])
    first, size = _plan(B, h, 10)
    for blocks, taken in ((10, True), (9, True), (8, True), (7, False), (11, False)):
        held = S.live()
        B.blb_plan_destroy(first)
        assert S.live() == held
        plan, own = _plan(B, h, blocks)
        assert S.live() - held == (0 if taken else own), blocks
        B.blb_plan_destroy(plan)
        B.blb_ctx_trim(h)
        for _ in range(3):
            B.blb_plan_destroy(_plan(B, h, 10)[0])
        first, same = _plan(B, h, 10)
        assert same == size
    B.blb_plan_destroy(first)
    B.blb_ctx_destroy(h)
    assert S.live() == 0


def case_temporaries_give_way_to_what_is_kept(S, B):
    """Under a budget that holds a plan, an executor and the context's tables but not a stack of temporaries
    beside them, the plan and the executor are made, whatever calls came before."""
    mb = 1 << 20
    h = B.blb_ctx_create(12, 2, 1, 2, 0, None)
    base = B.blb_ctx_device_bytes(h)
    B.blb_ctx_destroy(h)
    h = B.blb_ctx_create(12, 2, 1, 2, 0, None, base + 148 * mb)
    K = B.blb_keygen(h, 1, [16 * i for i in range(1, 16)] + [256 * j for j in range(1, 8)])
    plan, _ = _plan(B, h, 1)
    for _ in range(3):
        B.blb_plan_destroy(plan)
        plan, _ = _plan(B, h, 1)
    x = [_buf(B, 4 * N, 1) for _ in range(2)]
    y, ya = _buf(B, 4 * N, 1)
    E = B.blb_exec_create_cp(h, K, plan, [c for c, _ in x], [y])
    for _ in range(2):
        B.blb_matmul_cp(h, K, plan, [c for c, _ in x], [y])
    plan2, _ = _plan(B, h, 1)
    assert B.blb_ctx_device_bytes(h) <= base + 148 * mb
    B.blb_exec_destroy(E)
    for p in (plan, plan2):
        B.blb_plan_destroy(p)
    B.blb_keys_destroy(K)
    B.blb_ctx_destroy(h)
    assert S.live() == 0


def case_tables_are_in_coherent_memory(S, B):
    """The ring's host side, which kernels read, is allocated mapped and coherent."""
    h = B.blb_ctx_create(12, 2, 1, 2, 0, None)
    mapped, coherent = 0x2, 0x40000000  # hipHostMallocMapped, hipHostMallocCoherent
    assert S.host_flags() & (mapped | coherent) == mapped | coherent
    B.blb_ctx_destroy(h)


def case_kept_memory_is_bounded_with_several_threads(S, B):
    """Threads that destroy plans at the same moment (their waits for the device return together) keep no more
    than 1/32 of the device's memory between them, every time."""
    import threading
    mb = 1 << 20
    n, cap = 8, 40 * mb  # two plans of 16 MiB
    S.total(32 * cap)
    hs = [B.blb_ctx_create(12, 2, 1, 2, 0, 0x1000 * (t + 1)) for t in range(n)]
    for h in hs:  # (the temporaries grow to their size)
        for _ in range(3):
            B.blb_plan_destroy(_plan(B, h, 1)[0])
    for _ in range(200):
        plans = [_plan(B, h, 1)[0] for h in hs]
        rest = S.live() - n * 16 * mb
        S.meet(n)
        threads = [threading.Thread(target=B.blb_plan_destroy, args=(p,)) for p in plans]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        S.meet(0)
        assert S.live() - rest <= cap, f"{(S.live() - rest) / mb:.0f} MiB kept"
    for h in hs:
        B.blb_ctx_destroy(h)
    assert S.live() == 0


# ---------------------------------------------------------------------------------------
CASES = [n[len("case_"):] for n in list(globals()) if n.startswith("case_")]


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "host", "hip_stub.cpp"), "-o", so], check=True)
    return so


@pytest.mark.parametrize("case", CASES)
def test_host_path(stub, case):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub, case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-3000:]


if __name__ == "__main__":
    S = Stub(sys.argv[1])
    import paper_2508_19525_amd as B
    globals()["case_" + sys.argv[2]](S, B)
