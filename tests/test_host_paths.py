"""Host paths of libpr.so that a healthy GPU rarely takes, over a stand-in for
the HIP host runtime (hip_standin.c: kernels do nothing, failures are forced).
Each body runs in a process of its own with the stand-in preloaded.  No GPU."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, sys
import numpy as np
sys.path.insert(0, {root!r})
import paper_2603_01306_amd._binding as b
P = ctypes.c_void_p
si = ctypes.CDLL({so!r})
si.si_log.restype = ctypes.c_char_p
si.si_lose.argtypes = [ctypes.c_char_p]
si.si_fail_above.argtypes = [ctypes.c_size_t]
si.si_cost.argtypes = [ctypes.c_char_p, ctypes.c_double]
lib = b.load()
keep = []

def mem(x):
    a = np.ascontiguousarray(x)
    keep.append(a)
    return P(a.ctypes.data)

def zeros(*shape):
    return mem(np.zeros(shape))

def context(n, p, loss=0, max_batch=1):
    prob = b.PrProblem(X=mem(np.zeros((p, n), np.float32)).value, xdtype=b.F32, loss=loss, y=zeros(n).value, n=n, p=p)
    h = P()
    assert lib.pr_ctx_create(ctypes.byref(h), ctypes.byref(prob), max_batch, None) == 0
    return h

def nodes(m):
    return (b.PrNode * m)(*[b.PrNode(k=3, lambda2=0.5, M=2.0) for _ in range(m)])

def log():
    return [ln.split() for ln in si.si_log().decode().splitlines()]

def opts(**kw):
    o = b.PrOpts()
    lib.pr_opts_default(ctypes.byref(o))
    o.L = 1.0
    for k, v in kw.items():
        setattr(o, k, v)
    return ctypes.byref(o)

res = b.PrResult()
OK, EDEVICE, ENOMEM = 0, -3, -4
"""


@pytest.fixture(scope="session")
def standin(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("standin") / "hip_standin.so")
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_standin.c")
    subprocess.check_call(["gcc", "-std=gnu11", "-O1", "-Wall", "-shared", "-fPIC", "-o", so, src])
    return so


def run(so, body):
    env = dict(os.environ, LD_PRELOAD=":".join(filter(None, (so, os.environ.get("LD_PRELOAD")))))
    code = PRELUDE.format(root=ROOT, so=so) + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("p", [5000, 17000])
def test_lost_exchange_fails_the_dual_bound(standin, p):
    """A regulariser kernel whose workgroups lost each other leaves no bound."""
    run(standin, f"""
    p = {p}
    h, lb, ub = context(8, p), ctypes.c_double(7.0), ctypes.c_double(7.0)
    call = lambda: lib.pr_dual_bound(h, nodes(1), None, zeros(p), ctypes.byref(lb), ctypes.byref(ub))
    assert call() == OK and lb.value != 7.0
    lb.value = ub.value = 7.0
    si.si_lose(b"k_regularizer_x")
    assert call() == EDEVICE and lb.value == ub.value == 7.0
    si.si_lose(b"")
    assert call() == OK
    """)


@pytest.mark.parametrize("kernel", ["k_regularizer_x", "k_prox_x"])
def test_lost_exchange_fails_the_warm_start(standin, kernel):
    """... and no judged starting point, also where only the candidate's prox
    was lost."""
    run(standin, f"""
    p = 5000
    h, B0 = context(8, p), zeros(2, p)
    call = lambda: lib.pr_mlp_warm_start(h, nodes(2), 2, None, zeros(2, p), B0, None, None)
    assert call() == OK
    si.si_lose({kernel.encode()!r})
    assert call() == EDEVICE
    si.si_lose(b"")
    assert call() == OK
    """)


def test_lost_exchange_fails_the_gram_certificate(standin):
    run(standin, """
    h = context(32, 4224)
    assert lib.pr_ctx_enable_gram(h) == OK
    z = np.full(32, 7.0)
    call = lambda: lib.pr_solve(h, nodes(1), opts(max_iter=0), None, None, P(z.ctypes.data), ctypes.byref(res))
    si.si_lose(b"k_regularizer_x")
    assert call() == EDEVICE and np.all(z == 7.0)
    si.si_lose(b"")
    assert call() == OK and np.all(z == 0.0)
    """)


@pytest.mark.parametrize("kernel", ["k_node_init_x", "k_node_step_x"])
def test_lost_exchange_fails_the_solve(standin, kernel):
    """... whatever the first workgroup wrote into the node's state."""
    run(standin, f"""
    p = 17000
    h, x = context(8, p), np.full(p, 7.0)
    call = lambda: lib.pr_solve(h, nodes(1), opts(max_iter=3), None, P(x.ctypes.data), None, ctypes.byref(res))
    si.si_lose({kernel.encode()!r})
    assert call() == EDEVICE and np.all(x == 7.0)
    si.si_lose(b"")
    assert call() == OK and np.all(x == 0.0)
    """)


@pytest.mark.parametrize("p", [5000, 17000, 524288])
def test_lost_exchange_fails_the_calls_without_a_context(standin, p):
    """Any workgroup's loss counts, in every call and only in its own."""
    run(standin, f"""
    p = {p}
    v, st, x = zeros(p), mem(np.zeros(p, np.int8)), zeros(p)
    d = ctypes.c_double
    ref, t0, t1, g, gs = ctypes.byref, d(), d(), d(), d()
    calls = [(b"k_prox_x", lambda: lib.pr_prox(None, v, p, d(0.5), 3, d(2.0), st, x)),
             (b"k_prox_x", lambda: lib.pr_prox_noalloc(None, v, p, d(0.5), 3, d(2.0), st, x)),
             (b"k_prox_x", lambda: lib.pr_time_prox(None, v, p, d(0.5), 3, d(2.0), st, x, 2, ref(t0), ref(t1))),
             (b"k_regularizer_x", lambda: lib.pr_regularizer(None, v, v, p, 3, d(2.0), st, ref(g), ref(gs)))]
    for kernel, call in calls:
        for _ in range(2):
            assert call() == OK
            g.value = gs.value = 7.0
            si.si_lose(kernel)
            assert call() == EDEVICE and g.value == gs.value == 7.0
            si.si_lose(b"")
    """)


@pytest.mark.parametrize("cus", [256, 128, 32, 20, 4, 1])
def test_shared_vectors_fit_the_compute_units(standin, cus):
    """Workgroups that wait for one another number at most a quarter of the
    compute units the stream may use, cover the vector, and keep the shapes of
    the whole device where that is available; other vectors go through one
    workgroup."""
    run(standin, f"""
    cus = {cus}
    si.si_cus(cus)
    d = ctypes.c_double
    full = {{16385: (9, 4), 65536: (32, 4), 131072: (64, 4), 131073: (33, 8), 262145: (33, 16), 524288: (64, 16)}}
    for p in (1, 4096, 4097, 16384, *full, 524289):
        v, st, x, g = zeros(p), mem(np.zeros(p, np.int8)), zeros(p), d()
        h = context(8, p)
        si.si_clear()
        assert lib.pr_solve(h, nodes(1), opts(max_iter=3), None, None, None, ctypes.byref(res)) == OK
        assert lib.pr_dual_bound(h, nodes(1), None, v, ctypes.byref(g), ctypes.byref(g)) == OK
        assert lib.pr_prox(None, v, p, d(0.5), 3, d(2.0), st, x) == OK
        noalloc = lib.pr_prox_noalloc(None, v, p, d(0.5), 3, d(2.0), st, x)
        assert lib.pr_regularizer(None, v, None, p, 3, d(2.0), st, ctypes.byref(g), None) == OK
        shared = [(k, int(w)) for k, w, _ in log() if any(s in k for s in ("k_prox_x", "k_regularizer_x",
                                                                           "k_node_init_x", "k_node_step_x"))]
        one = [k for k, _, _ in log() if any(s in k for s in ("k_proxE", "k_prox_counted", "k_regularizerE"))]
        for k, w in shared:
            e = int(k.split("ILi")[1].split("E")[0])
            assert w == 1 or 4 * w <= cus, (p, k, w)
            assert w * e * 512 >= p > (w - 1) * e * 512, (p, k, w)
            if cus == 256 and p in full:
                assert (w, e) == full[p], (p, k, w)
        fits = p <= 4096 or any(-(-p // (512 * e)) <= max(1, cus // 4) for e in (4, 8, 16))
        assert bool(shared) == fits, (p, shared)
        assert bool(one) == (not fits), (p, one)
        lib.pr_ctx_destroy(h)
        del keep[:]
    """)


@pytest.mark.parametrize("stream", [1, 2])
def test_default_streams_by_handle(standin, stream):
    """hipStreamLegacy and hipStreamPerThread are streams like others."""
    run(standin, f"""
    s, p, d = P({stream}), 20000, ctypes.c_double
    v, st, x, g = zeros(p), mem(np.zeros(p, np.int8)), zeros(p), d()
    assert lib.pr_prox(s, v, p, d(0.5), 3, d(2.0), st, x) == OK
    assert lib.pr_prox_noalloc(s, v, p, d(0.5), 3, d(2.0), st, x) == OK
    assert lib.pr_regularizer(s, v, None, p, 3, d(2.0), st, ctypes.byref(g), None) == OK
    prob = b.PrProblem(X=mem(np.zeros((p, 8), np.float32)).value, xdtype=b.F32, loss=0, y=zeros(8).value, n=8, p=p)
    assert lib.pr_ctx_create(ctypes.byref(P()), ctypes.byref(prob), 1, s) == OK
    assert all(int(w) > 1 for k, w, _ in log() if "k_prox_x" in k or "k_regularizer_x" in k)
    """)


def test_wait_clock_counts_polling_time(tmp_path):
    """20 s of the limit are 20 s of looks a millisecond apart; an hour in which
    the wave did not run adds 10 ms."""
    src = tmp_path / "wait.cpp"
    src.write_text(r"""
#include "pr_wait.h"
int main() {
  const long long ms = 100000, limit = 20000 * ms;
  pr::WaitClock a, b;
  long long now = 5 * ms;
  int looks = 0;
  while (!a.expired(now, limit)) now += ms, looks++;
  if (looks != 20001) return 1;
  now = 7;
  for (int i = 0; i < 100; i++, now += ms)
    if (b.expired(now, limit)) return 2;
  now += 3600ll * 1000 * ms;
  if (b.expired(now, limit)) return 3;
  for (int i = 0; i < 1000; i++)
    if (b.expired(now += 3600ll * 1000 * ms, limit)) return 4;
  return b.spent == 99 * ms + 1001 * pr::kWaitStep ? 0 : 5;
}
""")
    exe = tmp_path / "wait"
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2603_01306_amd", "csrc"),
                           str(src), "-o", str(exe)])
    assert subprocess.run([str(exe)]).returncode == 0


@pytest.mark.parametrize("max_batch", [8, 256])
@pytest.mark.parametrize("loss", [0, 1])
def test_route_of_the_feature_images(standin, max_batch, loss):
    """One node goes through the batch's GEMMs only where two passes over X cost
    more than those, as timed for the context; two or more always."""
    run(standin, f"""
    for gemm, together in ((10.0, False), (100.0, False), (2.0, True)):
        si.si_cost(b"k_gemv", 6.0)
        si.si_cost(b"k_spfwd", 0.0)
        si.si_cost(b"k_gemm", gemm)
        h, F = context(128, 1024, loss={loss}, max_batch={max_batch}), mem(np.zeros((3, 1024, 8), np.uint16))
        for m in (1, 2, 3):
            si.si_clear()
            assert lib.pr_mlp_features(h, nodes(m), m, zeros(m, 1024), None, F, None) == OK
            assert any("k_gemm" in ln[0] for ln in log()) == (together or m > 1), (gemm, m)
        lib.pr_ctx_destroy(h)
    """)


@pytest.mark.parametrize("us,split", [(200.0, 32), (20.0, 32), (5.0, 16)])
def test_split_of_equal_times(standin, us, split):
    """Candidates whose cost differs by less than timing noise: always the larger
    split, so that a repeated run repeats its sums; not where its planes cost more."""
    run(standin, f"""
    si.si_cost(b"k_gemm", {us})
    h = context(1024, 512, max_batch=16)
    f, t = (ctypes.c_int32 * 1)(), (ctypes.c_int32 * 1)()
    assert lib.pr_batch_tuning(h, 1, f, t) == OK
    assert list(t) == [{split}], list(t)
    """)


def test_one_nodes_features_take_one_upload(standin):
    """The status of the node; its scalars go with the launch."""
    run(standin, """
    h, F = context(8, 300), mem(np.zeros((3, 300, 8), np.uint16))
    for m in (1, 3):
        si.si_clear()
        assert lib.pr_mlp_features(h, nodes(m), m, zeros(m, 300), None, F, None) == OK
        assert si.si_copies() == m
    """)


@pytest.mark.parametrize("p,ops", [(300, 7), (4096, 7), (4097, 8)])
def test_operations_of_a_one_node_feature_call(standin, p, ops):
    """Upload and launches together: seven, as many as the runtime waits for
    without a detour; longer vectors have their ranks counted in a launch."""
    run(standin, f"""
    h, F = context(8, {p}), mem(np.zeros((1, {p}, 8), np.uint16))
    si.si_clear()
    assert lib.pr_mlp_features(h, nodes(1), 1, zeros(1, {p}), None, F, None) == OK
    assert si.si_copies() + len(log()) == {ops}
    """)


def test_features_of_more_nodes_than_a_launch_takes(standin):
    run(standin, """
    m, p = 65600, 128
    h, F = context(128, p, max_batch=m), mem(np.zeros((m, p, 8), np.uint16))
    si.si_clear()
    assert lib.pr_mlp_features(h, nodes(m), m, zeros(m, p), None, F, None) == OK
    rows = [int(y) for k, _, y in log() if "k_feat_rows" in k]
    assert sum(rows) == m and max(int(y) for _, _, y in log()) <= 65535
    params = mem(np.zeros(b.MLP_NPARAM, np.float32))
    si.si_clear()
    lib.pr_mlp_warm_start(h, nodes(m), m, params, zeros(m, p), zeros(m, p), None, None)
    assert sum(int(y) for k, _, y in log() if "k_feat_rows" in k) == m
    """)


def test_features_without_room_for_a_batch(standin):
    """No room for a batch's scratch: the nodes go one by one, as they do on a
    context without the batched path."""
    run(standin, """
    h, F = context(128, 1024, max_batch=256), mem(np.zeros((3, 1024, 8), np.uint16))
    si.si_fail_above(1 << 20)
    for _ in range(2):
        si.si_clear()
        assert lib.pr_mlp_features(h, nodes(3), 3, zeros(3, 1024), None, F, None) == OK
        assert si.si_nulls() == 0 and not any("k_gemm" in ln[0] for ln in log())
        assert sum("k_feat_rows" in ln[0] for ln in log()) == 3
    """)


@pytest.mark.parametrize("max_batch", [1, 64])
@pytest.mark.parametrize("limit", [4000, 10000, 20000, 50000, 300000, 600000])
def test_first_use_allocations_that_fail_once(standin, max_batch, limit):
    """A call that could not get all its buffers says so each time, and the
    next one that can gets them all."""
    run(standin, f"""
    h, F, params = context(128, 1024, max_batch={max_batch}), mem(np.zeros((3, 1024, 8), np.uint16)), zeros(4801)
    feat = lambda: lib.pr_mlp_features(h, nodes(3), 3, zeros(3, 1024), None, F, None)
    warm = lambda: lib.pr_mlp_warm_start(h, nodes(3), 3, params, zeros(3, 1024), zeros(3, 1024), None, None)
    for call in (feat, warm, feat):
        si.si_fail_above({limit})
        first = call()
        assert first in (OK, ENOMEM) and call() == first
        si.si_fail_above(0)
        assert call() == OK and si.si_nulls() == 0
        h = context(128, 1024, max_batch={max_batch})
    """)


@pytest.mark.parametrize("dtype,n,p,one,two", [
    # few row steps, enough waves without LDS
    ("F32", 256, 16385, 0, 512), ("F32", 256, 10240, 0, 512), ("F32", 256, 8192, 0, 0), ("F32", 256, 8193, 0, 512),
    ("F32", 1020, 20480, 0, 512), ("F32", 1020, 20481, 427, 512),
    ("F32", 512, 14000, 438, 512), ("F32", 508, 14000, 0, 512), ("F64", 256, 16384, 512, 512),
    ("F64", 512, 20480, 0, 427),
    # four row steps: whole rounds, of two only if they fill the grid
    ("F32", 1024, 16385, 342, 342), ("F32", 1024, 8192, 0, 512), ("F32", 1024, 8193, 0, 0),
    ("F32", 1024, 10241, 321, 321),
    ("F32", 2300, 89989, 512, 512), ("F32", 5088, 4097, 0, 257), ("F32", 5092, 4097, 0, 0),
    ("F64", 1024, 14000, 438, 438), ("F64", 1024, 18000, 0, 375), ("F64", 512, 65536, 512, 512),
    # BF16 with two: every workgroup that is resident
    ("BF16", 5088, 16385, 342, 512), ("BF16", 2040, 8192, 0, 0), ("BF16", 2048, 8192, 0, 512),
    ("BF16", 10176, 10241, 321, 0),
    # columns 32 KiB apart, 16 with C = 4, 4 with many of them
    ("F32", 8192, 16384, 0, 0), ("F32", 8192, 60000, 0, 0), ("F32", 8064, 12000, 0, 0), ("F32", 8060, 12000, 375, 0),
    ("F64", 4096, 40000, 0, 0), ("F64", 4094, 40000, 500, 500), ("F64", 6144, 40000, 500, 0),
    ("F32", 4096, 20480, 0, 427), ("F32", 4096, 20481, 427, 427), ("F32", 4096, 8192, 0, 0),
    ("F32", 4092, 8192, 0, 512), ("BF16", 8192, 20480, 0, 0), ("BF16", 8192, 20481, 427, 0),
    ("F32", 1024, 65535, 512, 512), ("F32", 1024, 65536, 512, 0), ("BF16", 2048, 65536, 512, 512),
])
def test_kernel_of_the_transposed_product(standin, dtype, n, p, one, two):
    """Workgroups of the kernel with its right-hand sides in LDS, 0: the other."""
    run(standin, f"""
    n, p = {n}, {p}
    np_t = dict(F32=np.float32, F64=np.float64, BF16=np.uint16)[{dtype!r}]
    prob = b.PrProblem(X=mem(np.zeros((p, n), np_t)).value, xdtype=b.{dtype}, loss=0, y=zeros(n).value, n=n, p=p)
    h = P()
    assert lib.pr_ctx_create(ctypes.byref(h), ctypes.byref(prob), 1, None) == OK
    for call, want in ((lambda: lib.pr_gemv_t(h, zeros(n), zeros(p)), {one}),
                       (lambda: lib.pr_gemv_t2(h, zeros(n), zeros(n), zeros(p), zeros(p)), {two})):
        si.si_clear()
        assert call() == OK
        (name, grid, _), = log()
        assert (int(grid) if "k_gemv_l" in name else 0) == want, (name, grid)
    """)
