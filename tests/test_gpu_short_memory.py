"""Calls whose allocations fail: what has another layout to take takes it and
works, what has not returns an error, and either way neither the handle nor
the program's own HIP calls are left with it.

A child process loads a stand-in for hipMalloc (short_memory.c) that lets
chosen requests fail in the runtime itself."""

import os
import shutil
import subprocess
import sys

import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path[:0] = [sys.argv[2], sys.argv[3]]
import numpy as np
import torch
import spkgen, oracle
from paper_2011_00715_amd import spk
from gpu_util import mat_on_gpu, to_dev
from test_gpu_spmv import _scattered
hip = [l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64.so" in l][0]
shim.short_memory_real(ctypes.cast(ctypes.CDLL(hip).hipMalloc, ctypes.c_void_p))
torch.ones(1, device="cuda").add_(1)

def short(lo, hi=1 << 50, mask=1):
    shim.short_memory(ctypes.c_size_t(lo), ctypes.c_size_t(hi), mask)

def failed():
    left = shim.short_memory_left()
    shim.short_memory(ctypes.c_size_t(1), ctypes.c_size_t(0), 0)
    assert left == 0, "no request of this size was made"

def works(M, A, f32=False):
    torch.ones(1, device="cuda").add_(1)  # raises if an error was left behind
    x = np.random.default_rng(1).integers(-50, 50, A.n).astype(np.float64)
    ref = oracle.spmv(A, x)
    y = to_dev(np.full(A.n, np.nan))
    spk.mat_mult(M, to_dev(x), y)
    assert np.array_equal(y.cpu().numpy(), ref)
    if f32:
        y = to_dev(np.full(A.n, np.nan, np.float32))
        spk.mat_mult_f32(M, to_dev(x.astype(np.float32)), y)
        assert np.array_equal(y.cpu().numpy(), ref.astype(np.float32))
"""


@pytest.fixture(scope="module")
def child(tmp_path_factory):
    need_gpu()
    cc = shutil.which("gcc") or shutil.which("cc")
    if not cc:
        pytest.skip("no C compiler")
    so = str(tmp_path_factory.mktemp("shim") / "short_memory.so")
    subprocess.run([cc, "-shared", "-fPIC", "-O1", os.path.join(HERE, "short_memory.c"), "-o", so], check=True)

    def run(code):
        env = dict(os.environ, SPK_BINNED_ROWS="1")  # small matrices take the binned copy too
        r = subprocess.run([sys.executable, "-u", "-c", PRELUDE + code + "\nprint('done')", so, os.path.dirname(HERE),
                            HERE], capture_output=True, text=True, timeout=100, env=env)
        assert r.returncode == 0 and r.stdout.endswith("done\n"), r.stdout + r.stderr

    return run


def test_no_room_for_the_binned_copy(child):
    """The sliced family keeps to the slices, on request and by itself."""
    child("""
n = 40000
A = _scattered(n, [5] * (n - 1) + [3000], 7)
M = mat_on_gpu(spk, A)
short(20 * A.nnz)
spk.mat_set_kernel(M, spk.KERNEL_SLICED, 2048)
failed()
assert spk.KERNEL_NAMES[M.info.kernel] == "sliced" and M.info.lanes == 2048
works(M, A)
M.close()

n = 1 << 19
A = _scattered(n, [8] * (n - 1) + [4000], 3)
M = mat_on_gpu(spk, A)
assert spk.KERNEL_NAMES[M.info.kernel] == "sliced"
M.close()
short(20 * A.nnz)
M = mat_on_gpu(spk, A)
failed()
assert spk.KERNEL_NAMES[M.info.kernel] == "sliced"
works(M, A)
M.close()
""")


def test_an_error_is_not_left_behind(child):
    """A handle refused for want of memory leaves the program's own launches alone."""
    child("""
A = spkgen.laplace3d7(24)
csr = to_dev(A.rowptr), to_dev(A.col), to_dev(A.val)
M = mat_on_gpu(spk, A)
for lo, call in ((8 * A.nnz, lambda: spk.mat_create_csr(*csr)), (1, lambda: spk.server_create())):
    short(lo)
    try:
        call()
        raise SystemExit("created without memory")
    except spk.SpkError as e:
        assert e.status == spk.ENOMEM, e
    failed()
    works(M, A)
""")


def test_no_room_for_fp32_values(child):
    """A copy goes where its FP32 values do not fit: nothing is kept that no
    product uses."""
    child("""
n = 40000
A = _scattered(n, [5] * (n - 1) + [3000], 7)
M = mat_on_gpu(spk, A, flags=spk.MAT_MIXED)
before = M.info.device_bytes
short(4 * A.nnz, 4 * A.nnz + 8, mask=0b101)  # the binned FP32 values, not the slices' columns, their FP32 values
try:
    spk.mat_set_kernel(M, spk.KERNEL_SLICED, 2048)
    raise SystemExit("found room")
except spk.SpkError as e:
    assert e.status == spk.ENOMEM, e
failed()
spk.mat_set_kernel(M, spk.KERNEL_VECTOR, 8)
assert M.info.device_bytes == before
works(M, A, True)
spk.mat_set_kernel(M, spk.KERNEL_SLICED, 2048)
works(M, A, True)
""")


def test_no_room_for_two_copies(child):
    """From the binned copy to the slices: it makes room for them, and is there
    again where they do not fit even so."""
    child("""
n = 40000
A = _scattered(n, [5] * (n - 1) + [3000], 7)
M = mat_on_gpu(spk, A)
before = M.info.device_bytes
spk.mat_set_kernel(M, spk.KERNEL_SLICED, 2048)
binned = M.info.device_bytes
short(8 * A.nnz, mask=1)  # the slices' values, once
spk.mat_set_kernel(M, spk.KERNEL_SLICED, 4)
failed()
assert M.info.lanes == 4
works(M, A)
slices = M.info.device_bytes
assert slices == before + 12 * A.nnz + 4 * (8 * n + 1) + 8 * 8 * n
spk.mat_set_kernel(M, spk.KERNEL_SLICED, 2048)
assert M.info.device_bytes == binned
short(8 * A.nnz, mask=0b11)  # twice
try:
    spk.mat_set_kernel(M, spk.KERNEL_SLICED, 4)
    raise SystemExit("found room")
except spk.SpkError as e:
    assert e.status == spk.ENOMEM, e
failed()
assert M.info.lanes == 2048
works(M, A)
spk.mat_set_kernel(M, spk.KERNEL_SLICED, 2048)
assert M.info.device_bytes == binned
""")


def test_no_room_for_any_copy(child):
    """Without room for its layout a matrix takes a family that needs none, at
    creation and where a refused request took the layout down; the merge path
    does without half of its tiles."""
    child("""
n = 1 << 19
A = _scattered(n, [8] * (n - 1) + [40], 3)
csr = to_dev(A.rowptr), to_dev(A.col), to_dev(A.val)
short(8 * A.nnz, mask=0b1110)  # not the CSR arrays; the binned copy, the slices, SELL
M = spk.mat_create_csr(*csr)
failed()
assert spk.KERNEL_NAMES[M.info.kernel] in ("stream", "vector", "merge"), spk.KERNEL_NAMES[M.info.kernel]
works(M, A)
M.close()

n = 3000
A = _scattered(n, [3] * n, 4)
M = mat_on_gpu(spk, A)
spk.mat_set_kernel(M, spk.KERNEL_SELL, 16)
short(8 * A.nnz)  # the layout that would come back
try:
    spk.mat_set_kernel(M, spk.KERNEL_SELL, spk.SELL_SHARED)
    raise SystemExit("shared")
except spk.SpkError as e:
    assert e.status == spk.EINVAL, e
failed()
M.info = spk.mat_get_info(M)
assert spk.KERNEL_NAMES[M.info.kernel] in ("stream", "vector", "merge")
works(M, A)
spk.mat_set_kernel(M, spk.KERNEL_VECTOR, 4)
tiles = (A.n + A.nnz + 2047) // 2048
for mask in (1, 2, 4, 8):
    N = mat_on_gpu(spk, A)
    spk.mat_set_kernel(N, spk.KERNEL_VECTOR, 4)
    before = N.info.device_bytes
    short(4 * tiles, 8 * tiles, mask=mask)
    try:
        spk.mat_set_kernel(N, spk.KERNEL_MERGE, 0)
        raise SystemExit("found room")
    except spk.SpkError as e:
        assert e.status == spk.ENOMEM, e
    failed()
    N.info = spk.mat_get_info(N)
    assert spk.KERNEL_NAMES[N.info.kernel] == "vector" and N.info.device_bytes == before
    works(N, A)
    spk.mat_set_kernel(N, spk.KERNEL_MERGE, 0)
    works(N, A)
    N.close()
""")


@pytest.mark.parametrize("what", ["solve", "mixed", "single", "multi", "mg", "history"])
def test_no_room_for_a_workspace(child, what):
    """A solve that gets only some of its arrays is refused, and the next one
    has them all: each of the first requests fails once in its turn."""
    child(f"what = {what!r}" + """
A = spkgen.laplace3d7(24)
b = to_dev(spkgen.rhs_uniform(A.n, 0))
B = to_dev(np.stack([spkgen.rhs_uniform(A.n, s) for s in range(4)], 1))
X = torch.zeros_like(B) if what == "multi" else torch.zeros_like(b)

def solve(M, G, hist=None):
    X.zero_()
    if what == "multi":
        spk.ksp_solve_multi(M, B, X)
    elif what == "mg":
        spk.ksp_solve_mg(G, b, X, hist=hist)
    else:
        spk.ksp_solve(M, b, X, spk.ksp_opts(precision=spk.PREC_MIXED if what == "mixed" else spk.PREC_FP64,
                                            single_reduction=int(what == "single")), hist=hist)
    return X.clone()

def start():
    M = mat_on_gpu(spk, A)
    return M, spk.mg_create(M, (24, 24, 24)) if what == "mg" else None

M, G = start()
want = solve(M, G)
del M, G
refused = 0
for i in range(30):
    M, G = start()
    if what == "history":  # a longer one than the handle has
        solve(M, G, np.zeros(8))
    short(1, mask=1 << i)
    try:
        got = solve(M, G, np.zeros(64) if what == "history" else None)
        short(1, mask=0)
        assert torch.equal(got, want)
        break  # that many requests are not made
    except spk.SpkError as e:
        assert e.status == spk.ENOMEM, e
        refused += 1
    failed()
    for again in range(2):
        hist = np.full(8, np.nan)
        assert torch.equal(solve(M, G, hist if what in ("history", "mg") else None), want), (i, again)
        assert what not in ("history", "mg") or np.isfinite(hist[0])
    if G: G.close()
    M.close()
assert refused >= (1 if what in ("history", "mg") else 3) and i < 29
""")


def test_smoothing_in_one_pass_needs_no_memory(child):
    """Smoothing from zero that is a single pass over the matrix allocates
    nothing; more steps take the workspace."""
    child("""
A = spkgen.laplace3d7(24)
b = to_dev(spkgen.rhs_uniform(A.n, 0))
outs = []
for armed in (False, True):
    M = mat_on_gpu(spk, A)
    if not armed:
        spk.ksp_solve(M, b, torch.zeros_like(b))  # the workspace is there
    x, y, z, r = (torch.full_like(b, float("nan")) for _ in range(4))
    short(1, mask=int(armed))
    spk.pc_chebyshev(M, b, x, 1)
    spk.pc_chebyshev(M, b, y, 2)
    spk.pc_chebyshev(M, b, z, 1, r_out=r)
    assert shim.short_memory_left() == int(armed)
    if armed:
        try:
            spk.pc_chebyshev(M, b, z.clone(), 3)
            raise SystemExit("found room")
        except spk.SpkError as e:
            assert e.status == spk.ENOMEM, e
    failed()
    outs.append((x, y, z, r))
    M.close()
for got, want in zip(*outs):
    assert torch.equal(got, want) and torch.isfinite(got).all()
""")
