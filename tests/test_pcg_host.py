"""The host path of the PCG solves on a machine without a GPU: a stand-in for
the HIP runtime (hip_stub.cpp) counts graph launches, iterations and
synchronisations, and lets a solve converge after a set number of
iterations.  Each test runs in a process of its own, in which the stand-in
is loaded before the library."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, json, sys, types
sys.modules["torch"] = types.ModuleType("torch")   # its runtime is the stand-in
stub = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
stub.stub_set.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_char_p]
from paper_2609_04534_amd import tpfdm
class Vec:
    def __init__(self, n): self.a = (ctypes.c_double * n)()
    def data_ptr(self): return ctypes.addressof(self.a)
class Stream: cuda_stream = 0
def mesh(n, m):
    plan = tpfdm.Plan.mesh(n, (m, m, m), (1.0 / m,) * 3)
    plan.setup_inverse(tpfdm.OP_CELL)
    return plan, Vec(plan.vector_elems), Vec(plan.vector_elems), tpfdm.PCG(plan)
def counts():
    return [stub.stub_graph_launches(), stub.stub_iterations(), stub.stub_syncs()]
out = []
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("hip") / "hip_stub.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "hip_stub.cpp"), "-o", so], check=True)

    def run(body):
        r = subprocess.run([sys.executable, "-c", PRELUDE + body + "\nprint(json.dumps(out))", so],
                           cwd=os.path.dirname(HERE), capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout.splitlines()[-1])
    return run


def test_solve_done_at_its_start(stub):
    """A block-Jacobi solve that its start has finished launches no iterations,
    whatever check_every is, and neither preconditioner's does at maxit = 0."""
    out = stub("""
plan, b, x, cg = mesh(3, 4)
for k in (1, 16, 256):
    stub.stub_set(9, 1, b"")
    cg.solve(b, x, check_every=k, stream=Stream())
    out.append(counts()[:2])
mg = tpfdm.MG(plan)
for m in (None, mg):
    cg.set_multigrid(m)
    stub.stub_set(9, 0, b"")
    s = cg.solve(b, x, maxit=0, stream=Stream(), raise_on_failure=False)
    out.append(counts()[:2])
""")
    assert out == [[0, 0]] * 5


def test_vcycle_solve_reads_the_state_every_four_iterations(stub):
    """With a V-cycle the state is read after min(check_every, 4) iterations, for
    every check_every (9 iterations to convergence; one synchronisation per
    graph and one for the result), and a non-blocking solve enqueues exactly
    check_every iterations a step."""
    out = stub("""
plan, b, x, cg = mesh(3, 4)
mg = tpfdm.MG(plan)
cg.set_multigrid(mg)
for k in (1, 2, 3, 4, 5, 7, 13, 16, 17, 64):
    stub.stub_set(9, 0, b"")
    s = cg.solve(b, x, check_every=k, stream=Stream())
    blocking = counts() + [s["iterations"]]
    stub.stub_set(100, 0, b"")
    cg.begin(b, x, check_every=k, stream=Stream())
    steps = []
    while cg.poll() is None:
        steps.append(stub.stub_iterations())
    out.append([k, blocking, steps])
cg.destroy()
out.append(stub.stub_live_graphs())
""")
    assert out.pop() == 0
    for k, blocking, steps in out:
        g = min(k, 4)
        graphs = -(-9 // g)
        assert blocking == [graphs, graphs * g, graphs + 1, 9], k
        assert steps == [k * (i + 1) for i in range(-(-100 // k))] + [-(-100 // k) * k], k


@pytest.mark.parametrize("kernel", ["k_mg_restrict", "k_mg_smooth", "k_mg_tail", "k_pcg_aq", "k_pcg_axpy",
                                    "k_pcg_reduce_alpha", "k_pcg_dir"])
def test_failed_launch_in_an_iteration(stub, kernel):
    """A launch that fails while the iterations are captured fails the solve
    with that launch's error, leaves no graph without it, and the next solve
    captures anew."""
    out = stub("""
plan, b, x, cg = mesh(3, 8)
mg = tpfdm.MG(plan)
cg.set_multigrid(mg)
KERNEL = b"%s"
for begin in (False, True):
    stub.stub_set(9, 0, KERNEL)
    try:
        (cg.begin if begin else cg.solve)(b, x, stream=Stream())
        out.append("no error")
    except tpfdm.TpfdmError as e:
        out.append([e.status, stub.stub_graph_launches(), stub.stub_live_graphs()])
stub.stub_set(9, 0, b"")
out.append([cg.solve(b, x, stream=Stream())["iterations"], stub.stub_live_graphs()])
""" % kernel)
    assert out == [[-7, 0, 0], [-7, 0, 0], [9, 1]]


@pytest.mark.parametrize("n", [2, 3, 4])
def test_smoother_weight_stays_in_fp64(stub, n):
    """n <= 4: the table that the smoother's block inverse gets is D^{-1} itself
    (1 / (lam_i s_x + lam_j s_y + lam_k s_z) in the inner precision, here FP32);
    the Chebyshev weight is an FP64 argument of its own."""
    out = stub("""
N = %d
plan, b, x, cg = mesh(N, 8)
mg = tpfdm.MG(plan)
cg.set_multigrid(mg)
stub.stub_set(1, 0, b"")
E = (ctypes.c_float * (N ** 2 + N ** 3))()
w = ctypes.c_double()
for arg, dst in ((3, E), (4, w)):
    stub.stub_watch(b"k_mg_jacobi0", arg, ctypes.sizeof(dst))
    cg.solve(b, x, inner=tpfdm.F32, stream=Stream())
    stub.stub_watched(ctypes.byref(dst))
    cg.set_multigrid(mg)
S, lam = tpfdm.reference_eigen(N, 2.0, tpfdm.OP_CELL)
out = [list(E), w.value, S.reshape(-1).tolist(), lam.tolist()]
""" % n)
    import math

    import numpy as np
    E, w, S, lam = out
    lam = np.array(lam) / 8.0   # s_d = h on cubes of edge length 1/8
    d = 1.0 / (lam[:, None, None] + lam[None, :, None] + lam[None, None, :])
    assert np.allclose(E[:n * n], S, rtol=1.2e-7, atol=1e-7)
    assert np.allclose(E[n * n:], d.reshape(-1), rtol=1.2e-7, atol=0.0)
    assert abs(w - 1.0 / (1.1 - 0.9 * math.cos(math.pi / 6.0))) < 1e-14
