"""Builds of one plan on several streams and threads at once, where J runs on the plan's side stream (B of
64 MB and more): each call has its own scratch and outputs, and every result is bitwise that of the call alone."""
import ctypes
import threading

import pytest

import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2404_09452_amd import _native as N  # noqa: E402
from paper_2404_09452_amd import dfjk as G  # noqa: E402


class Call:
    """dfjk_build or dfjk_build_uks of one plan with its own orbitals, scratch, outputs and stream."""

    def __init__(self, plan, kind, C):
        self.plan, self.kind, self.C = plan, kind, torch.as_tensor(C, device="cuda").contiguous()
        self.stream = torch.cuda.Stream()
        self.nocc, n = C.shape[1], ctypes.c_size_t()
        if kind == "uks":
            G._check(N.lib().dfjk_build_uks_bytes(plan._h, self.nocc, self.nocc - 2, 0, ctypes.byref(n)))
            self.Cb = self.C[:, 2:].contiguous()
        else:
            G._check(N.lib().dfjk_build_bytes(plan._h, self.nocc, 0, 0, ctypes.byref(n)))
        self.scratch = torch.empty(n.value, dtype=torch.uint8, device="cuda")
        m = 3 if kind == "uks" else 2
        self.out = [torch.zeros(plan.nao, plan.nao, dtype=torch.float64, device="cuda") for _ in range(m)]
        self.out.append(torch.zeros(2, dtype=torch.float64, device="cuda"))

    def run(self):
        p = [ctypes.c_void_p(t.data_ptr()) for t in self.out]
        end = (ctypes.c_void_p(self.scratch.data_ptr()), self.scratch.numel(), ctypes.c_void_p(self.stream.cuda_stream))
        C = ctypes.c_void_p(self.C.data_ptr())
        if self.kind == "uks":
            Cb = ctypes.c_void_p(self.Cb.data_ptr())
            G._check(N.lib().dfjk_build_uks(self.plan._h, C, self.nocc, Cb, self.nocc - 2, 0, *p, *end))
        else:
            G._check(N.lib().dfjk_build(self.plan._h, C, self.nocc, None, 0, *p, *end))

    def result(self):
        self.stream.synchronize()
        return [t.clone() for t in self.out]


@pytest.fixture(scope="module")
def calls():
    z, x = W.water_cluster(9, W.cluster_box(9), 109)
    mol = W.make_molecule(z, x)
    S = W.overlap_by_quadrature(mol)
    plan = G.Plan.from_molecule(mol).screen().setup()
    assert plan.info()["nf"] * plan.info()["naux_pad"] * 8 >= 64e6
    out = [Call(plan, kind, W.occupied_orbitals(S, mol.nelec // 2, 40 + i))
           for i, kind in enumerate(("uks", "build", "uks", "build"))]
    torch.cuda.synchronize()
    alone = []
    for c in out:
        c.run()
        alone.append(c.result())
    yield out, alone
    plan.close()


def same(a, b):
    torch.cuda.synchronize()
    return all(torch.equal(x, y) for x, y in zip(a, b))


def test_threads_share_a_plan(calls):
    """Four threads, each repeating its build on its own stream."""
    out, alone = calls
    ok = [True] * len(out)

    def work(i):
        for _ in range(25):
            out[i].run()
            ok[i] &= same(out[i].result(), alone[i])
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(out))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(ok), ok


@pytest.mark.parametrize("captured", [0, 1])
def test_builds_beside_a_capture(calls, captured):
    """Builds on other streams while a build (twice in the graph) is being captured, then replays of the
    graph between eager builds."""
    out, alone = calls
    g = torch.cuda.CUDAGraph()
    c = out[captured]
    with torch.cuda.graph(g, stream=c.stream, capture_error_mode="relaxed"):
        c.run()
        for other in (2, 3):
            out[other].run()
        c.run()
        for other in (2, 3):
            out[other].run()
    for other in (2, 3):
        assert same(out[other].result(), alone[other])
    for _ in range(3):
        for t in c.out:
            t.zero_()
        g.replay()
        for other in (2, 3):
            out[other].run()
        assert same(c.out, alone[captured])
        for other in (2, 3):
            assert same(out[other].result(), alone[other])
        c.run()
        assert same(c.result(), alone[captured])
