"""dfjk_build_static (the build that allocates nothing: its scratch is a
static device array of the library) against dfjk_build, through the C ABI.
Two calls in a row, the second with a smaller molecule, each compared with
the workspace build of the same input; then an int8 build and the density
route; a molecule too large for the 64 MiB array is refused before any work
is enqueued."""
import ctypes

import numpy as np
import pytest

import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2404_09452_amd import _native as N  # noqa: E402
from paper_2404_09452_amd import dfjk as G  # noqa: E402


def rel(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


def case(n):
    if n == 1:
        z, x = W.water_monomer()
    else:
        z, x = W.water_cluster(n, W.cluster_box(n), 100 + n)
    mol = W.make_molecule(z, x)
    S = W.overlap_by_quadrature(mol)
    C = W.occupied_orbitals(S, mol.nelec // 2, 7 + n)
    return mol, C


def _compare(plan, prec, **inp):
    ref = [t.cpu().numpy() for t in plan.build(precision=prec, **inp)]
    got = [t.cpu().numpy() for t in plan.build_static(precision=prec, **inp)]
    torch.cuda.synchronize()
    # the same arithmetic; only the aux slab (hence the split-K sum order) may differ
    tol = 1e-12 if prec == "fp64" else 1e-9
    assert rel(got[0], ref[0]) <= 1e-12
    assert rel(got[1], ref[1]) <= tol
    assert abs(got[2][0] - ref[2][0]) <= 1e-12 * abs(ref[2][0])
    assert abs(got[2][1] - ref[2][1]) <= tol * abs(ref[2][1])
    return got


def test_static_build_matches_workspace_build_twice_then_smaller():
    for n in (3, 1):                      # second call: a smaller molecule
        mol, C = case(n)
        plan = G.Plan.from_molecule(mol).screen().setup()
        _compare(plan, "fp64", C=C)
        plan.close()


def test_static_build_int8_and_density_route():
    mol, C = case(2)
    plan = G.Plan.from_molecule(mol).screen().setup()
    _compare(plan, "int8", C=C)
    D = 2.0 * C @ C.T
    _compare(plan, "fp64", D=D)
    plan.close()


@pytest.mark.parametrize("n,prec", [(3, "fp64"), (3, "int8_fast"), (10, "int8_fast")])
def test_static_build_after_autotuning(n, prec):
    """The autotuner's tile and splits in the static scratch (3 waters: one slab, as in the workspace
    build), and a size at which many tuned shapes no longer fit it while the built-in one does."""
    mol, C = case(n)
    plan = G.Plan.from_molecule(mol).screen().setup()
    plan.autotune(C, precision=prec)
    if n == 3:
        _compare(plan, prec, C=C)
    else:   # other slabs, so other scale blocks: the format's 1e-6 Eh
        E = plan.build_static(C=C, precision=prec)[2]
        ref = plan.build(C=C)[2]
        assert abs(float(E[1] - ref[1])) <= 1e-6
    plan.close()


def test_static_build_refuses_a_molecule_beyond_the_array():
    mol, C = case(12)
    plan = G.Plan.from_molecule(mol).screen().setup()
    dev = torch.device("cuda")
    Cd = torch.as_tensor(C, device=dev)
    J = torch.full((plan.nao, plan.nao), 7.0, dtype=torch.float64, device=dev)
    K = torch.full_like(J, 7.0)
    E = torch.full((2,), 7.0, dtype=torch.float64, device=dev)
    rc = N.lib().dfjk_build_static(plan._h, ctypes.c_void_p(Cd.data_ptr()), C.shape[1], None, 0,
                                   ctypes.c_void_p(J.data_ptr()), ctypes.c_void_p(K.data_ptr()),
                                   ctypes.c_void_p(E.data_ptr()), None)
    assert rc == 4                                            # DFJK_E_OOM
    assert b"static scratch" in N.lib().dfjk_last_error()
    torch.cuda.synchronize()
    assert bool((J == 7.0).all()) and bool((E == 7.0).all())  # outputs untouched
    plan.close()
