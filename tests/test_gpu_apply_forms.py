"""Block applies on both sides of the count at which FP64 blocks take the form for launches that fill
the chip, whole and by colours: against the stored inverse times r in float64, and a case stepped
alone (one form) and in a batch beyond the count (the other), bit for bit.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1903_06304_amd import inputs as I  # noqa: E402

pytestmark = pytest.mark.gpu


def _case(p, nx, ny, seed):
    from paper_1903_06304_amd import lmfr
    mesh = I.Mesh(nx, ny, p, (0.0, 2 * np.pi, 0.0, 2 * np.pi))
    prm = I.Params(order=p, n_elem=mesh.E, mach_ref=0.3, reynolds=100.0, viscous=True, kappa=1.0)
    g = lmfr.Context(prm, *mesh.connectivity())
    g.set_geometry(*mesh.nodes(0.0))
    q = I.uniform_flow(mesh, prm)
    q += 0.02 * np.random.default_rng(seed).uniform(-1.0, 1.0, q.shape)
    return mesh, g, torch.tensor(q, device="cuda")


@pytest.mark.parametrize("p", [1, 2, 3, 4])
@pytest.mark.parametrize("nx,ny", [(1, 1), (89, 23), (64, 32), (683, 3), (96, 45)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_apply_is_the_stored_inverse(p, nx, ny, prec):
    mesh, g, q = _case(p, nx, ny, 3)
    E, nb = mesh.E, 4 * mesh.Np
    g.block_jacobi_factor(q, 20.0, 3.0, prec)
    X = g.get_inverse()
    r = torch.tensor(np.random.default_rng(4).standard_normal(q.shape), device="cuda")
    rE = r.permute(1, 0, 2).reshape(E, 1, nb)
    z = g.block_jacobi_apply(r).permute(1, 0, 2).reshape(E, nb)
    # two sums of nb products in different orders, each off by at most nb u |X| |r|
    bar = 2 * nb * 2.0 ** -53 * (X.abs() * rE.abs()).sum(2)
    assert bool(((z - (X * rE).sum(2)).abs() <= bar).all())


@pytest.mark.parametrize("p,nx,ny", [(3, 46, 45), (3, 64, 66), (4, 46, 45), (4, 64, 66)])
@pytest.mark.parametrize("precond", [0, 2])
def test_alone_and_in_a_batch(p, nx, ny, precond):
    from paper_1903_06304_amd import lmfr
    _, g, q = _case(p, 6, 4, 1)
    _, g2, q2 = _case(p, nx, ny, 2)
    kw = dict(tol_pseudo=1e-8, tol_res=1e-6, krylov=20, max_lin_it=20, max_newton=1, jac_lag=2, prec="fp64")
    g.set_option("preconditioner", precond)
    alone = q.clone()
    g.bdf2_step(alone, None, 0.01, **kw)
    assert not torch.equal(alone, q) and torch.isfinite(alone).all()
    batch = lmfr.Batch([g, g2])
    batch.set_option("preconditioner", precond)
    x, y = q.clone(), q2.clone()
    batch.bdf2_step([x, y], None, [lmfr.step_opts(0.01, **kw)] * 2)
    assert torch.equal(x, alone)
