"""Reads past the last-level cache: the block apply and the Gram-Schmidt kernels take loads that leave
no line there once blocks and basis exceed it.

* The block apply with the blocks alone (within the cache) and after a reserve whose basis takes both
  past it: bit for bit the same, and D z = r to rounding for one of them.
* A linear solve whose basis passes the cache inside the cycle: it meets its tolerance in the operator
  (twice, for the rounding of dq = q1 - q and of the two operator forms), and the fused and separate
  re-orthogonalisations, which share no launch, agree bit for bit.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1903_06304_amd import inputs as I  # noqa: E402

pytestmark = pytest.mark.gpu

LLC = 256 << 20


def _problem(nx, ny, p):
    from paper_1903_06304_amd import lmfr
    mesh = I.Mesh(nx, ny, p, (0.0, 2 * np.pi, 0.0, 2 * np.pi))
    prm = I.Params(order=p, n_elem=mesh.E, mach_ref=0.2, reynolds=100.0, viscous=True, kappa=1.0)
    rng = np.random.default_rng(11)
    q = I.uniform_flow(mesh, prm)
    du, dv = I.random_solenoidal_velocity(mesh, rng, rms=0.2, kmax=2)
    q[1] += du
    q[2] += dv
    g = lmfr.Context(prm, *mesh.connectivity())
    g.set_geometry(*mesh.nodes(0.0))
    return mesh, g, torch.tensor(q, device="cuda")


@pytest.mark.parametrize("prec,size", [("fp64", 8), ("fp32", 4), ("bf16", 2)])
@pytest.mark.parametrize("p,nx,ny", [(1, 121, 119), (2, 81, 79), (3, 61, 59), (4, 51, 49)])
def test_streamed_blocks_are_bitwise(p, nx, ny, prec, size):
    mesh, g, q = _problem(nx, ny, p)
    E, nb = mesh.E, 4 * mesh.Np
    assert E * nb * nb * size <= LLC < E * nb * nb * size + 157 * E * nb * 8
    r = torch.tensor(np.random.default_rng(3).standard_normal((4, E, mesh.Np)), device="cuda")
    g.set_option("keep_blocks", 1)
    g.block_jacobi_factor(q, 20.0, 3.0, prec)
    z = g.block_jacobi_apply(r).clone()
    if prec == "fp64":
        # |D z - r| <= nb u cond(D) |r| with cond(D) below 1e3 at these coefficients
        D = g.get_blocks().contiguous()
        res = torch.bmm(D, z.permute(1, 0, 2).reshape(E, nb, 1).contiguous()).reshape(E, nb)
        assert float((res - r.permute(1, 0, 2).reshape(E, nb)).norm()) <= nb * 1.2e-16 * 1e3 * float(r.norm())
    g.reserve(156, prec)
    g.block_jacobi_factor(q, 20.0, 3.0, prec)
    assert torch.equal(z, g.block_jacobi_apply(r))


def test_streamed_basis():
    out = []
    for fused in (0, 1):
        mesh, g, q = _problem(130, 128, 3)
        g.set_option("gram_schmidt", 2)
        g.set_option("fused_gram_schmidt", fused)
        dtau, tol = 0.2, 1e-6
        q1 = q.clone()
        st = g.steady_solve(q1, dtau0=dtau, dtau_min=1e-3, tol_pseudo=1e-30, tol_res=tol, krylov=70, max_lin_it=900,
                            max_steps=1)
        # 32 vectors and more pass the cache
        assert 32 * q.numel() * 8 > LLC and 32 < st["gmres_its"] < 900
        dq = q1 - q
        R = g.residual(q)
        rel = float((R - g.bdf_operator(q, dq, 0.0, 1.0 / dtau)).norm() / R.norm())
        print(f"[streamed] fused={fused}: {st['gmres_its']} its, {rel:.2e}", flush=True)
        assert rel <= 2 * tol
        out.append(q1)
    assert torch.equal(out[0], out[1])
