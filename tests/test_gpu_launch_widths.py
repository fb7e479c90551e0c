"""Default workgroup widths: element counts on both sides of every line of the rule (workgroups on
the fullest compute unit), residual and derivatives bit for bit those of each explicit width.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1903_06304_amd import inputs as I  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("viscous", [True, False])
@pytest.mark.parametrize("kind", ["affine", "curved", "moving"])
@pytest.mark.parametrize("p,nx,ny", [(1, 107, 103), (2, 80, 80), (2, 80, 81), (2, 127, 100), (3, 64, 80), (3, 65, 80), (3, 64, 97),
                                     (3, 64, 128), (3, 97, 100), (3, 103, 100), (4, 8, 127), (4, 35, 40), (4, 50, 60), (4, 64, 64), (4, 64, 65)])
def test_default_width_is_bitwise(p, nx, ny, kind, viscous):
    from paper_1903_06304_amd import lmfr
    moving = kind == "moving"
    mesh = I.Mesh(nx, ny, p, (0.0, 2.0, 0.0, 2.0),
                  I.map_deforming(0.05) if moving else I.map_curved(0.05) if kind == "curved" else I.map_affine, moving=moving)
    prm = I.Params(order=p, n_elem=mesh.E, mach_ref=0.3, reynolds=30.0, viscous=viscous, moving=moving, kappa=1.0)
    g = lmfr.Context(prm, *mesh.connectivity())
    g.set_geometry(*mesh.nodes(0.07 if moving else 0.0))
    rng = np.random.default_rng(p * nx + ny)
    q = 1.0 + 0.1 * rng.standard_normal((4, mesh.E, mesh.Np))
    q[0] *= prm.gas_constant
    q, v = torch.tensor(q, device="cuda"), torch.tensor(rng.standard_normal(q.shape), device="cuda")

    def run():
        return (g.residual(q), g.jvp(q, v), *g.jvp(q, v, want_residual=True), g.bdf_operator(q, v, 20.0, 3.0))

    ref = run()
    for lanes in (64, 128):
        g.set_option("tile_lanes", lanes)
        for a, b in zip(ref, run()):
            assert torch.isfinite(a).all() and torch.equal(a, b), lanes
