"""Default launch shapes against one workgroup per tile, bit for bit: tile counts below, at and just
above the workgroups the device holds (where the default turns to workgroups that stay) and with a
ragged last round, for the residual, J v and the Newton operator through its packs.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1903_06304_amd import inputs as I  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["affine", "curved", "moving"])
@pytest.mark.parametrize("p,nx,ny", [(1, 91, 89), (2, 67, 61), (2, 72, 71), (3, 64, 64), (3, 65, 64), (3, 91, 90), (4, 51, 50),
                                     (4, 64, 80)])
def test_default_shape_is_bitwise(kind, p, nx, ny):
    from paper_1903_06304_amd import lmfr
    moving = kind == "moving"
    mesh = I.Mesh(nx, ny, p, (0.0, 2.0, 0.0, 2.0),
                  I.map_deforming(0.05) if moving else I.map_curved(0.05) if kind == "curved" else I.map_affine, moving=moving)
    prm = I.Params(order=p, n_elem=mesh.E, mach_ref=0.3, reynolds=30.0, viscous=True, moving=moving, kappa=1.0)
    g = lmfr.Context(prm, *mesh.connectivity())
    g.set_geometry(*mesh.nodes(0.07 if moving else 0.0))
    rng = np.random.default_rng(2)
    q = 1.0 + 0.1 * rng.standard_normal((4, mesh.E, mesh.Np))
    q[0] *= prm.gas_constant
    q, v = torch.tensor(q, device="cuda"), torch.tensor(rng.standard_normal(q.shape), device="cuda")
    g.set_option("operator_packs", 1)

    def run():
        return g.residual(q), g.jvp(q, v), g.bdf_operator(q, v, 20.0, 3.0)

    ref = run()
    for lanes in (64, 128):
        for grid in (1 << 24, 1000):
            g.set_option("tile_lanes", lanes)
            g.set_option("tile_grid", grid)
            for a, b in zip(ref, run()):
                assert torch.isfinite(a).all() and torch.equal(a, b), (lanes, grid)
