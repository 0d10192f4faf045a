"""The shared-tap gridder where the last 64 taps of a footprint leave fewer lanes with a tap than the 16 whose
registers the matrix products read: S^2 mod 64 = 4 (supports 14, 18, 30, 34), 1 (17) and, below one step, 9 (3), at
the shapes of 64 registers (16 waves, one plane a workgroup), plain, batched and reproducible.

Tolerance as for runs of every length: float32 tables and eight float32 products a tap, 5e-7 relative L2."""
import numpy as np
import pytest

from oracle import gridding, kernels, mueller
from test_gpu_shared_runs import TOL, rel, workload

torch = pytest.importorskip("torch")
pg = pytest.importorskip("paper_2206_15117_amd.polgrid")

pytestmark = pytest.mark.gpu

LENGTHS = 4 * [2, 3, 4, 5, 6, 7, 8, 1, 8, 2, 7, 3, 6, 4, 5, 1]  # 18 rows a wave


@pytest.mark.parametrize("support", [3, 14, 17, 18, 30, 34])
def test_few_lanes_with_a_tap(support):
    geom, uvw, vis, jones = workload(support, LENGTHS, 4, 40 + support)
    want = gridding.grid(geom, kernels.make_tables(geom, mueller.phi_grid(jones, 0.2)), uvw, vis)
    kg = pg.make_kernels(geom, 4, pg.KIND_GRID, jones=jones, eps_null=0.2)
    dv, du = torch.from_numpy(vis).cuda(), torch.from_numpy(uvw).cuda()
    for chunk in (1024, 20):
        p = pg.plan(kg, du, max_chunk=chunk).set_launch(3, 16, 16, 1, 1, 0)
        assert rel(pg.grid(p, kg, dv).cpu().numpy(), want) < TOL, chunk
        assert rel(pg.grid(p, kg, dv, deterministic=True).cpu().numpy(), want) < TOL, chunk
        out = torch.zeros((4, geom.n, geom.n), dtype=torch.complex64, device="cuda")
        b = pg.batch([(p, kg, dv, out)])
        b.grid()
        assert rel(out.cpu().numpy(), want) < TOL, chunk
        assert np.isfinite(want).all()
