"""The corrector's splits of an element over waves: few elements (the output
tiles spread over waves, the split the oracle tests of the corrector run) and
more than one per SIMD (13 copies of the mesh where degree 7 takes a third
split), with a last workgroup that is not full.  The same elements in copies
of one mesh must give the same result in all.  They accumulate every output over the same terms in the same order, so they may
differ by the rounding of a few hundred products at most: 1e-13 of the norm."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2108_10565_amd import mesh as pmesh  # noqa: E402
from paper_2108_10565_amd import workload as wl  # noqa: E402
from paper_2108_10565_amd.ader import AderSolver  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [13, 6])
@pytest.mark.parametrize("N,copies", [(N, 4) for N in range(8)] + [(7, 13)])
def test_splits_agree(N, copies, nq):
    print(f"[gpu] corrector splits N={N} nq={nq} copies={copies}", flush=True)
    M = pmesh.periodic_cube(4)
    n, rng = M.n, np.random.default_rng(700 + N)
    if nq == 13:
        A, B, C, E = wl.jacobians(wl.make_small(1, 4, seed=44).meta["materials"])
    else:
        A, B, C, E = wl.maxwell_jacobians(rng.uniform(1, 10, 4), rng.uniform(1, 2, 4), rng.uniform(0, 5, 4))
    pick = rng.integers(0, 4, n)
    s = AderSolver(N, M, np.stack([A, B, C], axis=1)[pick], E[pick])
    Q = torch.from_numpy(rng.standard_normal((n, nq, s.B))).cuda()
    Qint = torch.from_numpy(1e-6 * rng.standard_normal((n, nq, s.B))).cuda()
    ref = s.correct(Q.clone(), Qint)
    # copies of the mesh and three more elements of the last copy: 1,283 or 4,163
    idx = torch.cat([torch.arange(n)] * copies + [torch.arange(3)]).cuda()
    shift = n * torch.cat([torch.arange(copies).repeat_interleave(n), torch.full((3,), copies - 1)]).cuda()
    for name in ("star", "E", "Gp", "Gm", "nb_code"):
        setattr(s, name, getattr(s, name)[idx].contiguous())
    s.neighbor = (s.neighbor[idx] + shift[:, None]).to(torch.int32).contiguous()
    got = s.correct(Q[idx].contiguous(), Qint[idx].contiguous())
    torch.cuda.synchronize()
    want = ref[idx]
    err = ((got - want).norm(dim=(1, 2)) / want.norm(dim=(1, 2))).max()
    assert float(err) <= 1e-13, float(err)
