"""The solve kernel at the edges of its tiles: two full workgroups and a
partial one per degree (the tile table of the build), and the couplings that
decide between its forms -- a partner without a source of its own, possibly in
another wave; a quantity that is both stiff and coupled; a chain -- next to
ordinary elements.  Expected values: the one-element-per-workgroup reference
kernel, an independent implementation held to the oracle by the parity tests;
bar: the 1e-10 per element and quantity of those tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pool as opool  # noqa: E402
from paper_2108_10565_amd import api  # noqa: E402
from paper_2108_10565_amd import build as pbuild  # noqa: E402
from paper_2108_10565_amd import workload as wl  # noqa: E402

import parity  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-10


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _couplings(w, elems):
    """E of w with one coupling form per workgroup of `elems` elements."""
    E, s = w.E.copy(), 1.0 / w.dt
    first, tail = elems, w.n - 1
    E[first, 0, 9] = 0.3 * s                    # partner without a diagonal source
    E[w.n // 2, 6, 6] = -2.0 * s                # stiff and coupled (u <- uf)
    E[tail, 3, 4], E[tail, 4, 5], E[tail, 4, 4] = 0.2 * s, -0.4 * s, -3.0 * s   # chain
    return E


@pytest.mark.parametrize("precision", [dict(precision="fp64"), dict(precision="fp32_refine", refine_steps=2)],
                         ids=["fp64", "fp32_refine2"])
@pytest.mark.parametrize("N", range(8))
def test_tile_edges_and_couplings(N, precision):
    elems = pbuild.solve_table(13)[N][1]
    print(f"[gpu] solve tiles N={N} elements per workgroup {elems} {precision}", flush=True)
    w = wl.make_small(N, 2 * elems + 1, seed=400 + N)
    for E in (w.E, _couplings(w, elems)):
        args = (_dev(w.Q0), _dev(w.star), _dev(E), w.dt, N)
        Qr, Ir = api.predict(*args, reference_kernel=True)
        Q, Qi = api.predict(*args, **precision)
        torch.cuda.synchronize()
        parity.check(Q.cpu().numpy(), Qr.cpu().numpy(), TOL, "Q")
        parity.check(Qi.cpu().numpy(), Ir.cpu().numpy(), TOL, "Qint")


@pytest.mark.parametrize("N", range(4))
def test_tile_edges_maxwell(N):
    elems = pbuild.solve_table(6)[N][1]
    print(f"[gpu] solve tiles Maxwell N={N} elements per workgroup {elems}", flush=True)
    w = wl.make_maxwell(N, 2 * elems + 1, seed=500 + N)
    Xo, Io = opool.solve_many(N, w.star, w.E, w.Q0, w.dt)
    Q, Qi = api.predict(_dev(w.Q0), _dev(w.star), _dev(w.E), w.dt, N)
    torch.cuda.synchronize()
    parity.check(Q.cpu().numpy(), Xo, TOL, "Q")
    parity.check(Qi.cpu().numpy(), Io, TOL, "Qint")
