"""Kernels at the edges of the build's tiles, against the oracle: the
six-quantity solve kernels of every degree over two full workgroups and a
partial one (the float32 chain's residual and correction too), and the corrector
at the degrees that no other test holds to an independent result."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pool as opool  # noqa: E402
from paper_2108_10565_amd import api  # noqa: E402
from paper_2108_10565_amd import build as pbuild  # noqa: E402
from paper_2108_10565_amd import workload as wl  # noqa: E402

import parity  # noqa: E402
import test_gpu_ader as gpu_ader  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-10
PRECISIONS = {"fp64": dict(precision="fp64"), "fp32_refine2": dict(precision="fp32_refine", refine_steps=2)}
_ORACLE = {}


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("precision", list(PRECISIONS))
@pytest.mark.parametrize("N", range(8))
def test_six_quantities(N, precision):
    elems = pbuild.solve_table(6)[N][1]
    print(f"[gpu] six-quantity tile edges N={N} elements per workgroup {elems} {precision}", flush=True)
    w = wl.make_maxwell(N, 2 * elems + 1, seed=480 + N)
    if N not in _ORACLE:
        _ORACLE[N] = opool.solve_many(N, w.star, w.E, w.Q0, w.dt)
    Xo, Io = _ORACLE[N]
    Q, Qi = api.predict(_dev(w.Q0), _dev(w.star), _dev(w.E), w.dt, N, **PRECISIONS[precision])
    torch.cuda.synchronize()
    parity.check(Q.cpu().numpy(), Xo, TOL, "Q")
    parity.check(Qi.cpu().numpy(), Io, TOL, "Qint")


@pytest.mark.parametrize("system,N", [("poro_heterogeneous", 5), ("maxwell", 3), ("maxwell", 5), ("maxwell", 7)])
def test_corrector(system, N):
    gpu_ader.test_corrector_matches_oracle(system, N)
