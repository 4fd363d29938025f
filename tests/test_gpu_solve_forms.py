"""Forms of the source and star matrices that the solve kernel tells apart, one
per workgroup of the build's tile table: a coupled quantity whose partner has no
source of its own, in the partner's wave or in another (one element further); a
quantity that is both stiff and coupled; a chain of two couplings; star rows of
more than six columns; and a last workgroup of one ordinary element.  Expected
values: the oracle where not said otherwise; bar: the 1e-10 per element and
quantity of the parity tests.  What each form may cost is bounded as well."""
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
PRECISIONS = {"fp64": dict(precision="fp64"), "fp32_refine2": dict(precision="fp32_refine", refine_steps=2)}
_ORACLE = {}


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _make(nq, N, n, seed):
    return wl.make_small(N, n, seed=seed) if nq == 13 else wl.make_maxwell(N, n, seed=seed)


def _forms(nq, N):
    """Workload, E and the elements that are checked (each form's and, next to
    it, an ordinary one of the same workgroup)."""
    elems = pbuild.solve_table(nq)[N][1]
    n = 4 * elems + 1
    w = _make(nq, N, n, 420 + N)
    E, s = w.E.copy(), 1.0 / w.dt
    a, b, c, d = 0, elems + 1, 2 * elems, 3 * elems
    assert elems >= 2 and len({e // elems for e in (a, b, c, d, n - 1)}) == 5
    far = 9 if nq == 13 else 4
    for e in (a, b):
        E[e, far, far] = 0.0
        E[e, 0, 0] = 0.0
        E[e, 0, far] = 0.3 * s
    stiff, partner = (6, 10) if nq == 13 else (0, 5)
    E[c, stiff, stiff], E[c, stiff, partner] = -2.0 * s, 0.4 * s
    E[d, 3, 3] = E[d, 4, 4] = E[d, 5, 5] = 0.0
    E[d, 3, 4], E[d, 4, 5] = 0.2 * s, -0.4 * s
    return w, E, sorted({a, a + 1, b, b - 1, c, c + 1, d, d + 1, n - 1})


@pytest.mark.parametrize("precision", list(PRECISIONS))
@pytest.mark.parametrize("nq", [13, 6])
@pytest.mark.parametrize("N", range(8))
def test_one_form_per_workgroup(N, nq, precision):
    print(f"[gpu] solve forms N={N} nq={nq} {precision}", flush=True)
    w, E, ids = _forms(nq, N)
    if (N, nq) not in _ORACLE:
        _ORACLE[(N, nq)] = opool.solve_many(N, w.star[ids], E[ids], w.Q0[ids], w.dt)
    Xo, Io = _ORACLE[(N, nq)]
    Q, Qi = api.predict(_dev(w.Q0), _dev(w.star), _dev(E), w.dt, N, **PRECISIONS[precision])
    torch.cuda.synchronize()
    parity.check(Q.cpu().numpy()[ids], Xo, TOL, "Q")
    parity.check(Qi.cpu().numpy()[ids], Io, TOL, "Qint")


@pytest.mark.parametrize("precision", list(PRECISIONS))
@pytest.mark.parametrize("N", [1, 3, 6, 7])
def test_star_rows_of_every_length(N, precision):
    """One star row of 6, 7, 12 or 13 columns in a workgroup of its own (the
    kernel takes six at a time), next to ordinary elements, and a workgroup of
    rows of every length.  Expected values: the one-element-per-workgroup
    reference kernel, which applies the same block elimination; such rows let
    the solution grow by up to 1e24, where the oracle's dense solve has no
    digit left."""
    print(f"[gpu] star rows N={N} {precision}", flush=True)
    elems = pbuild.solve_table(13)[N][1]
    w = wl.make_small(N, 5 * elems + 1, seed=460 + N)
    star, rng = w.star.copy(), np.random.default_rng(461 + N)

    def fill(e, row, columns):
        star[e, :, row, :] = 0.0
        pick = rng.permutation(13)[:columns]
        star[e][:, row, pick] = rng.standard_normal((3, columns)) * np.abs(w.star[e]).max() * 1e-3

    for g, columns in enumerate((6, 7, 12, 13)):
        fill(g * elems + g % elems, (3 * g + 1) % 13, columns)
    for row in range(13):
        fill(4 * elems, row, row + 1)
    args = (_dev(w.Q0), _dev(star), _dev(w.E), w.dt, N)
    Xr, Ir = api.predict(*args, reference_kernel=True)
    Q, Qi = api.predict(*args, **PRECISIONS[precision])
    torch.cuda.synchronize()
    parity.check(Q.cpu().numpy(), Xr.cpu().numpy(), TOL, "Q")
    parity.check(Qi.cpu().numpy(), Ir.cpu().numpy(), TOL, "Qint")


def _ms(call):
    call()
    best = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        best.append(a.elapsed_time(b))
    return min(best)


@pytest.mark.parametrize("nq,N,n", [(13, 6, 16384), (13, 3, 65536), (6, 5, 32768)])
def test_general_source_keeps_pace(nq, N, n):
    """A level of couplings adds one round of exchange per chunk to the solve
    of an ordinary E, no more than that solve itself: at most 1 + levels times
    its time (it was 16 times for one level at N = 6, 150 times for twelve,
    while the couplings were read from memory for every mode and time)."""
    print(f"[gpu] general source pace nq={nq} N={N}", flush=True)
    w = _make(nq, N, 64, 430 + N)
    pick = torch.arange(n, device="cuda") % 64
    star, Q0 = _dev(w.star)[pick].contiguous(), _dev(w.Q0)[pick].contiguous()
    Q = torch.empty((n, nq, w.Q0.shape[2], N + 1), dtype=torch.float64, device="cuda")
    Qi = torch.empty((n, nq, w.Q0.shape[2]), dtype=torch.float64, device="cuda")
    one = w.E.copy()
    one[:, 0, nq - 2] = 0.3 / w.dt
    full = w.E + np.triu(np.full((nq, nq), 0.1 / w.dt), 1)
    times = []
    for E in (w.E, one, full):
        Ed = _dev(E)[pick].contiguous()
        times.append(_ms(lambda: api.predict(Q0, star, Ed, w.dt, N, Q=Q, Qint=Qi)))
    print(f"  ordinary {times[0]:.3f} ms, one level {times[1]:.3f}, {nq - 1} levels {times[2]:.3f}", flush=True)
    assert times[1] <= 2 * times[0] and times[2] <= nq * times[0]


@pytest.mark.parametrize("nq", [13, 6])
def test_degree_zero_skips_the_star_matrices(nq):
    """Degree 0 has no green update and does without the star matrices, which
    are three quarters of its input: a large call takes less than half the time
    of degree 1, which needs them and four times the degrees of freedom (it was
    91 against 105 us, and 15.5 against 26, while degree 0 read them)."""
    print(f"[gpu] degree 0 pace nq={nq}", flush=True)
    n, times = 65536, []
    for N in (0, 1):
        w = _make(nq, N, 64, 440 + N)
        pick = torch.arange(n, device="cuda") % 64
        Q0, star, E = (_dev(a)[pick].contiguous() for a in (w.Q0, w.star, w.E))
        Q = torch.empty((n, nq, w.Q0.shape[2], N + 1), dtype=torch.float64, device="cuda")
        Qi = torch.empty((n, nq, w.Q0.shape[2]), dtype=torch.float64, device="cuda")
        times.append(_ms(lambda: [api.predict(Q0, star, E, w.dt, N, Q=Q, Qint=Qi) for _ in range(20)]))
    print(f"  degree 0 {times[0] / 20:.4f} ms, degree 1 {times[1] / 20:.4f}", flush=True)
    assert times[0] < times[1] / 2


@pytest.mark.parametrize("N,n", [(3, 65536), (4, 32768), (6, 16384)])
def test_long_star_rows_keep_pace(N, n):
    """A star row of 13 columns takes three passes of the green update: at most
    three times the ordinary time (it was 4 to 5 times while the dense rows were
    read from memory for every mode)."""
    print(f"[gpu] long star rows pace N={N}", flush=True)
    w = wl.make_small(N, 64, seed=470 + N)
    pick = torch.arange(n, device="cuda") % 64
    Q0, E = _dev(w.Q0)[pick].contiguous(), _dev(w.E)[pick].contiguous()
    Q = torch.empty((n, 13, w.Q0.shape[2], N + 1), dtype=torch.float64, device="cuda")
    Qi = torch.empty((n, 13, w.Q0.shape[2]), dtype=torch.float64, device="cuda")
    longer = w.star.copy()
    longer[:, :, 4, :] += np.random.default_rng(471).standard_normal((64, 3, 13)) * np.abs(w.star).max() * 1e-3
    times = []
    for star in (w.star, longer):
        sd = _dev(star)[pick].contiguous()
        times.append(_ms(lambda: api.predict(Q0, sd, E, w.dt, N, Q=Q, Qint=Qi)))
    print(f"  ordinary {times[0]:.3f} ms, one row of 13 columns {times[1]:.3f}", flush=True)
    assert times[1] <= 3 * times[0]
