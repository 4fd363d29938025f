"""Autotuner of the solve kernel's tile shape per quantity count and degree.

The tile shape is (waves per workgroup, elements per workgroup, modes per
chunk, waves per SIMD the registers are held to, X buffers, modes per chunk of
the correction and the residual): how many elements one workgroup predicts
together, how many modes of a degree block go through LDS at once and with how
many barriers, and how many waves share a SIMD.  They trade occupancy and lane
use against LDS, registers and how widely Khat is shared, so the best shape is
measured, not derived.

Two phases, because kernels are compiled on the host and timed on the GPU:

    python -m paper_2108_10565_amd.autotune build   [--nq 13 6] [--degrees 3 4 5 6]
        compiles, for every quantity count, degree and candidate shape, the
        fused kernels with that shape and links a variant library
        ``_tune/libstp_q{nq}_n{N}_{shape}.so`` (the other degrees and the C ABI
        come from the regular build's objects);

    python -m paper_2108_10565_amd.autotune measure [--nq 13 6] [--degrees ..] [--out DIR]
        loads the variants of a degree and times them in turn on seeded
        synthetic elements (HIP events on one stream, median of several
        rounds): the float64 predictor, the float32 chain, and the float32
        chain with one refinement, whose residual and correction are what the
        last entry of the shape is for; checks that every variant computes the
        same outputs as the first in each; and writes ``tiles.json`` for
        build.py.  The shape in use stays unless another's three times sum to
        less by more than KEPT_WITHIN, the spread of such sums between runs.

The candidate in use is always among those measured.  Candidates that do not
compile (LDS or register limits, a broadcast too close to a write) are skipped.
The chain on the matrix cores has its own shapes (``tiles`` in tiles.json),
which this program keeps as they are.
"""
from __future__ import annotations

import argparse
import concurrent.futures as cf
import ctypes
import json
import os
import sys
import time

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
TUNE_DIR = os.path.join(PKG, "_tune")
CANDIDATES = {
    13: {0: [(1, 4, 1, 2, 1, 1), (2, 9, 1, 2, 1, 1), (4, 16, 1, 2, 1, 1)],
         1: [(1, 2, 3, 3, 1, 3), (2, 4, 3, 3, 1, 3), (4, 9, 3, 3, 1, 3)],
         2: [(1, 1, 6, 4, 1, 6), (2, 3, 3, 4, 2, 6), (2, 3, 6, 4, 1, 3), (2, 3, 6, 4, 1, 6), (4, 6, 6, 4, 1, 6)],
         3: [(4, 4, 5, 4, 2, 5), (4, 4, 10, 3, 1, 5), (4, 4, 10, 3, 1, 10), (8, 9, 5, 4, 2, 5)],
         4: [(4, 3, 5, 3, 2, 5), (4, 3, 10, 3, 1, 5), (4, 3, 10, 3, 1, 7), (4, 3, 15, 2, 1, 7)],
         5: [(4, 3, 3, 3, 2, 3), (4, 3, 9, 3, 1, 2), (4, 3, 9, 3, 1, 3), (8, 6, 5, 2, 2, 3)],
         6: [(4, 2, 10, 2, 2, 10), (8, 5, 10, 2, 2, 10), (8, 5, 14, 2, 1, 7), (8, 5, 14, 2, 1, 10)],
         7: [(8, 4, 4, 2, 2, 3), (8, 4, 4, 2, 2, 4), (8, 4, 6, 2, 1, 4)]},
    6: {0: [(1, 10, 1, 2, 1, 1), (2, 20, 1, 2, 1, 1), (4, 40, 1, 2, 1, 1)],
        1: [(1, 5, 3, 3, 1, 3), (2, 10, 3, 3, 1, 3)],
        2: [(1, 3, 6, 4, 1, 6), (2, 7, 6, 4, 1, 3), (2, 7, 6, 4, 1, 6)],
        3: [(4, 10, 5, 4, 2, 5), (4, 10, 10, 3, 1, 4), (4, 10, 10, 3, 1, 5)],
        4: [(4, 8, 5, 3, 2, 5), (4, 8, 10, 3, 1, 5), (4, 8, 10, 3, 1, 7)],
        5: [(4, 6, 3, 3, 2, 3), (4, 6, 9, 3, 1, 2), (4, 6, 9, 3, 1, 3)],
        6: [(4, 6, 4, 2, 2, 4), (4, 6, 7, 2, 1, 3), (4, 6, 7, 2, 1, 4)],
        7: [(8, 10, 3, 2, 2, 3), (8, 10, 7, 2, 1, 3), (8, 10, 8, 2, 1, 3)]}}
ELEMENTS = {0: 262144, 1: 262144, 2: 262144, 3: 131072, 4: 65536, 5: 65536, 6: 32768, 7: 16384}
POOL = 384          # generated elements the timed ones are gathered from
KEPT_WITHIN = 0.015
# paths: (precision, refinement steps, bound of the relative difference between
# two shapes' outputs: their sums run in another order)
PATHS = {"float64": (0, 0, 1e-12), "float32 chain": (1, 0, 1e-2), "float32, 1 refinement": (1, 1, 1e-8)}


METHOD = (f"milliseconds per call of each path on gathered synthetic elements, candidates in turn, median of the rounds, "
          f"HIP events on one stream; the shape in use stays unless another's sum is lower by {100 * KEPT_WITHIN:g}%")


def candidates(nq: int, N: int):
    """The shapes tried, the one in use first."""
    from . import build as b
    used = b.solve_table(nq)[N]
    return [used] + [c for c in CANDIDATES[nq][N] if c != used]


def shape_name(shape) -> str:
    return "x".join(str(v) for v in shape)


def variant_path(nq: int, N: int, shape) -> str:
    return os.path.join(TUNE_DIR, f"libstp_q{nq}_n{N}_{shape_name(shape)}.so")


def build_variants(counts, degrees, jobs: int | None = None, verbose: bool = True):
    from . import build as b
    objs = dict((o, cmd) for cmd, o in b._objects())
    if not all(os.path.exists(o) for o in objs):
        if verbose:
            print("[autotune] running the regular build first", flush=True)
        b.build()
    os.makedirs(TUNE_DIR, exist_ok=True)
    tune_obj = os.path.join(b.BUILD, "tune")
    os.makedirs(tune_obj, exist_ok=True)
    work = [(nq, N, shape, os.path.join(tune_obj, f"kernel_fused_q{nq}_n{N}_{shape_name(shape)}.o"))
            for N in sorted(degrees, reverse=True) for nq in counts for shape in candidates(nq, N)]
    tiles = b.tile_table()

    def one(item):
        nq, N, shape, obj = item
        try:
            b.compile_fused(b.fused_object_cmd(N, tiles[N], shape, obj, nq), obj)
        except RuntimeError as exc:
            lines = str(exc).splitlines()
            return item, next((l for l in lines if "error:" in l or "too close" in l), lines[-1]).split("error: ")[-1][:200]
        others = [o for o in objs if os.path.basename(o) != b.fused_object_name(nq, N)]
        b._run([b.HIPCC, f"--offload-arch={b.ARCH}", "-shared", "-fPIC", "-o", variant_path(nq, N, shape)] + others + [obj])
        return item, None

    failed = {}
    with cf.ThreadPoolExecutor(max_workers=jobs or min(8, os.cpu_count() or 4)) as ex:
        for item, err in ex.map(one, work):
            nq, N, shape, _ = item
            if verbose:
                print(f"[autotune] nq={nq} N={N} {shape_name(shape)}: {'built' if err is None else 'skipped: ' + err}",
                      flush=True)
            if err is not None:
                failed[f"{nq}:{N}:{shape_name(shape)}"] = err
    json.dump({"failed": failed}, open(os.path.join(TUNE_DIR, "build.json"), "w"), indent=1)
    return failed


def _load(path):
    lib = ctypes.CDLL(path)
    vp, i64, dbl, sz, ci = ctypes.c_void_p, ctypes.c_int64, ctypes.c_double, ctypes.c_size_t, ctypes.c_int
    lib.stp_create.argtypes = [ctypes.POINTER(vp)]
    lib.stp_predict_nq.argtypes = [vp, vp, ci, ci, i64, dbl, vp, vp, vp, vp, vp, ci, ci, vp, sz, ctypes.c_uint]
    lib.stp_predict_nq.restype = ci
    h = vp()
    if lib.stp_create(ctypes.byref(h)) != 0:
        raise RuntimeError(f"stp_create failed in {path}")
    return lib, h


def measure_degree(nq: int, N: int, rounds: int):
    """{shape: {path: median ms}} of the built candidates."""
    import torch

    from . import api
    from . import workload as wl
    n = ELEMENTS[N]
    w = wl.make_small(N, POOL, seed=900 + N) if nq == 13 else wl.make_maxwell(N, POOL, seed=900 + N)
    pick = torch.arange(n, device="cuda") % POOL
    Q0, star, E = (torch.from_numpy(a).cuda()[pick].contiguous() for a in (w.Q0, w.star, w.E))
    Q = torch.empty((n, nq, wl.n_modes(N), N + 1), dtype=torch.float64, device="cuda")
    Qi = torch.empty((n, nq, wl.n_modes(N)), dtype=torch.float64, device="cuda")
    size = api.workspace_size(N, n, "fp32_refine", 1, nq)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream()
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    built = [s for s in candidates(nq, N) if os.path.exists(variant_path(nq, N, s))]
    libs = {s: _load(variant_path(nq, N, s)) for s in built}

    def call(shape, path):
        lib, h = libs[shape]
        prec, steps, _ = PATHS[path]
        st = lib.stp_predict_nq(h, ctypes.c_void_p(stream.cuda_stream), nq, N, n, float(w.dt), ptr(star), ptr(E), ptr(Q0),
                                ptr(Q), ptr(Qi), prec, steps, ptr(ws) if steps else None, size if steps else 0, 0)
        if st != 0:
            raise RuntimeError(f"stp_predict_nq returned {st} ({variant_path(nq, N, shape)})")

    out = {s: {} for s in built}
    for path, (_, _, bound) in PATHS.items():
        times, ref = {s: [] for s in built}, None
        for s in built:
            call(s, path)
            sample = Q[:POOL].clone()
            ref = sample if ref is None else ref
            diff = float(((sample - ref).norm() / ref.norm()).cpu())
            if not diff <= bound:
                raise RuntimeError(f"{variant_path(nq, N, s)}: other outputs ({path}: {diff:.2e})")
        for _ in range(rounds):
            for s in built:  # in turn
                a, b_ = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                call(s, path)
                b_.record()
                torch.cuda.synchronize()
                times[s].append(a.elapsed_time(b_))
        for s in built:
            out[s][path] = sorted(times[s])[rounds // 2]
    for s in built:
        print(f"[autotune] nq={nq} N={N} n={n} {shape_name(s)}: "
              + ", ".join(f"{p} {out[s][p]:.4f} ms" for p in PATHS), flush=True)
    return out


def measure(counts, degrees, out_dir: str, rounds: int = 9):
    import torch

    from . import build as b
    doc = json.load(open(b.TILES))
    if doc.get("measurements", {}).get("method") != METHOD:
        doc["measurements"] = {"method": METHOD, "elements": {str(N): n for N, n in ELEMENTS.items()},
                               "ms": {str(nq): {} for nq in CANDIDATES}}
    doc["measurements"].update(device=f"{torch.cuda.get_device_name(0)} ({b.ARCH})", date=time.strftime("%Y-%m-%d"))
    for nq in counts:
        for N in degrees:
            res = measure_degree(nq, N, rounds)
            total = {s: sum(r.values()) for s, r in res.items()}
            if not total:
                raise RuntimeError(f"no variants of degree {N} with {nq} quantities in {TUNE_DIR}: run the build phase")
            used, best = b.solve_table(nq)[N], min(total, key=total.get)
            if used not in total or total[best] < (1 - KEPT_WITHIN) * total[used]:
                used = best
            doc["solve"][str(nq)][str(N)] = list(used)
            doc["measurements"]["ms"][str(nq)][str(N)] = {
                shape_name(s): {p: round(t, 4) for p, t in r.items()} for s, r in res.items()}
            torch.cuda.empty_cache()
    os.makedirs(out_dir, exist_ok=True)
    path = os.path.join(out_dir, "tiles.json")
    json.dump(doc, open(path, "w"), indent=1)
    print(f"[autotune] wrote {path}: {doc['solve']}", flush=True)
    return doc


def main(argv=None):
    ap = argparse.ArgumentParser(description=__doc__.split("\n\n")[0])
    ap.add_argument("phase", choices=["build", "measure"])
    ap.add_argument("--nq", type=int, nargs="+", default=sorted(CANDIDATES, reverse=True), choices=sorted(CANDIDATES))
    ap.add_argument("--degrees", type=int, nargs="+", default=list(range(0, 8)))
    ap.add_argument("--out", default=TUNE_DIR,
                    help="directory of the measured tiles.json (copy it over the package's)")
    ap.add_argument("--jobs", type=int, default=None)
    args = ap.parse_args(argv)
    if args.phase == "build":
        failed = build_variants(args.nq, args.degrees, args.jobs)
        print(f"[autotune] built; {len(failed)} candidate(s) skipped", flush=True)
    else:
        measure(args.nq, args.degrees, args.out)


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    main()
