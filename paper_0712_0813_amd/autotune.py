"""Launch-configuration autotuner for the step pass.

For one lattice class (dims, N, field count, storage precision) it times every
candidate launch configuration on a scratch simulation with seeded
preheating-shaped fields (HIP events around a few steps, through
ce_time_steps), keeps the fastest, and stores it in a JSON cache keyed by the
GPU architecture and the class.  `apply` sets a cached choice on a
simulation.  Timing runs only through the C ABI; nothing here computes the
evolution.

    python -m paper_0712_0813_amd.autotune --dims 3 --N 1024 --nfields 2
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time
from typing import Dict, List, Optional, Sequence, Tuple

import numpy as np

from . import ce

CACHE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "tune_cache.json")
_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)


def source_hash() -> str:
    """Hash of every kernel source, the public header and the build script: a
    cached choice is used only while these are unchanged."""
    h = hashlib.sha256()
    csrc = os.path.join(_PKG, "csrc")
    files = sorted(os.path.join(csrc, f) for f in os.listdir(csrc) if f.endswith((".hip", ".hpp", ".h")))
    files += [os.path.join(_ROOT, "include", "ce.h"), os.path.join(_PKG, "build.py")]
    for f in files:
        h.update(os.path.basename(f).encode())
        with open(f, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def class_key(arch: str, dims: int, N: int, nfields: int, precision: int) -> str:
    return f"{arch}/d{dims}/N{N}/nf{nfields}/{'fp64' if precision == ce.CE_FP64 else 'fp32'}"


_ARCH = None
KFD_NODES = "/sys/class/kfd/kfd/topology/nodes"


def _kfd_arch() -> Optional[str]:
    """gfx target of the first GPU node in the kernel driver's topology
    (gfx_target_version = major * 10000 + minor * 100 + stepping), read
    without initialising any GPU runtime."""
    root = KFD_NODES
    try:
        nodes = sorted(os.listdir(root), key=lambda n: int(n) if n.isdigit() else 1 << 30)
    except OSError:
        return None
    for n in nodes:
        try:
            with open(os.path.join(root, n, "properties")) as fh:
                props = dict(line.split()[:2] for line in fh if len(line.split()) >= 2)
        except (OSError, ValueError):
            continue
        v = int(props.get("gfx_target_version", "0") or 0)
        if v:
            return f"gfx{v // 10000}{(v // 100) % 100:x}{v % 100:x}"
    return None


def gpu_arch() -> str:
    """The GPU architecture name (e.g. gfx950) used in cache keys.  Read from
    the driver's topology; torch is asked only if that is unavailable (torch
    cannot initialise its own runtime once the library has initialised HIP
    in the same process, so it is not the first choice)."""
    global _ARCH
    if _ARCH is None:
        _ARCH = _kfd_arch()
        if _ARCH is None:
            try:
                import torch
                _ARCH = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
            except Exception:
                _ARCH = "unknown"
    return _ARCH


def chunk_lengths(N: int, max_chunks: int = 16) -> List[int]:
    """z-chunk lengths for the tiled pass: every power of two from 2 to N that
    divides N, and the near-even splits of N into 1..max_chunks chunks (the
    last chunk of such a split is shorter, e.g. 342 + 342 + 340 for 1024)."""
    out = set()
    z = 2
    while z <= N:
        if N % z == 0:
            out.add(z)
        z *= 2
    for nz in range(1, min(N, max_chunks) + 1):
        planes = -(-N // nz)
        if planes >= 2 and -(-N // planes) == nz:
            out.add(planes)
    return sorted(out)


def candidates(dims: int, N: int, grids: Sequence[int] = (0, 512, 768, 1024)) -> List[Tuple[int, ...]]:
    """Launch configurations (kernel, sites/thread, lanes/row, block, planes, grid);
    grid 0 is the library's evened resident grid.  Power-of-two chunks are
    tried with every grid, ragged chunk splits with the evened grid."""
    out = []
    if dims == 3:
        for (v, l, b) in ce.TILED_SHAPES:
            tx, ty = v * l, b // l
            if N % tx or N % ty:
                continue
            for z in chunk_lengths(N):
                for g in (grids if N % z == 0 else (0,)):
                    out.append((ce.CE_KERNEL_TILED3D, v, l, b, z, g))
    if dims == 2 and N % 256 == 0:
        for rows in (4, 8, 16, 32, 64, 128):
            if N % rows == 0:
                for g in grids:
                    out.append((ce.CE_KERNEL_STREAM2D, 4, 64, 256, rows, g))
    for g in (0, 1024, 2048, 4096):
        out.append((ce.CE_KERNEL_DIRECT, 0, 0, 0, 0, g))
    return out


MAX_STEP_BLOCK = 4096   # what ce_set_step_block takes


def _load_cache(path: str) -> Dict[str, dict]:
    if os.path.exists(path):
        with open(path) as fh:
            return json.load(fh)
    return {}


def tune_lattice(dims: int, N: int, nfields: int) -> "Lattice":
    """The lattice a class is tuned on: the 1024^3 expanding two-field
    workload (its coupling, time step, grid spacing and seed) at this size."""
    from .workloads import LATTICE1024_EXPANDING as W
    return W.with_(dims=dims, N=N, nfields=nfields, L=W.dx * N)


def tune(dims: int, N: int, nfields: int, precision: int = ce.CE_FP32, steps: int = 8,
         warmup: int = 3, cache_path: str = CACHE, verbose: bool = False, finalists: int = 4,
         final_steps: int = 40) -> dict:
    """Time every candidate (screening), re-time the `finalists` fastest and
    the library default with more steps twice, and record the fastest in the
    cache with the source hash it was measured on."""
    lat = tune_lattice(dims, N, nfields)
    arch = gpu_arch()
    results = []
    with ce.Simulation(dims, N, nfields, lat.L, lat.dt, lam=lat.lam, G=lat.G, mu2=lat.mu2,
                       expansion=lat.expansion, kappa=lat.kappa, precision=precision) as s:
        try:
            s.generate(ce.lattice_init_spec(lat))
        except ce.CeError as e:
            # device generation covers N a power of two up to 2048; other
            # sizes take the same seeded recipe from the host
            if e.status != ce.CE_EINVAL:
                raise
            from .inputs import make_initial
            phi, phid = make_initial(lat.seed, dims, N, lat.L, nfields, lat.m_eff2(), amp=lat.amp,
                                     background=lat.background)
            s.load(phi, phid)
            del phi, phid
        # no graph is captured (every call is shorter than a step block), and
        # launches whose steps can stay on the chip are timed that way
        most = min(max(steps, warmup, final_steps), MAX_STEP_BLOCK - 1)
        s.set_step_block(most + 1)

        def timed(n: int) -> float:
            return sum(s.time_steps(min(most, n - k)) for k in range(0, n, most)) / n

        def warm() -> None:
            for k in range(0, warmup, most):
                s.step(min(most, warmup - k))

        default = s.get_launch().as_tuple()
        screen = []
        for cfg in candidates(dims, N):
            try:
                s.set_launch(*cfg)
            except ce.CeError:
                continue
            warm()
            ms = timed(steps)
            chosen = s.get_launch().as_tuple()
            screen.append((ms, chosen))
            if verbose:
                print(f"{chosen} {ms:.4f} ms/step", file=sys.stderr, flush=True)
        screen.sort()
        finals = []
        for _, c in screen:
            if c not in finals:
                finals.append(c)
            if len(finals) == finalists:
                break
        if default not in finals:
            finals.append(default)
        for cfg in finals:
            s.set_launch(*cfg)
            warm()
            ms = min(timed(final_steps) for _ in range(2))
            results.append((ms, cfg))
            if verbose:
                print(f"final {cfg} {ms:.4f} ms/step", file=sys.stderr, flush=True)
    results.sort()
    best_ms, best = results[0]
    default_ms = min((ms for ms, c in results if c == default), default=float("nan"))
    entry = {"launch": list(best), "ms_per_step": best_ms, "default_launch": list(default),
             "default_ms_per_step": default_ms, "screened": len(screen), "finalists": len(results),
             "source_hash": source_hash(), "tuned_at": time.strftime("%Y-%m-%d %H:%M:%S")}
    _store(cache_path, class_key(arch, dims, N, nfields, precision), entry)
    return entry


def _store(cache_path: str, key: str, entry: dict) -> None:
    cache = _load_cache(cache_path)
    cache[key] = entry
    tmp = cache_path + ".tmp"
    with open(tmp, "w") as fh:
        json.dump(cache, fh, indent=1, sort_keys=True)
    os.replace(tmp, cache_path)


def member_candidates(dims: int, N: int) -> List[Tuple[int, ...]]:
    """Pool-member configurations: tiled with one tile per block, or direct."""
    out = []
    if dims == 3:
        for (v, l, b) in ce.TILED_SHAPES:
            tx, ty = v * l, b // l
            if N % tx or N % ty:
                continue
            z = 4
            while z <= N:
                tiles = (N // tx) * (N // ty) * (N // z)
                if N % z == 0 and tiles <= 4096:
                    out.append((ce.CE_KERNEL_TILED3D, v, l, b, z, tiles))
                z *= 2
    if dims == 2 and N % 256 == 0:
        for rows in (4, 8, 16, 32, 64):
            if N % rows == 0:
                groups = -(-(N // 256) * (N // rows) // 4)
                if groups <= 4096:
                    out.append((ce.CE_KERNEL_STREAM2D, 4, 64, 256, rows, groups))
    nq = N ** dims // 4
    out.append((ce.CE_KERNEL_DIRECT, 0, 0, 0, 0, max(1, min(2048, (nq + 255) // 256))))
    return out


def tune_pool(dims: int, N: int, nfields: int, count: int = 64, precision: int = ce.CE_FP32,
              block: int = 20, cache_path: str = CACHE, verbose: bool = False) -> dict:
    """Time pool blocks of `count` lattices of one class for every member
    configuration; cache the fastest under the class key prefixed 'pool/'."""
    from .inputs import make_initial
    L = 10.0 * N / 64
    dt = 0.01
    arch = gpu_arch()
    phi, phid = make_initial(3, dims, N, L, nfields, [3.0] + [100.0] * (nfields - 1))
    params = ce.make_params(dims, N, nfields, L, dt, G=(0.0, 100.0, 100.0), expansion=True, kappa=2.94,
                            precision=precision)
    default = tuple(ce.ce_pool_launch_for(params).as_tuple())
    results = []
    for cfg in member_candidates(dims, N):
        with ce.Pool(1 << 40) as pool:
            try:
                ids = [pool.admit(params, phi, phid, 10 ** 6, launch=cfg) for _ in range(count)]
            except ce.CeError:
                continue
            # poll with diagnostics waits for every block enqueued so far
            pool.run_block(block)
            pool.poll(ids[0])
            t0 = time.perf_counter()
            pool.run_block(block)
            pool.poll(ids[0])
            ms = (time.perf_counter() - t0) * 1e3 / block
        results.append((ms, cfg))
        if verbose:
            print(f"pool {cfg} {ms:.4f} ms/step ({count} lattices)", file=sys.stderr, flush=True)
    results.sort()
    best_ms, best = results[0]
    entry = {"launch": list(best), "ms_per_step": best_ms, "lattices": count, "default_launch": list(default),
             "default_ms_per_step": min((ms for ms, c in results if c == default), default=float("nan")),
             "candidates": len(results), "source_hash": source_hash(),
             "tuned_at": time.strftime("%Y-%m-%d %H:%M:%S")}
    _store(cache_path, "pool/" + class_key(arch, dims, N, nfields, precision), entry)
    return entry


def lookup_entry(dims: int, N: int, nfields: int, precision: int = ce.CE_FP32, arch: Optional[str] = None,
                 cache_path: str = CACHE, pool: bool = False) -> Optional[dict]:
    """The cached entry of a class if it was measured on the current sources
    (same source hash), else None."""
    cache = _load_cache(cache_path)
    key = ("pool/" if pool else "") + class_key(arch or gpu_arch(), dims, N, nfields, precision)
    e = cache.get(key)
    if not e or e.get("source_hash") != source_hash():
        return None
    return e


def lookup(dims: int, N: int, nfields: int, precision: int = ce.CE_FP32, arch: Optional[str] = None,
           cache_path: str = CACHE, pool: bool = False) -> Optional[Tuple[int, ...]]:
    e = lookup_entry(dims, N, nfields, precision, arch, cache_path, pool)
    return tuple(e["launch"]) if e else None


def apply(sim: "ce.Simulation", precision: int = ce.CE_FP32, cache_path: str = CACHE) -> bool:
    """Set the cached launch for this simulation's class; False if none."""
    cfg = lookup(sim.dims, sim.N, sim.nfields, precision, cache_path=cache_path)
    if cfg is None:
        return False
    sim.set_launch(*cfg)
    return True


def main(argv=None):
    ap = argparse.ArgumentParser()
    ap.add_argument("--dims", type=int, default=3)
    ap.add_argument("--N", type=int, nargs="+", default=[1024])
    ap.add_argument("--nfields", type=int, nargs="+", default=[2])
    ap.add_argument("--fp64", action="store_true")
    ap.add_argument("--steps", type=int, default=8)
    ap.add_argument("--cache", default=CACHE)
    ap.add_argument("--pool", type=int, default=0,
                    help="tune pool members with this many lattices per block instead")
    args = ap.parse_args(argv)
    prec = ce.CE_FP64 if args.fp64 else ce.CE_FP32
    for N in args.N:
        for nf in args.nfields:
            if args.pool:
                # about 2^28 site-fields per tuning block, 4..pool lattices
                count = int(max(4, min(args.pool, 2 ** 28 // (N ** args.dims * nf))))
                e = tune_pool(args.dims, N, nf, count=count, precision=prec, cache_path=args.cache,
                              verbose=True)
            else:
                e = tune(args.dims, N, nf, prec, steps=args.steps, cache_path=args.cache, verbose=True)
            print(json.dumps({"dims": args.dims, "N": N, "nfields": nf, "pool": args.pool, **e}), flush=True)


if __name__ == "__main__":
    main()
