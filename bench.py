"""Benchmark: compact Life on the Sierpinski triangle vs the bounding-box grid.

Workload (N=1): level-16 Sierpinski triangle, replicas (0,0),(1,0),(0,1),
43,046,721 compact cells, uint8 states from a Bernoulli(0.5) SplitMix64 start
(seed 2201), B3/S23 steps ping-ponging between two compact buffers.  One
"step" is one B3/S23 update of every cell.  The K timed steps are one
sqz_compact_run call, in the run form the library picks for K steps: from 10
steps (and for even counts below) one launch that holds all 243 tiles on the
chip for all K steps, exchanging ring subtrees every 31 steps; otherwise
launches of up to 31 steps.  The other form is timed beside it.  The
same steps on the 65536 x 65536 bounding-box grid give the speedup (these
comparison runs go first, so the headline is not the process's first GPU
work); the
level-20 triangle (3.49e9 cells, 20 steps, Bernoulli(0.3)) gives the largest
workload.

Roofline: a level-16 run touches HBM at its ends only; it is bound by the
vector-ALU issue of a step and by the latency of its chain of LDS accesses.
`roofline` reports counter-measured VALU wave-instructions per dispatch (from
the committed rocprofv3 summary of the same kernel source and dispatch size)
over the live dispatch time, against the chip's peak of two wave64 instructions
per CU per clock; HBM bytes are secondary fields.  The level-20 run is bound by
HBM and reports the counters' bytes.

Prints one JSON line.  Inputs are resident in HBM before timing starts.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "compact cell-updates/s vs expanded bounding-box on 1 MI355X; HBM GB/s % of peak"
TRIANGLE = (2, [(0, 0), (1, 0), (0, 1)])
HBM_PEAK_GBS = 8000.0  # MI355X HBM3E
BYTES_PER_UPDATE = 2   # one byte read, one byte written per cell per step
NUM_CUS, CLOCK_HZ = 256, 2.4e9  # MI355X compute units and peak engine clock


def log(msg: str) -> None:
    print(msg, file=sys.stderr, flush=True)


def time_steps(torch, step, steps: int, warmup: int):
    """Run `warmup` untimed then `steps` timed calls of step(i); HIP events on the
    current stream (the stream the library launches on).  Returns seconds."""
    for i in range(warmup):
        step(i)
    torch.cuda.synchronize()
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for i in range(steps):
        step(warmup + i)
    end.record()
    torch.cuda.synchronize()
    return start.elapsed_time(end) / 1e3


# Most Life steps a launch of a run takes here: tiles sliced across subtrees (the
# triangle) and bit rows (the carpet)
STEPS_PER_LAUNCH = {3: 31, 8: 15}


def run_launches(F, steps: int) -> int:
    """Launches over all cells that sqz_compact_run makes for `steps` steps: of nearly
    equal step counts, at most STEPS_PER_LAUNCH each; where their number has not the
    parity of `steps`, the triangle's last one updates in place, the carpet takes one more."""
    if F.run_steps_per_launch < 2:
        return steps
    n = -(-steps // STEPS_PER_LAUNCH[F.k])
    return n + (1 if F.k == 8 and n % 2 != steps % 2 else 0)


def compact_run(torch, F, seed, p, steps, warmup, impl="auto", form="auto"):
    """Seconds for `steps` Life steps after `warmup` untimed ones.  impl "auto" runs
    them as one sqz_compact_run_form call (the library's step loop, in run form
    `form`); other impls launch one step at a time."""
    a = F.fill_bernoulli(seed, p)
    b = torch.empty_like(a)
    if impl == "auto":
        x = F.compact_run(a, b, warmup, form=form)
        y = b if x is a else a
        torch.cuda.synchronize()
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        F.compact_run(x, y, steps, form=form)
        end.record()
        torch.cuda.synchronize()
        sec = start.elapsed_time(end) / 1e3
    else:
        bufs = (a, b)

        def step(i):
            F.compact_step(bufs[i & 1], bufs[(i + 1) & 1], impl=impl)

        sec = time_steps(torch, step, steps, warmup)
    del a, b
    return sec


def bb_run(torch, F, seed, p, steps, warmup):
    a = F.fill_bernoulli(seed, p, layout="expanded")
    b = torch.empty_like(a)
    bufs = (a, b)

    def step(i):
        F.expanded_step(bufs[i & 1], bufs[(i + 1) & 1])

    sec = time_steps(torch, step, steps, warmup)
    del a, b
    torch.cuda.empty_cache()
    return sec


def run_source_hash() -> str:
    import hashlib

    src = os.path.join(ROOT, "paper_2201_00613_amd", "csrc")
    h = hashlib.sha256()
    for f in ("slice.hip", "slice_device.h", "tile_device.h", "common.h"):
        h.update(open(os.path.join(src, f), "rb").read())
    return h.hexdigest()[:16]


def profiled_counters(profile: str, workload: str):
    """Counter figures of a run kernel (bytes and vector-ALU instructions per
    dispatch) from a committed rocprofv3 summary under profiles/, if the kernel
    source is unchanged since it was taken (sha256 prefix of the run kernels' sources)."""
    import re

    path = os.path.join(ROOT, "profiles", profile)
    if not os.path.exists(path):
        return None
    m = re.search(r"```json\n(.*?)\n```", open(path).read(), re.S)
    if not m:
        return None
    rec = json.loads(m.group(1))
    if rec["workload"] != workload or rec["source_sha256_16"] != run_source_hash():
        return None
    return rec


# Vector-ALU peak of the chip: the datasheet's binary32 vector rate, 157.3 TFLOP/s at
# 2.4 GHz on 256 CUs, is 256 FLOP per CU per clock, i.e. 128 lanes of fused
# multiply-add, two 64-lane wave-instructions per CU per clock.
VALU_PEAK_PER_CU_CLOCK = 157.3e12 / (NUM_CUS * CLOCK_HZ) / 128
VALU_PEAK_G = VALU_PEAK_PER_CU_CLOCK * NUM_CUS * CLOCK_HZ / 1e9


def counter_roofline(rec, steps: int, sec: float, launches: int, cells: int, profile: str):
    """Roofline of a Life run from a committed profile's counters per dispatch (of the
    same number of steps) over the live launch time: VALU wave-instructions against the
    chip's peak or, where the profile says that HBM bounds the kernel, its HBM bytes
    against the peak bandwidth.  None when the profile does not hold a dispatch of this
    many steps."""
    if not rec:
        return None
    per = steps // launches if launches and steps % launches == 0 else None
    entry = rec["dispatch"].get(str(per)) if per else None
    if entry is None:
        return None
    launch_s = sec / launches
    valu = entry["valu_insts"] / launch_s / 1e9
    traffic = entry["traffic_bytes"] / launch_s / 1e9
    out = {"traffic": traffic, "traffic_unit": "GB/s",
           "traffic_vs_algorithmic": entry["traffic_bytes"] / (BYTES_PER_UPDATE * cells),
           "valu_per_cu_clock": valu * 1e9 / NUM_CUS / CLOCK_HZ,
           "counters_from": f"profiles/{profile} (dispatches of {per} steps; source hash {rec['source_sha256_16']})"}
    if rec["bound"] == "hbm":
        return {"bound": "hbm", "achieved": traffic, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": traffic / HBM_PEAK_GBS, **out}
    return {"bound": "alu", "achieved": valu, "peak": VALU_PEAK_G, "unit": "G VALU wave-instructions/s",
            "frac": valu / VALU_PEAK_G, "note": rec["note"], **out}


def cpu_baseline(r: int, seed: int, p: float, min_sec: float, max_steps: int) -> dict:
    """The oracle (plain C, OpenMP, lambda + 8 nu per cell) stepping the same workload:
    whole steps from the same start until min_sec have elapsed (at most max_steps)."""
    import oracle

    O = oracle.Fractal(*TRIANGLE, r)
    state = O.fill_compact(seed, p)
    steps, t0 = 0, time.perf_counter()
    while steps < max_steps and (steps == 0 or time.perf_counter() - t0 < min_sec):
        state = O.life_compact(state)
        steps += 1
    sec = time.perf_counter() - t0
    return {"value": O.N * steps / sec, "unit": "cell-updates/s", "cores": oracle.num_threads(), "kind": "oracle",
            "sample": f"{steps} full B3/S23 step(s) of the level-{r} triangle ({O.N} cells each), {sec:.1f} s",
            "cpu_model": cpu_model(), "single_core": single_core_baseline(r, seed, p)}


def cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


SINGLE_CORE = '''
import sys, time
sys.path.insert(0, {root!r})
import oracle
O = oracle.Fractal({s}, {offs!r}, {r})
state = O.fill_compact({seed}, {p})
t0 = time.perf_counter()
O.life_compact(state, 0, {cells})
print(time.perf_counter() - t0, oracle.num_threads())
'''


def single_core_baseline(r: int, seed: int, p: float, cells: int = 1 << 21) -> dict:
    """The oracle on one host thread (a child process with OMP_NUM_THREADS=1): one step
    of the first `cells` compact cells of the same workload."""
    import subprocess

    code = SINGLE_CORE.format(root=ROOT, s=TRIANGLE[0], offs=[list(o) for o in TRIANGLE[1]], r=r, seed=seed, p=p,
                              cells=cells)
    env = dict(os.environ, OMP_NUM_THREADS="1")
    try:
        res = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=300)
        sec, threads = res.stdout.split()
        return {"value": cells / float(sec), "unit": "cell-updates/s", "cores": int(threads),
                "sample": f"one B3/S23 step of compact cells [0, {cells}) of the level-{r} triangle, {float(sec):.2f} s"}
    except (subprocess.SubprocessError, ValueError) as e:
        return {"value": None, "error": str(e)[:200]}


def maps_leg(torch, F, seed, p, steps: int) -> dict:
    """Scalar look-up-table maps vs matrix-core (int8 MFMA) maps at the benchmark level:
    lambda over every compact index, nu over every fractal point, and the thread-level
    Life step with each (one lambda and eight nu per cell)."""
    idx = torch.arange(F.cells, dtype=torch.int64, device="cuda")
    xy = torch.empty((F.cells, 2), dtype=torch.int32, device="cuda")
    back = torch.empty(F.cells, dtype=torch.int64, device="cuda")
    res = {"cells": F.cells, "steps": steps}
    for impl in ("scalar", "mfma"):
        sl = time_steps(torch, lambda i: F.lambda_map(idx, impl=impl, out=xy), steps, 2)
        sn = time_steps(torch, lambda i: F.nu_map(xy, impl=impl, out=back), steps, 2)
        life = "cell" if impl == "scalar" else "cell_mfma"
        sc = compact_run(torch, F, seed, p, steps, 2, impl=life)
        res[impl] = {"lambda_ms": sl * 1e3 / steps, "lambda_maps_per_s": F.cells * steps / sl,
                     "nu_ms": sn * 1e3 / steps, "nu_maps_per_s": F.cells * steps / sn,
                     "life_impl": life, "life_ms_per_step": sc * 1e3 / steps,
                     "life_cell_updates_per_s": F.cells * steps / sc}
    res["mfma_speedup"] = {k: res["scalar"][k] / res["mfma"][k] for k in ("lambda_ms", "nu_ms", "life_ms_per_step")}
    del idx, xy, back
    torch.cuda.empty_cache()
    return res


def blocks_leg(torch, F, seed, p, steps: int) -> dict:
    """The block-size / memory trade-off at the benchmark level: for blocks of side
    rho = 2^m, Life steps on micro-block storage (k^(r-m) blocks of rho x rho bytes)
    and with the lambda(omega) approach (expanded n x n array, workgroups over the
    compact grid of blocks).  Memory is the two state buffers."""
    res = {"cells": F.cells, "steps": steps, "expanded_bytes_x2": 2 * F.n * F.n, "micro_blocks": [],
           "lambda_omega": []}
    a = F.fill_bernoulli(seed, p)
    for m in range(0, 7):
        nbytes = F.microblock_bytes(m)
        x = F.microblock_pack(a, m)
        y = torch.empty_like(x)
        bufs = (x, y)
        sec = time_steps(torch, lambda i: F.microblock_step(bufs[i & 1], bufs[(i + 1) & 1], m), steps, 2)
        res["micro_blocks"].append({"rho": 2 ** m, "bytes_x2": 2 * nbytes, "mrf": F.n * F.n / nbytes,
                                    "ms_per_step": sec * 1e3 / steps, "cell_updates_per_s": F.cells * steps / sec})
        del x, y, bufs
    del a
    torch.cuda.empty_cache()
    e = F.fill_bernoulli(seed, p, layout="expanded")
    f = e.clone()
    bufs = (e, f)
    for m in range(0, 7):
        sec = time_steps(torch, lambda i: F.lambda_omega_step(bufs[i & 1], bufs[(i + 1) & 1], m), steps, 2)
        res["lambda_omega"].append({"rho": 2 ** m, "ms_per_step": sec * 1e3 / steps,
                                    "cell_updates_per_s": F.cells * steps / sec})
    del e, f, bufs
    torch.cuda.empty_cache()
    return res


def batch_leg(torch, sqz, steps: int) -> dict:
    """512 instances drawn from seed over triangle, carpet and Vicsek (1e4..1e7 cells
    each), Bernoulli(0.5), `steps` steps as one graph replay after autotuning."""
    from paper_2201_00613_amd import workloads as W

    inst = W.batch_instances(512, 2201)
    cache, fr = {}, []
    for name, s, offs, r, seed in inst:
        if (name, r) not in cache:
            cache[(name, r)] = sqz.Fractal(s, offs, r)
        fr.append(cache[(name, r)])
    B = sqz.Batch(fr)
    seeds = [x[4] for x in inst]
    a = B.fill_bernoulli(seeds, 0.5)
    b = B.empty_state()
    wg = B.autotune(a, b)
    a = B.fill_bernoulli(seeds, 0.5, out=a)
    B.run(a, b, steps)  # capture + warm-up
    a = B.fill_bernoulli(seeds, 0.5, out=a)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    B.run(a, b, steps)
    e1.record()
    torch.cuda.synchronize()
    sec = e0.elapsed_time(e1) / 1e3
    res = {"instances": len(inst), "cells": B.total_cells, "steps": steps, "ms_per_step": sec * 1e3 / steps,
           "cell_updates_per_s": B.total_cells * steps / sec,
           "algorithmic_gbs_per_step": 2 * B.total_cells * steps / sec / 1e9, "wg_per_cu": wg, "graph": True,
           "steps_per_launch": B.steps_per_launch, "tiled_launch": B.tiled_launch,
           "mix": {k: sum(1 for x in inst if x[0] == k) for k in ("triangle", "carpet", "vicsek")}}
    # the same run with each launch form of the tiled instances (tuned steps per launch and grid)
    chosen = res["tiled_launch"]
    res["ms_per_step_by_tiled_form"] = {}
    for form in ("groups", "persistent", "per_tile"):
        B.set_tiled_launch(form)
        a = B.fill_bernoulli(seeds, 0.5, out=a)
        B.run(a, b, steps)  # capture + warm-up
        a = B.fill_bernoulli(seeds, 0.5, out=a)
        torch.cuda.synchronize()
        e0.record()
        B.run(a, b, steps)
        e1.record()
        torch.cuda.synchronize()
        res["ms_per_step_by_tiled_form"][form] = e0.elapsed_time(e1) / steps
    B.set_tiled_launch(chosen["form"])
    del a, b, B, fr, cache
    torch.cuda.empty_cache()
    return res


def repeat_stats(torch, F, seed, p, steps: int, reps: int, form: str = "auto") -> dict:
    """Mean and standard error of ms per step over `reps` further timed runs of the
    same `steps` (each one sqz_compact_run_form call on freshly filled buffers)."""
    import statistics

    ms = [compact_run(torch, F, seed, p, steps, 2, form=form) * 1e3 / steps for _ in range(reps)]
    return {"n": reps, "mean_ms_per_step": statistics.fmean(ms),
            "stderr_ms_per_step": statistics.stdev(ms) / len(ms) ** 0.5 if reps > 1 else 0.0,
            "min_ms_per_step": min(ms), "max_ms_per_step": max(ms)}


def carpet_life_leg(torch, sqz, steps: int) -> dict:
    """Life on the level-9 Sierpinski carpet (134,217,728 cells; bit-row tiles, up to
    fifteen steps per launch), Bernoulli(0.5), `steps` steps as one sqz_compact_run call, after
    an untimed run of the same steps (a first run in the process is measurably slower)."""
    from paper_2201_00613_amd import workloads as W

    F = sqz.Fractal(*W.CARPET, 9)
    sec = compact_run(torch, F, 2201, 0.5, steps, steps)
    launches = run_launches(F, steps)
    res = {"fractal": "sierpinski carpet s=3 k=8", "level": 9, "cells": F.cells, "steps": steps,
           "steps_per_launch": steps / launches, "launches": launches, "ms_per_step": sec * 1e3 / steps,
           "cell_updates_per_s": F.cells * steps / sec,
           "algorithmic_gbs_per_launch": BYTES_PER_UPDATE * F.cells * launches / sec / 1e9}
    del F
    torch.cuda.empty_cache()
    return res


GOLDEN_C5 = os.path.join(ROOT, "tests", "golden", "carpet_r9_diffusion.npz")


def golden_error(torch, F, field, dtype: str, offset: float, steps: int):
    """Error of the level-9 carpet diffusion after `steps` steps against the stored
    binary64 values (tests/golden/carpet_r9_diffusion.npz, written from the CPU
    oracle): max |u - u64| over the stored cells over the binary64 field's infinity
    norm.  None when no stored checkpoint has this step count."""
    import numpy as np

    if not os.path.exists(GOLDEN_C5):
        return None
    g = np.load(GOLDEN_C5, allow_pickle=False)
    hit = [i for i, t in enumerate(g["steps"]) if int(t) == steps]
    if not hit or int(g["level"]) != F.r or abs(float(g["coef"]) - 0.1) > 1e-12 or int(g["seed"]) != 2201:
        return None
    i = hit[0]
    u = field if dtype == "f32" else F.bf16_decode(field, offset)
    got = u[torch.from_numpy(g["idx"]).cuda()].double().cpu().numpy()
    return {"t": steps, "cells": int(g["idx"].size),
            "value": float(np.max(np.abs(got - g["values"][i])) / g["inf_norm"][i]),
            "bar": 1e-5 if dtype == "f32" else 2e-2}


MASS_EVERY = 100  # diffusion steps between binary64 mass reductions (and one at the end)


def diffusion_leg(torch, sqz, steps: int) -> dict:
    """Carpet r=9 (134,217,728 cells), coef 0.1, U(0,1) start: binary32 and bfloat16
    (offset storage, stochastic rounding) for `steps` steps, with a binary64 mass
    reduction on the device every MASS_EVERY steps and at the end inside the timed
    region (each into its own work buffer, read after the clock stops); the mass
    drift at every checkpoint and the error against the stored binary64 values."""
    from paper_2201_00613_amd import MASS_WORK_DOUBLES
    from paper_2201_00613_amd import workloads as W

    F = sqz.Fractal(*W.CARPET, 9)
    res = {"fractal": "sierpinski carpet s=3 k=8", "level": 9, "cells": F.cells, "coef": 0.1, "steps": steps,
           "tile_level": F.xtile_level}
    u = F.fill_uniform(2201)
    m0 = float(F.mass_f64(u))
    mean = m0 / F.cells
    for dtype, nbytes in (("f32", 8), ("bf16", 4)):
        if dtype == "f32":
            a, b = u.clone(), torch.empty_like(u)
            kw = {}
            offset = 0.0
        else:
            a = F.bf16_encode(u, mean)
            b = torch.empty_like(a)
            kw = {"rounding": "stochastic", "seed": 17}
            offset = mean
        F.diffuse_run(a, b, 2, 0.1, dtype=dtype, **kw)  # warm-up (result discarded)
        a = u.clone() if dtype == "f32" else F.bf16_encode(u, mean)
        nchk = max(1, (steps + MASS_EVERY - 1) // MASS_EVERY)
        work = torch.empty((nchk, MASS_WORK_DOUBLES), dtype=torch.float64, device=u.device)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        src, dst, done, r = a, b, 0, a
        for i in range(nchk):
            n = min(MASS_EVERY, steps - done)
            r = F.diffuse_run(src, dst, n, 0.1, dtype=dtype, first_step=done, **kw)
            if r is dst:
                src, dst = dst, src
            done += n
            F.mass_f64(r, dtype=dtype, offset=offset, work=work[i])
        e1.record()
        torch.cuda.synchronize()
        sec = e0.elapsed_time(e1) / 1e3
        drift = [(float(m) - m0) / m0 for m in work[:, 0].cpu()]
        res[dtype] = {"ms_per_step": sec * 1e3 / steps, "cell_updates_per_s": F.cells * steps / sec,
                      "algorithmic_gbs": nbytes * F.cells * steps / sec / 1e9,
                      "hbm_frac": nbytes * F.cells * steps / sec / 1e9 / HBM_PEAK_GBS,
                      "mass_every": MASS_EVERY, "mass_rel_drift": drift[-1],
                      "mass_rel_drift_max": max(drift, key=abs)}
        err = golden_error(torch, F, r, dtype, offset, steps)
        if err is not None:
            res[dtype]["rel_error_vs_binary64"] = err
        del a, b, r
    del u, F
    torch.cuda.empty_cache()
    return res


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=20,
                    help="untimed steps first, in the timed run's form")
    ap.add_argument("--level", type=int, default=16)
    ap.add_argument("--impl", default="auto", choices=["auto", "tile", "cell"])
    ap.add_argument("--form", default="auto", choices=["auto", "launches", "resident"],
                    help="run form of sqz_compact_run_form (auto: the library's choice for the step count)")
    ap.add_argument("--bb-steps", type=int, default=10)
    ap.add_argument("--r20-steps", type=int, default=20)
    ap.add_argument("--no-bb", action="store_true")
    ap.add_argument("--no-r20", action="store_true")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-batch", action="store_true")
    ap.add_argument("--no-diffusion", action="store_true")
    ap.add_argument("--no-carpet-life", action="store_true")
    ap.add_argument("--carpet-life-steps", type=int, default=30)
    ap.add_argument("--no-maps", action="store_true")
    ap.add_argument("--no-blocks", action="store_true")
    ap.add_argument("--blocks-steps", type=int, default=5)
    ap.add_argument("--maps-steps", type=int, default=10)
    ap.add_argument("--reps", type=int, default=10, help="further timed runs for mean / standard error")
    ap.add_argument("--batch-steps", type=int, default=50)
    ap.add_argument("--diffusion-steps", type=int, default=1000)
    ap.add_argument("--cpu-seconds", type=float, default=10.0)
    ap.add_argument("--cpu-max-steps", type=int, default=8)
    ap.add_argument("--copy-bytes", type=int, default=0,
                    help="only time a plain device copy of this many bytes (counter calibration)")
    ap.add_argument("--p", type=float, default=None, help="Bernoulli start density of --profile-run (default 0.5)")
    ap.add_argument("--profile-run", type=int, default=0,
                    help="only run the headline workload: one untimed and three timed runs of this many steps in "
                         "--form (every dispatch of a profiled kernel then has the same size)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only; --gpus {args.gpus} is not supported (the library has a "
              "sharding design but nothing here runs on more than one device)", file=sys.stderr)
        return 2

    import torch

    import paper_2201_00613_amd as sqz

    torch.cuda.set_device(0)
    if args.copy_bytes:
        src = torch.ones(args.copy_bytes, dtype=torch.uint8, device="cuda")
        dst = torch.empty_like(src)
        sec = time_steps(torch, lambda i: dst.copy_(src), args.steps, args.warmup)
        gbs = 2 * args.copy_bytes / (sec / args.steps) / 1e9
        print(json.dumps({"copy_bytes": args.copy_bytes, "ms_per_copy": sec * 1e3 / args.steps,
                          "gbs_read_plus_write": gbs}), flush=True)
        return 0
    seed, p, r = 2201, 0.5, args.level
    F = sqz.Fractal(*TRIANGLE, r)
    form = args.form
    if args.profile_run:
        pp = args.p if args.p is not None else p
        sec = [compact_run(torch, F, seed, pp, args.profile_run, args.profile_run, form=form)]
        sec += [compact_run(torch, F, seed, pp, args.profile_run, 0, form=form) for _ in range(2)]
        print(json.dumps({"profile_run": args.profile_run, "form": form, "level": r, "bernoulli_p": pp,
                          "ms_per_step": [x * 1e3 / args.profile_run for x in sec]}), flush=True)
        return 0
    if args.impl != "auto":
        used = "one step per launch"
    elif form == "resident" or (form == "auto" and F.auto_run_form(args.steps) == "resident"):
        used = "resident"
    else:
        used = "launches"
    log(f"[bench] triangle r={r}: {F.cells} cells, tile level {F.tile_level}, impl {args.impl}, run form {used}")
    # The comparison legs (the bounding-box baseline, the other run form, one step per
    # launch) run first: they are reported beside the headline, whose W warm-up and K
    # timed steps then find the device past its first work of the process (code
    # loaded, clocks up).
    bsec = bb_run(torch, F, seed, p, args.bb_steps, 2) if not args.no_bb else None
    other = None
    if used == "resident":
        other = ("launches", compact_run(torch, F, seed, p, args.steps, args.warmup, "auto", "launches"))
    elif used == "launches" and args.impl == "auto" and F.resident_run:
        other = ("resident", compact_run(torch, F, seed, p, args.steps, args.warmup, "auto", "resident"))
    s1 = None
    if args.impl == "auto" and F.run_steps_per_launch >= 2:
        s1 = compact_run(torch, F, seed, p, args.steps, args.warmup, "tile")
    # the warm-up steps run in the form the timed steps use (AUTO may pick the other
    # form for the W warm-up steps alone), so the timed call is not its kernel's first
    sec = compact_run(torch, F, seed, p, args.steps, args.warmup, args.impl,
                      used if used in ("resident", "launches") else form)
    ups = F.cells * args.steps / sec
    ms = sec * 1e3 / args.steps
    launches = {"resident": 1, "launches": run_launches(F, args.steps)}.get(used, args.steps)
    # algorithmic bytes per launch: each launch reads and writes every cell once
    gbs = BYTES_PER_UPDATE * F.cells * launches / sec / 1e9
    log(f"[bench] compact: {ms:.4f} ms/step ({launches} launches), {ups:.4e} cell-updates/s, "
        f"{gbs:.1f} GB/s algorithmic per launch")

    out = {
        "metric": METRIC, "value": ups, "unit": "cell-updates/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "u8", "data": "synthetic",
        "config": {"workload": f"sierpinski-triangle-r{r}-life-b3s23", "fractal": "sierpinski triangle s=2 k=3",
                   "level": r, "cells": F.cells, "bernoulli_p": p, "seed": seed, "impl": args.impl,
                   "run_form": used, "tile_level": F.tile_level, "launches": launches,
                   "steps_between_exchanges" if used == "resident" else "steps_per_launch":
                       STEPS_PER_LAUNCH[F.k] if used == "resident" else args.steps / launches,
                   "note": "2 x 43 MB working set is Infinity-Cache resident" if r == 16 else ""},
    }
    hbm = {"algorithmic_gbs_per_launch": gbs, "frac_of_hbm_peak": gbs / HBM_PEAK_GBS,
           # 2 B per cell-update over the step time: the bytes one-step launches would move
           "step_equivalent_gbs": BYTES_PER_UPDATE * F.cells * args.steps / sec / 1e9}
    profiles = {"resident": "k_slice_run_triangle_r16.md", "launches": "k_slice_triangle_r16.md"}
    profile = profiles.get(used)
    rec = profiled_counters(profile, out["config"]["workload"]) if profile else None
    note = "no committed counter profile for this kernel source and step count"
    out["roofline"] = counter_roofline(rec, args.steps, sec, launches, F.cells, profile)
    if not out["roofline"] and used == "resident":  # HBM is touched at the ends of the run only
        out["roofline"] = {"bound": "alu", "achieved": None, "peak": VALU_PEAK_G, "unit": "G VALU wave-instructions/s",
                           "frac": None, "traffic": None, "note": note}
    elif not out["roofline"]:
        out["roofline"] = {"bound": "hbm", "achieved": gbs, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                           "frac": gbs / HBM_PEAK_GBS, "traffic": None, "note": note}
    out["roofline"]["hbm"] = hbm
    if other and other[0] == "launches":
        sl = other[1]
        nl = run_launches(F, args.steps)
        out["launches_form"] = {"ms_per_step": sl * 1e3 / args.steps, "cell_updates_per_s": F.cells * args.steps / sl,
                                "launches": nl, "algorithmic_gbs_per_launch": BYTES_PER_UPDATE * F.cells * nl / sl / 1e9}
        rl = profiled_counters(profiles["launches"], out["config"]["workload"])
        roof = counter_roofline(rl, args.steps, sl, nl, F.cells, profiles["launches"])
        if roof:
            out["launches_form"]["roofline"] = roof
        log(f"[bench] {nl} launches: {sl * 1e3 / args.steps:.4f} ms/step")
    elif other and other[0] == "resident":
        sr = other[1]
        out["resident_form"] = {"ms_per_step": sr * 1e3 / args.steps, "cell_updates_per_s": F.cells * args.steps / sr,
                                "launches": 1}
        rr = profiled_counters(profiles["resident"], out["config"]["workload"])
        roof = counter_roofline(rr, args.steps, sr, 1, F.cells, profiles["resident"])
        if roof:
            out["resident_form"]["roofline"] = roof
        log(f"[bench] resident run: {sr * 1e3 / args.steps:.4f} ms/step")
    if s1 is not None:
        out["one_step_per_launch"] = {"ms_per_step": s1 * 1e3 / args.steps,
                                      "cell_updates_per_s": F.cells * args.steps / s1,
                                      "algorithmic_gbs": BYTES_PER_UPDATE * F.cells * args.steps / s1 / 1e9}
        log(f"[bench] one step per launch: {s1 * 1e3 / args.steps:.4f} ms/step")
    if args.reps > 0:
        out["repeats"] = repeat_stats(torch, F, seed, p, args.steps, args.reps, form)
    out["memory_reduction_factor"] = F.n * F.n / F.cells  # n^2 bytes expanded vs N bytes compact
    out["paper_context"] = {"hardware": "NVIDIA A100-40GB", "speedup_vs_bb": "~12x (level 16, its best block size)",
                            "memory_reduction_factor": "~315x at level 20; 99.8x at level 16 (rho = 1)",
                            "note": "the paper's figures, context only"}
    if bsec is not None:
        bb_ups = F.cells * args.bb_steps / bsec
        bb_ms = bsec * 1e3 / args.bb_steps
        log(f"[bench] bounding box: {bb_ms:.3f} ms/step, {bb_ups:.4e} useful cell-updates/s")
        out["bb"] = {"ms_per_step": bb_ms, "useful_cell_updates_per_s": bb_ups,
                     "expanded_cells_per_s": F.n * F.n * args.bb_steps / bsec,
                     "algorithmic_gbs": 2 * F.n * F.n / (bsec / args.bb_steps) / 1e9, "steps": args.bb_steps}
        out["speedup_vs_bb"] = ups / bb_ups
    if not args.no_blocks:
        out["block_layouts"] = bl = blocks_leg(torch, F, seed, p, args.blocks_steps)
        log("[bench] micro-blocks rho/ms: " + ", ".join(f"{d['rho']}:{d['ms_per_step']:.3f}" for d in bl["micro_blocks"]))
        log("[bench] lambda(omega) rho/ms: " + ", ".join(f"{d['rho']}:{d['ms_per_step']:.3f}" for d in bl["lambda_omega"]))
    if not args.no_maps:
        out["map_variants"] = m = maps_leg(torch, F, seed, p, args.maps_steps)
        log(f"[bench] maps scalar vs mfma: lambda {m['scalar']['lambda_ms']:.3f} / {m['mfma']['lambda_ms']:.3f} ms, "
            f"nu {m['scalar']['nu_ms']:.3f} / {m['mfma']['nu_ms']:.3f} ms, "
            f"cell Life {m['scalar']['life_ms_per_step']:.3f} / {m['mfma']['life_ms_per_step']:.3f} ms/step")
    del F
    torch.cuda.empty_cache()
    if not args.no_r20:
        F20 = sqz.Fractal(*TRIANGLE, 20)
        s20 = compact_run(torch, F20, seed, 0.3, args.r20_steps, 2)
        ms20 = s20 * 1e3 / args.r20_steps
        l20 = run_launches(F20, args.r20_steps)
        gbs20 = BYTES_PER_UPDATE * F20.cells * l20 / s20 / 1e9
        out["r20"] = {"cells": F20.cells, "steps": args.r20_steps, "launches": l20, "ms_per_step": ms20,
                      "memory_reduction_factor": F20.n * F20.n / F20.cells,
                      "repeats": repeat_stats(torch, F20, seed, 0.3, args.r20_steps, min(args.reps, 5)) if args.reps > 0 else None,
                      "ms_per_launch": s20 * 1e3 / l20, "cell_updates_per_s": F20.cells * args.r20_steps / s20,
                      "algorithmic_gbs_per_launch": gbs20, "hbm_frac": gbs20 / HBM_PEAK_GBS,
                      "step_equivalent_gbs": BYTES_PER_UPDATE * F20.cells * args.r20_steps / s20 / 1e9,
                      "bernoulli_p": 0.3}
        p20 = "k_slice_triangle_r20.md"
        roof = counter_roofline(profiled_counters(p20, "sierpinski-triangle-r20-life-b3s23"), args.r20_steps, s20, l20,
                                F20.cells, p20)
        if roof:
            out["r20"]["roofline"] = roof
        log(f"[bench] r=20: {ms20:.3f} ms/step, {l20} launches, {gbs20:.1f} GB/s per launch "
            f"({100 * gbs20 / HBM_PEAK_GBS:.1f}% of HBM peak)")
        del F20
        torch.cuda.empty_cache()
    if not args.no_batch:
        out["batch"] = batch_leg(torch, sqz, args.batch_steps)
        log(f"[bench] batch: {out['batch']['instances']} instances, {out['batch']['cells']} cells, "
            f"{out['batch']['ms_per_step']:.3f} ms/step, {out['batch']['cell_updates_per_s']:.3e} cell-updates/s")
    if not args.no_carpet_life:
        out["carpet_life"] = cl = carpet_life_leg(torch, sqz, args.carpet_life_steps)
        log(f"[bench] carpet r=9 Life: {cl['ms_per_step']:.4f} ms/step, {cl['cell_updates_per_s']:.3e} cell-updates/s "
            f"({cl['steps_per_launch']} steps per launch)")
    if not args.no_diffusion:
        out["diffusion"] = diffusion_leg(torch, sqz, args.diffusion_steps)
        d = out["diffusion"]
        log(f"[bench] diffusion carpet r=9: f32 {d['f32']['ms_per_step']:.4f} ms/step ({d['f32']['algorithmic_gbs']:.0f} GB/s), "
            f"bf16 {d['bf16']['ms_per_step']:.4f} ms/step ({d['bf16']['algorithmic_gbs']:.0f} GB/s)")
    if not args.no_cpu:
        out["cpu_baseline"] = cpu_baseline(r, seed, p, args.cpu_seconds, args.cpu_max_steps)
        log(f"[bench] cpu oracle: {out['cpu_baseline']['value']:.3e} cell-updates/s "
            f"on {out['cpu_baseline']['cores']} threads")
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
