"""Kernel-shape tuner for the FP32C particle kernel (targets per lane x workgroup size).

For each size bucket of single-set launches, and for the batched persistent launch of 64
uneven wakes, the library's own tuner (``vpm_autotune``) times every shape variant with HIP
events on wake-shaped inputs; all timings, and the library's own spread of the same sets as "0",
are written to a JSON cache keyed by the GPU architecture and a hash of the kernel sources, with
the fastest shape as the plan where it beats that spread by more than 1 % and 0 (no plan)
elsewhere.  The binding applies a matching cache (``vpm_set_plan``) when it first loads the library.

Usage (on the GPU):  python -m paper_2511_11430_amd.tune [--out PATH] [--quick]
"""
import argparse
import hashlib
import json
import os
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
DEFAULT_CACHE = os.path.join(HERE, "tune_cache.json")
# Up to 131072 targets the library's spread is no shape of the table, and its shorter FP32 sums are a
# reason of their own for it (u of 20000 flight particles 1.0e-7, 2.1e-7 in a shape), so these are not tuned.
TUNED_FROM = 131073
SINGLE_SIZES = [262144, 1048576]


def source_hash():
    h = hashlib.sha256()
    # the sources of the kernels being timed (the pair kernels and their device math)
    for f in ("pair_forward.hip", "device_math.h"):
        with open(os.path.join(HERE, "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


GAIN = 0.99  # a shape becomes the plan below this share of the own spread's time


def _plan(batched, n, x, g, s, off, reps, log):
    """Times every shape and the library's own spread of the sets: (variant or 0, {variant: ms})."""
    import torch

    from . import F32C, _lib, vpm_autotune, vpm_eval_velocity_stretching
    best, ms = vpm_autotune(x, g, s, src_off=off, reps=reps)
    _lib.load().vpm_set_plan(F32C, batched, n, n, 0)
    own = float("inf")
    for r in range(reps + 1):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        vpm_eval_velocity_stretching(x, g, s, src_off=off)
        e1.record()
        e1.synchronize()
        if r:  # (the first run is not timed)
            own = min(own, e0.elapsed_time(e1))
    times = {"0": own, **{str(v): t for v, t in enumerate(ms, 1)}}
    for v, t in times.items():
        log(f"{'batched' if batched else 'single'} N={n} variant {v}: {t:.3f} ms")
    return best if ms[best - 1] < GAIN * own else 0, times


def tune(out=DEFAULT_CACHE, quick=False, log=print):
    """Runs the library's tuner (vpm_autotune: HIP-event timings of every shape on the
    caller's stream) and times the library's own spread on forward-flight wakes of each size
    bucket and on the 64 uneven wakes of the batched launch, then writes the timings and
    choices to the JSON cache."""
    import numpy as np
    import torch

    from . import workloads as W

    dev = torch.device("cuda:0")
    f32 = lambda a: torch.tensor(np.ascontiguousarray(W.to_f32(a)), dtype=torch.float32, device=dev)
    plans = []
    sizes = SINGLE_SIZES[:1] if quick else SINGLE_SIZES
    for i, n in enumerate(sizes):
        c = W.config3(n=n)
        x, g, s = f32(c["x"]), f32(c["gamma"]), f32(c["sigma"])
        best, ms = _plan(0, n, x, g, s, None, 2 if n >= 262144 else 3, log)
        lo = sizes[i - 1] + 1 if i > 0 else TUNED_FROM
        hi = sizes[i] if i + 1 < len(sizes) else 1 << 31
        plans.append({"batched": 0, "n_lo": lo, "n_hi": hi, "variant": best, "ms": ms, "n": n})
        del x, g, s
    # batched persistent launch over the 64 uneven wakes
    wakes = W.config5(scale=0.25 if quick else 1.0)
    off = [0]
    for w in wakes:
        off.append(off[-1] + w["x"].shape[1])
    cat = lambda k: np.concatenate([W.to_f32(w[k]) for w in wakes], axis=-1)
    xw = torch.tensor(cat("x"), dtype=torch.float32, device=dev)
    gw = torch.tensor(cat("gamma"), dtype=torch.float32, device=dev)
    sw = torch.tensor(cat("sigma"), dtype=torch.float32, device=dev)
    best, ms = _plan(1, off[-1], xw, gw, sw, off, 2, log)
    plans.append({"batched": 1, "n_lo": 0, "n_hi": 1 << 31, "variant": best, "ms": ms,
                  "n": off[-1]})
    props = torch.cuda.get_device_properties(0)
    cache = {"arch": getattr(props, "gcnArchName", "gfx950").split(":")[0], "device": props.name,
             "hip": torch.version.hip, "source_hash": source_hash(), "created": time.strftime("%Y-%m-%d %H:%M:%S"),
             "plans": plans}
    with open(out, "w") as f:
        json.dump(cache, f, indent=1)
    apply_cache(out)
    return cache


def apply_cache(path=None):
    """Apply a tuning cache to the loaded library if it matches the kernel sources; returns the
    number of plans applied (0 if none or stale)."""
    from . import F32C, _lib
    path = path or os.environ.get("VPM_TUNE_CACHE", DEFAULT_CACHE)
    try:
        with open(path) as f:
            cache = json.load(f)
    except (OSError, ValueError):
        return 0
    if cache.get("source_hash") != source_hash():
        return 0
    lib = _lib.load()
    n = 0
    for p in cache.get("plans", []):
        if lib.vpm_set_plan(F32C, int(p["batched"]), int(p["n_lo"]), int(p["n_hi"]), int(p["variant"])) == 0:
            n += 1
    return n


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--out", default=DEFAULT_CACHE)
    ap.add_argument("--quick", action="store_true")
    args = ap.parse_args()
    cache = tune(args.out, args.quick, log=lambda m: print(m, flush=True))
    print(json.dumps({p["n"]: p["variant"] for p in cache["plans"]}), flush=True)


if __name__ == "__main__":
    sys.exit(main())
