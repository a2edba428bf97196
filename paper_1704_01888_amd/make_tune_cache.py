"""Tune the sweep shapes of this GPU and write them as a cache file.

    python -m paper_1704_01888_amd.make_tune_cache [path]

For every lattice side with a choice of shapes up to 256 and the population
classes 1-3 (R_cap from 2^11 to 2^14, 2^14 to 2^17, above), `Context.tune`
times every shape on a run of R = 8000, 50000 or 200000 replicas (theta = 10):
with q = 10 for the four-site kernel, with q = 40 for what that does not take
(left out where the shape is the same).
From 96x96 on 1500 replicas fill the GPU: those sides have class 0 too.  The
fastest shape becomes the entry, but one that the file already has stays if it
is within 6 % of the fastest: launches that end in a partial round of waves
differ by as much between neighbouring populations of one class.  The entries
go to `path` (by default the package's cache file beside this module, which
`Context` loads when it is created; lines of other architectures in it are
kept).  Classes of 200000 replicas are skipped where a population buffer would
exceed 16 GB.
"""
from __future__ import annotations

import json
import os
import sys

from . import Context, tune_cache_path

SIDES = (8, 12, 16, 20, 24, 32, 48, 64, 96, 128, 192, 256)
POPULATIONS = (1500, 8000, 50000, 200000)
STATES = (10, 40)
KEEP = 0.94


def main(path: str | None = None) -> str:
    import torch

    ctx = Context(0, tune_cache=False)
    arch = torch.cuda.get_device_properties(ctx.device).gcnArchName.split(":")[0]
    path = path or tune_cache_path(ctx.device)
    lines = [json.loads(ln) for ln in open(path) if ln.strip()] if os.path.exists(path) else []
    had = {(e["L"], e["q_large"], e["r_class"]): (e["lanes"], e["waves_per_block"]) for e in lines if e["arch"] == arch}
    lines = [e for e in lines if e["arch"] != arch]
    quads = set()
    for L in SIDES:
        for q in STATES:
            for R in POPULATIONS:
                if R * L * L > 16 << 30 or (R < 2048 and L < 96):
                    continue
                e = ctx.tune(L, q, R)
                for t in e["timed"]:
                    if (t["lanes"], t["waves_per_block"]) == had.get((L, e["q_large"], e["r_class"]), had.get((L, 0, e["r_class"]))) and \
                            t["attempts_per_ns"] >= KEEP * e["attempts_per_ns"]:
                        e = t
                shape = tuple(e[k] for k in ("r_class", "lanes", "waves_per_block"))
                line = {"arch": arch, **{k: e[k] for k in ("L", "q_large", "r_class", "lanes", "waves_per_block")},
                        "attempts_per_ns": round(e["attempts_per_ns"], 3)}
                print(json.dumps(line), flush=True)
                if q <= 32:
                    quads.add((L, *shape))
                elif (L, *shape) in quads:      # (the entry of q_large 0 serves it)
                    continue
                lines.append(line)
    with open(path, "w") as f:
        f.writelines(json.dumps(e) + "\n" for e in lines)
    ctx.close()
    return path


if __name__ == "__main__":
    print(main(sys.argv[1] if len(sys.argv) > 1 else None), file=sys.stderr)
