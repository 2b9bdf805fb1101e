"""Measured problems behind the limits of strips (strips_choice, strip_tiles_choice and row_strip_tiles_choice in csrc/hgemm_api.hip).

    python -m paper_2512_02551_amd.strips gather --seed 1 --count 4000 --against LIB --out FILE    # on the GPU; FILE: lines to add to a check file
    python -m paper_2512_02551_amd.strips evaluate [FILE ...]                       # CPU; the built library's choices, by range

csrc/strips_check.jsonl.gz holds 12000 problems (seed 1) of 1 to 320 rows of A on both sides of the limits, half of round sizes as layers have them, a
fifth with padded rows of B: {"shape": [M, N, K], "tn", "ldb", "before": kernel, "strips": kernel, "us": [[before, strips] from HBM, from the cache]}.
"before" is the choice of a build without strips (--against: one of commit 8df821b), "strips" what the tile rule gives with its limits left out.
Both are timed in turn by their specs in the built library; shapes of the dispatch tables, calls that share a launch and problems that "before"
ran on strips of 16 rows of B already are left out.
"""
from __future__ import annotations

import argparse
import ctypes
import gzip
import json
import math
import os

from .few_rows import number

_HERE = os.path.dirname(os.path.abspath(__file__))
CHECK = os.path.join(_HERE, "csrc", "strips_check.jsonl.gz")
CUS = 256
WIDTHS = [512, 640, 768, 896, 1024, 1152, 1280, 1408, 1536, 1664, 1792, 1920, 2048, 2304, 2560, 2816, 3072, 3328, 3584, 3840, 4096, 4352, 4608, 5120, 5504,
          5632, 6144, 6400, 6656, 7168, 7680, 8192, 9216, 10240, 11008, 11264, 12288]


def strips_spec(M, N, K, tn):
    """The tile rule without its limits; None where one workgroup for every compute unit does not cover the problem."""
    if not tn:
        strips = -(-N // 32)
        mr = 16 if -(-M // 16) * strips <= CUS else 32 if M > 32 and -(-M // 32) * strips <= CUS else 0
        return f"skinny,sk=1,nr=32,mr={mr}" if M > 16 and mr else None
    if M <= 16 or (M <= 32 and (K < 1024 or K > 6144 or -(-M // 16) * -(-N // 16) > CUS)):
        nr = 16 * -(-N // 4096)
        return None if nr > 48 or N % 16 else "skinny,sk=1" + (f",nr={nr}" if nr > 16 else "")
    best = None
    for a in range(16, min(64, M + 15) + 1, 16):
        for b in range(16, 65, 16):
            if -(-M // a) * -(-N // b) <= CUS and a + b <= 96 and (best is None or (a + b, abs(a - b)) < (sum(best), abs(best[0] - best[1]))):
                best = (a, b)
    return f"skinny,sk=1,nr={best[1]},mr={best[0]}" if best else None


def problem(rng):
    def size(lo, hi, step=1):
        return int(min(max(round(lo * (hi / lo) ** rng.random() / step) * step, lo), hi))

    def width(lo, hi):
        kind = rng.random()
        return rng.choice([w for w in WIDTHS if lo <= w <= hi]) if kind < 0.5 else size(lo, hi, 64) if kind < 0.7 else size(lo, hi, 8)

    kind = rng.random()
    if kind < 0.3:
        M, N, K, tn = size(17, 320), width(64, 8192), width(640, 3072), False
    elif kind < 0.65:
        M, N, K, tn = size(17, 320), width(64, 8192), width(896, 7168), True
    else:
        M, N, K, tn = size(1, 32), width(64, 12288), width(256, 12288) if rng.random() < 0.6 else size(4096, 32768, 64), True
    return M, N, K, tn, ((K if tn else N) + 8 * rng.randint(1, 64)) if rng.random() < 0.2 else 0


def gather(seed: int, count: int, against: str, path: str):
    import random

    import torch

    import paper_2512_02551_amd as hg

    hg.load()
    other = ctypes.CDLL(os.path.abspath(against))
    sh = torch.cuda.current_stream().cuda_stream
    rng = random.Random(seed)
    pool = torch.randn(1 << 26, device="cuda").mul_(0.02).half().repeat(12)
    c = torch.empty(1 << 22, dtype=torch.float16, device="cuda")

    def timed(p, sets, reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        p.run_many(reps, sets, sh)
        e1.record()
        e1.synchronize()
        return e0.elapsed_time(e1) / reps * 1e3

    done = 0
    with open(path, "w") as f:
        while done < count:
            M, N, K, tn, ldb = problem(rng)
            lay = hg.Layouts.make(b_col_major=tn, ldb=ldb)
            text, i64 = ctypes.create_string_buffer(512), ctypes.c_int64
            assert other.hgemm_plan_choice(i64(M), i64(N), i64(K), ctypes.byref(lay), text, ctypes.c_size_t(512)) == 0
            source, before = text.value.decode().split(": ", 1)
            strips = strips_spec(M, N, K, tn)
            joins = "sk=1," in before and before.startswith("mfma") and "ph=1" not in before and 2 * (M * K + K * N + M * N) <= 8 << 20
            if source == "table" or strips is None or joins or (tn and before.startswith("skinny") and "ra=1" not in before):
                continue
            rows = (N if tn else K) * (ldb or (K if tn else N))
            elems = (M * K + 127) // 128 * 128 + (rows + 127) // 128 * 128
            n = max(1, min(64, pool.numel() // elems, int(6e8 // (2 * elems)) + 1))
            if n * elems > pool.numel():
                continue
            assert M * N <= c.numel(), (M, N, K)
            sets = [(pool.data_ptr() + 2 * i * elems, pool.data_ptr() + 2 * (i * elems + (M * K + 127) // 128 * 128), c.data_ptr()) for i in range(n)]
            plans = [hg.Plan(M, N, K, lay, s) for s in (before, strips)]
            reps = max(4, min(48, int(400 / timed(plans[0], sets, 6))))
            us = []
            for some in (sets, sets[:1]):
                times = [[], []]
                for r in range(6):
                    for k in (0, 1) if r % 2 else (1, 0):
                        times[k].append(timed(plans[k], some, reps))
                us.append([round(sorted(t[1:])[2], 2) for t in times])
            for p in plans:
                p.destroy()
            f.write(json.dumps({"shape": [M, N, K], "tn": tn, "ldb": ldb, "before": before, "strips": strips, "us": us}) + "\n")
            done += 1
            if done % 500 == 0:
                f.flush()
                print(f"{done} problems", flush=True)


def load(paths):
    rows = []
    for p in paths:
        with (gzip.open(p, "rt") if p.endswith(".gz") else open(p)) as f:
            rows += [json.loads(line) for line in f]
    return rows


def takes(r):
    """Does the built library run the problem on strips?"""
    import paper_2512_02551_amd as hg

    return hg.plan_choice(*r["shape"], hg.Layouts.make(b_col_major=r["tn"], ldb=r["ldb"])).split(": ", 1)[1] == r["strips"]


def figures(rows):
    """(problems, strips over before from HBM and from the cache, slower by 3 % from HBM and from the cache, by 10 %)"""
    ratio = [[r["us"][w][1] / r["us"][w][0] for r in rows] for w in (0, 1)]
    return (len(rows), *(round(math.exp(sum(map(math.log, x)) / len(x)), 3) for x in ratio), *(sum(v > 1.03 for v in x) for x in ratio), *(sum(v > 1.1 for v in x) for x in ratio)) if rows else (0,)


def evaluate(rows):
    kinds = {"row-major B": lambda r: not r["tn"], "column-major B, blocks of rows": lambda r: r["tn"] and "mr=" in r["strips"], "column-major B, all rows": lambda r: r["tn"] and "mr=" not in r["strips"]}
    print("problems, strips / before from HBM, from the cache, slower by more than 3 % from HBM, from the cache, by 10 % from HBM, from the cache")
    for name, kind in kinds.items():
        some = [r for r in rows if kind(r)]
        taken = {id(r): takes(r) for r in some}
        print(f"{name}: taken {figures([r for r in some if taken[id(r)]])}, left {figures([r for r in some if not taken[id(r)]])}")
        tile = lambda r: number(r["strips"], "mr") + number(r["strips"], "nr") if "mr=" in r["strips"] else -(-r["shape"][1] // 4096)      # noqa: E731
        step = 512 if "mr=" in some[0]["strips"] else 2048
        for key in sorted({(tile(r), r["shape"][2] // step) for r in some}):
            part = [r for r in some if (tile(r), r["shape"][2] // step) == key]
            if len(part) >= 10:
                print(f"  {'rows of A and B' if step == 512 else 'blocks of 4096 columns'} {key[0]}, K {key[1] * step}-: taken {figures([r for r in part if taken[id(r)]])}, left {figures([r for r in part if not taken[id(r)]])}")


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    sub = ap.add_subparsers(dest="cmd", required=True)
    g_ = sub.add_parser("gather")
    g_.add_argument("--seed", type=int, required=True)
    g_.add_argument("--count", type=int, required=True)
    g_.add_argument("--against", required=True, metavar="LIB")
    g_.add_argument("--out", required=True)
    e_ = sub.add_parser("evaluate")
    e_.add_argument("files", nargs="*", default=[CHECK])
    args = ap.parse_args()
    if args.cmd == "gather":
        gather(args.seed, args.count, args.against, args.out)
    else:
        evaluate(load(args.files))
