#!/usr/bin/env python3
"""Tile-shape search for the kernel families of libli.so.

For each family and table slot, every compiled candidate is forced in turn
(li_tune_force) and the ordinary entry point is timed with HIP events on
the current stream (1 warm-up, then the mean of `reps` calls); the fastest
candidate is written to the table (li_tune_set) and the table is saved as
text (li_tune_save), which li.py loads at import.  The table that comes with
the library has entries for the 16-bit products only: the FP32 products, the
symmetric contractions and the batches go by the measured rules of
csrc/tune.cpp, which searched entries override (an entry of the FP32 products
holds for every reduction length of its output size).  They are searched only
when --only names them.

Representative problems per table slot (li_tune_key:
the GEMM families key by the output's area, which for the square problems
searched here is the bit length of the side; the symmetric contractions by
the order of the result and the class of the reduction length): square
GEMMs 256 .. 8192, the 2048^4 two-GEMM chain's shape, covariance of
M = 128 .. 4096 features with N = M, 2 M, 4 M and 8 M samples, syrk of
order 256 .. 4096 with rank N / 4, N, 4 N and 16 N, and square
reduced-precision GEMMs.  For the grouped plans, the shape class per
bucket is searched on plans of 64 rectangular problems of one kind with
sizes drawn log-uniform inside the bucket (32 to 1024, the batch's range):
each class is forced while the plan is built and the graph launch is
timed.

Usage: python -m paper_2312_13170_amd.autotune [--out PATH] [--quick] [--only FAMILIES]
"""
import argparse
import json
import os
import sys

import torch

HERE = os.path.dirname(os.path.abspath(__file__))
if os.path.dirname(HERE) not in sys.path:
    sys.path.insert(0, os.path.dirname(HERE))

from paper_2312_13170_amd import li, synth  # noqa: E402


def time_call(fn, reps):
    fn()
    torch.cuda.synchronize()
    s = torch.cuda.Event(enable_timing=True)
    e = torch.cuda.Event(enable_timing=True)
    s.record()
    for _ in range(reps):
        fn()
    e.record()
    torch.cuda.synchronize()
    return s.elapsed_time(e) / reps


def gemm_case(n):
    A = torch.from_numpy(synth.uniform_pm1(90, "A", (n, n))).cuda()
    B = torch.from_numpy(synth.uniform_pm1(90, "B", (n, n))).cuda()
    C = torch.from_numpy(synth.uniform_pm1(90, "C", (n, n))).cuda()
    return (n, n, n), lambda: li.li_gemm(n, n, n, 1.5, A, B, 1.2, C)


def syrk_case(m, n):
    X = torch.from_numpy(synth.uniform_pm1(91, "X", (n, m))).cuda()
    Y = torch.empty_like(X)
    mean = torch.empty(m, dtype=torch.float64, device="cuda")
    cov = torch.empty((m, m), device="cuda")
    ws = torch.empty(li.li_stats_workspace_bytes(m, n) // 8 + 1, dtype=torch.float64, device="cuda")
    return (m, m, n), lambda: li.li_covariance(m, n, X, Y, mean, cov, ws)


def lp_case(n, prec):
    A = torch.from_numpy(synth.uniform_pm1(92, "A", (n, n))).cuda()
    B = torch.from_numpy(synth.uniform_pm1(92, "B", (n, n))).cuda()
    C = torch.empty((n, n), device="cuda")
    ws = torch.empty(li.li_gemm_ex_workspace_bytes(n, n, n, prec) // 4 + 1, device="cuda")
    return (n, n, n), lambda: li.li_gemm_ex(n, n, n, 1.0, A, B, 0.0, C, prec, ws)


def rank_case(n, k):
    A = torch.from_numpy(synth.uniform_pm1(93, "A", (n, k))).cuda()
    C = torch.from_numpy(synth.uniform_pm1(93, "C", (n, n))).cuda()
    ws = torch.empty(li.li_syrk_workspace_bytes(n, k) // 4 + 1, device="cuda")
    return (n, n, k), lambda: li.li_syrk(n, k, 1.5, A, 1.2, C, ws)


def warm_up(fn, seconds=0.5):
    """Run until the GPU has left its idle clocks, so the first candidates
    are not timed at a lower clock than the last."""
    import time
    t0 = time.perf_counter()
    while time.perf_counter() - t0 < seconds:
        for _ in range(10):
            fn()
        torch.cuda.synchronize()


def search(kernel, cases, reps, log, passes=2):
    for label, (shape, fn) in cases:
        slot = li.li_tune_key(kernel, *shape)
        n = li.li_tune_num_candidates(kernel)
        warm_up(fn)
        # every candidate timed in `passes` sweeps, the best sweep kept, so
        # clock drift during a sweep does not decide the winner
        times = {}
        for p in range(passes):
            order = range(n) if p % 2 == 0 else range(n - 1, -1, -1)
            for idx in order:
                li.li_tune_force(kernel, idx)
                t = time_call(fn, reps)
                times[idx] = min(times.get(idx, t), t)
        li.li_tune_force(kernel, -1)
        best = min(times, key=times.get)
        li.li_tune_set(kernel, slot, best)
        rec = {"kernel": kernel, "case": label, "slot": slot, "best": best,
               "candidate": li.li_tune_candidate(kernel, best),
               "ms": {str(k): round(v, 4) for k, v in times.items()}}
        log.append(rec)
        print(json.dumps(rec), flush=True)


def grouped_problems(kind, bucket, count=64, seed=94):
    """`count` problems of one kind whose sizes lie in one bucket (bit length
    `bucket` of the largest size), drawn log-uniform in [2^(b-1), 2^b) and
    clipped to the batch range [32, 1024]; returns the problems and the
    buffers they point to."""
    import numpy as np
    lo, hi = max(32, 1 << (bucket - 1)), min(1024, (1 << bucket) - 1)
    rng = np.random.default_rng(seed + bucket + 17 * kind)

    def draw():
        return int(min(hi, max(lo, round(float(np.exp(rng.uniform(np.log(lo), np.log(hi + 1))))))))

    keep, probs = [], []
    for t in range(count):
        if kind == li.LI_PROBLEM_GEMM:
            M, N, K = draw(), draw(), draw()
            A = torch.from_numpy(synth.uniform_pm1(seed, "A%d" % t, (M, K))).cuda()
            B = torch.from_numpy(synth.uniform_pm1(seed, "B%d" % t, (K, N))).cuda()
            C = torch.from_numpy(synth.uniform_pm1(seed, "C%d" % t, (M, N))).cuda()
            keep += [A, B, C]
            probs.append(li.make_problem(kind, M, N, K, 1.5, 1.2, A, B, C))
        else:
            M, N = draw(), draw()
            X = torch.from_numpy(synth.uniform_pm1(seed, "X%d" % t, (N, M))).cuda()
            Y = torch.empty_like(X)
            mean = torch.empty(M, dtype=torch.float64, device="cuda")
            cov = torch.empty((M, M), device="cuda")
            keep += [X, Y, mean, cov]
            probs.append(li.make_problem(kind, M, N, 0, 1.0, 0.0, X, None, cov, Y, mean))
    return probs, keep


def search_grouped(kernel, kind, buckets, reps, log, passes=2):
    """Shape class per size bucket for the grouped plans: a plan of problems
    of that bucket is built with each class forced and its graph launch
    timed."""
    for bucket in buckets:
        probs, keep = grouped_problems(kind, bucket)
        n = li.li_tune_num_candidates(kernel)
        times = {}
        for p in range(passes):
            for idx in (range(n) if p % 2 == 0 else range(n - 1, -1, -1)):
                li.li_tune_force(kernel, idx)
                plan = li.li_group_plan_create(probs)
                li.li_tune_force(kernel, -1)
                warm_up(plan.launch, 0.2)
                t = time_call(plan.launch, reps)
                plan.close()
                times[idx] = min(times.get(idx, t), t)
        best = min(times, key=times.get)
        li.li_tune_set(kernel, bucket, best)
        rec = {"kernel": kernel, "case": "grouped %s bucket %d" % ("gemm" if kind == 0 else "cov", bucket),
               "bucket": bucket, "best": best, "candidate": li.li_tune_candidate(kernel, best),
               "ms": {str(k): round(v, 4) for k, v in times.items()}}
        log.append(rec)
        print(json.dumps(rec), flush=True)
        del keep


# the families whose choices the table holds; those of the others are rules
DEFAULT_FAMILIES = "lp"


def parser():
    p = argparse.ArgumentParser()
    p.add_argument("--out", default=os.path.join(HERE, "tune_gfx950.txt"))
    p.add_argument("--log", default=None, help="also write the timings as JSON lines")
    p.add_argument("--quick", action="store_true", help="fewer sizes and repetitions")
    p.add_argument("--only", default=DEFAULT_FAMILIES,
                   help="comma list of the families to search (gemm, syrk, rows, lp, grouped); "
                        "the table's other entries are kept as loaded, and searched entries of "
                        "the others than lp override the measured rules (default: %(default)s)")
    return p


def main():
    a = parser().parse_args()
    only = set(a.only.split(","))
    torch.cuda.set_device(0)
    li.li_init()
    reps = 3 if a.quick else 10
    log = []
    if "gemm" in only:
        gsizes = [512, 2048] if a.quick else [256, 512, 1024, 2048, 4096, 8192]
        search(li.LI_KERNEL_GEMM_F32, [("gemm %d" % n, gemm_case(n)) for n in gsizes], reps, log)
    if "syrk" in only:
        ssizes = [512, 2048] if a.quick else [128, 256, 512, 1024, 2048, 4096]
        ratios = [1, 2] if a.quick else [1, 2, 4, 8]
        search(li.LI_KERNEL_SYRK_F32, [("cov M=%d N=%d" % (m, r * m), syrk_case(m, r * m))
                                       for m in ssizes for r in ratios], reps, log)
    if "rows" in only:
        rsizes = [1024, 2048] if a.quick else [256, 512, 1024, 2048, 4096]
        ranks = [(1, 1)] if a.quick else [(1, 4), (1, 1), (4, 1), (16, 1)]
        search(li.LI_KERNEL_SYRK_ROWS, [("syrk N=%d K=%d" % (n, n * p // q), rank_case(n, n * p // q))
                                        for n in rsizes for p, q in ranks], reps, log)
    if "lp" in only:
        lsizes = [2048, 8192] if a.quick else [1024, 2048, 4096, 8192]
        search(li.LI_KERNEL_GEMM_LP, [("bf16 %d" % n, lp_case(n, "bf16")) for n in lsizes], reps, log)
        search(li.LI_KERNEL_GEMM_LP_SPLIT, [("bf16x3 %d" % n, lp_case(n, "bf16x3")) for n in lsizes], reps,
               log)
    if "grouped" in only:
        # grouped plans: the batch draws sizes in [32, 1024], buckets 6 to 11
        gb = [7, 9, 11] if a.quick else [6, 7, 8, 9, 10, 11]
        search_grouped(li.LI_KERNEL_GROUPED_GEMM, li.LI_PROBLEM_GEMM, gb, reps, log)
        search_grouped(li.LI_KERNEL_GROUPED_COV, li.LI_PROBLEM_COVARIANCE, gb, reps, log)
    li.li_tune_save(a.out)
    if a.log:
        with open(a.log, "w") as f:
            for r in log:
                f.write(json.dumps(r) + "\n")
    print("table written to", a.out, flush=True)


if __name__ == "__main__":
    main()
