"""Timings behind the automatic choice of a product's launch.

The choice (choose_gemm in csrc/api.cpp) takes the entry with the smallest
estimated time; the estimates' constants (kSplit in csrc/gemm_split.hip and
gemm_mfma_us in csrc/gemm_mfma.hip) describe an MI355X.  ``measure`` times every
entry on every shape of ``shapes()`` (graph-replayed, so without the host's
part) and writes one CSV row per shape; ``check`` compares the present choice
and the present estimates with such a file, which needs no GPU:

    python perf/gemm_choice.py measure profiles/gemm_choice_timings.csv
    python perf/gemm_choice.py check profiles/gemm_choice_timings.csv

After a change to a kernel: measure, adjust the entry's constants until
``check`` shows no shape far behind its best entry, and keep the new file.
"""
from __future__ import annotations

import csv
import ctypes
import math
import os
import random
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

from paper_2502_19405_amd import repops  # noqa: E402

CUS = 256  # compute units of an MI355X
LARGE = (0, 2, 5, 8, 9)  # entries of gemm_mfma.hip that the choice knows or knew
FIELDS = ("m", "n", "k", "batch", "ta", "tb", "causal")


def shapes(count: int = 520, seed: int = 1):
    """Products of the package's workloads and their ragged neighbours: small
    squares, few rows (decoding), linear layers and their gradients, attention's
    batched and causal products."""
    rng = random.Random(seed)

    def log(lo, hi):
        return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))

    dims = [(768, 3072), (3072, 768), (768, 768), (4096, 4096), (4096, 14336), (14336, 4096)]
    out = []
    while len(out) < count:
        kind = rng.choice(["any", "small", "decode", "layer", "layer", "grad", "scores", "scores",
                           "values", "values", "values", "short"])
        s = dict(m=1, n=1, k=1, batch=1, ta=0, tb=0, causal=0)
        if kind == "any":
            s.update(m=log(1, 4096), n=log(1, 14336), k=log(1, 14336), ta=rng.randint(0, 1),
                     tb=rng.randint(0, 1), batch=rng.choice([1, 1, 1, 3, 8]))
        elif kind == "small":
            s.update(m=log(64, 2048), n=log(64, 2048), k=log(64, 2048), ta=rng.randint(0, 1),
                     tb=rng.randint(0, 1))
        elif kind == "decode":
            k, n = rng.choice(dims)
            s.update(m=log(1, 64), n=n, k=k, tb=rng.randint(0, 1))
        elif kind == "layer":
            k, n = rng.choice(dims)
            s.update(m=log(16, 4096), n=n, k=k, tb=rng.randint(0, 1))
        elif kind == "grad":
            m, n = rng.choice(dims)
            s.update(m=m, n=n, k=log(16, 4096), ta=1)
        elif kind == "short":
            s.update(m=log(64, 4096), n=log(64, 8192), k=rng.choice([32, 64, 96, 128, 192, 256]),
                     tb=rng.randint(0, 1), batch=rng.choice([1, 1, 4, 12]))
        else:
            heads, d = rng.choice([(12, 64), (32, 128)])
            seq, batch = log(16, 1024), heads * rng.randint(1, 4)
            step = rng.choice([1, 16, 64])
            seq = max(step, seq // step * step)
            if kind == "scores":
                s.update(m=seq, n=seq, k=d, batch=batch, tb=1, causal=rng.choice([0, 1, 1]))
            else:
                s.update(m=seq, n=d, k=seq, batch=batch, causal=rng.choice([0, 2, 2]))
        elements = s["batch"] * (s["m"] * s["k"] + s["k"] * s["n"] + s["m"] * s["n"])
        if 2 * s["batch"] * s["m"] * s["n"] * s["k"] <= 3e11 and elements <= 1 << 28:
            out.append(s)
    return out


def _args(s):
    i64, i32 = ctypes.c_int64, ctypes.c_int32
    return (ctypes.byref(repops.Order().c()), i64(s["batch"]), i64(s["m"]), i64(s["n"]),
            i64(s["k"]), i64(s.get("lda") or (s["m"] if s["ta"] else s["k"])), i32(s["ta"]),
            i64(s.get("ldb") or (s["k"] if s["tb"] else s["n"])), i32(s["tb"]), i32(s["causal"]),
            i32(s.get("cus", CUS)))


def choice(s):
    """(kind, index) of REPOPS_LAUNCH_AUTO for a shape (dense rows unless it names
    lda or ldb) on a device of CUS compute units."""
    kind, index = ctypes.c_uint32(), ctypes.c_uint32()
    repops.load().repops_internal_gemm_choice(*_args(s), ctypes.byref(kind), ctypes.byref(index))
    return kind.value, index.value


def estimate(s, index):
    """Estimated us of matrix-core entry `index`; 0 where the choice does not
    offer it."""
    fn = repops.load().repops_internal_gemm_estimate
    fn.restype = ctypes.c_double
    return fn(*_args(s), ctypes.c_uint32(index))


def measure(path):
    import torch

    names = repops.gemm_configs(repops.LAUNCH_GEMM_MFMA)
    entries = [i for i, n in enumerate(names) if i in LARGE or "/k" in n]
    gen = torch.Generator(device="cuda:0").manual_seed(0)

    def tensor(*size):
        return torch.randn(*size, device="cuda:0", generator=gen)

    def graph_us(call, once):
        reps = max(1, min(64, int(400 / once)))
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(reps):
                call()
        # Long enough for the clock to settle where this kernel holds it (a few
        # replays after something else run up to 10% off, more for some entries).
        times, spent = [], 0.0
        while spent < 15.0 or len(times) < 4:
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            g.replay()
            b.record()
            b.synchronize()
            spent += a.elapsed_time(b)
            times.append(a.elapsed_time(b) * 1e3 / reps)
        late = sorted(times[len(times) // 2:])
        return late[len(late) // 2]

    big = tensor(4096, 4096)
    out = torch.empty_like(big)
    with open(path, "w", newline="") as f:
        w = csv.writer(f)
        w.writerow([*FIELDS, *[names[i] for i in entries]])
        for at, s in enumerate(shapes()):
            m, n, k, b = s["m"], s["n"], s["k"], s["batch"]
            A, B, C = tensor(b, m * k), tensor(b, k * n), torch.empty(b, m * n, device="cuda:0")
            lda, ldb = (m if s["ta"] else k), (k if s["tb"] else n)
            sa, sb, sc = (0, 0, 0) if b == 1 else (m * k, k * n, m * n)
            best = {}
            for _ in range(2):
                for _ in range(8):  # the clock falls between shapes
                    repops.matmul(big, big, out=out)
                for i in entries:
                    launch = repops.Launch(repops.LAUNCH_GEMM_MFMA, (i,))

                    def call():
                        repops.bmm_raw(b, 1, m, n, k, A, sa, 0, lda, s["ta"], B, sb, 0, ldb, s["tb"],
                                       1.0, C, sc, 0, n, launch=launch, causal=s["causal"])
                    call()
                    x, y = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                    x.record()
                    call()
                    y.record()
                    y.synchronize()
                    best[i] = min(best.get(i, math.inf), graph_us(call, x.elapsed_time(y) * 1e3))
            w.writerow([*[s[x] for x in FIELDS], *["%.2f" % best[i] for i in entries]])
            f.flush()
            print(at, s, flush=True)


def recorded(path):
    """[(shape, {entry index: us})] of a measured file."""
    index = {n: i for i, n in enumerate(repops.gemm_configs(repops.LAUNCH_GEMM_MFMA))}
    with open(path, newline="") as f:
        return [({x: int(row[x]) for x in FIELDS},
                 {index[n]: float(v) for n, v in row.items() if n in index})
                for row in csv.DictReader(f)]


def check(path):
    rows = recorded(path)
    names = repops.gemm_configs(repops.LAUNCH_GEMM_MFMA)
    loss, off, taken = [], {}, {}
    for s, us in rows:
        _, index = choice(s)
        loss.append((us[index] / min(us.values()), s, index, min(us, key=us.get), us))
        taken[index] = taken.get(index, 0) + 1
        for i, t in us.items():
            e = estimate(s, i)
            if e > 0 and t < 1.5 * min(us.values()):  # where the estimate matters
                off.setdefault(i, []).append(abs(e / t - 1))
    loss.sort(key=lambda x: -x[0])
    print("time of the chosen entry over the best one: geometric mean %.3f, above 1.1: %d of %d" % (
        math.exp(sum(math.log(x[0]) for x in loss) / len(loss)), sum(x[0] > 1.1 for x in loss),
        len(loss)))
    for r, s, index, best, us in loss[:20]:
        print("  %.2f  %s  %s %.1f us, best %s %.1f us" % (r, s, names[index], us[index],
                                                          names[best], us[best]))
    for i in sorted(off):
        print("%-24s taken %3d, estimate off by %4.1f%% (mean)" % (
            names[i], taken.get(i, 0), 100 * sum(off[i]) / len(off[i])))


if __name__ == "__main__":
    {"measure": measure, "check": check}[sys.argv[1]](sys.argv[2])
