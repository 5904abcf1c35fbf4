"""The choice between the cuts of the gather kernel and the slab kernel against the timings it was made from
(profiles/cut_sweep.csv: us of every product in every cut).  No GPU."""
import csv
import ctypes
import math
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CUTS = ["whole_64", "whole_128", "wide_by_2", "wide_by_4", "by_2", "by_4", "by_8", "slab"]
ROWS = {"aligned": 0, "any": 1, "images": 2}


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("choice") / "choice_probe.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_2203_05016_amd", "csrc"), os.path.join(HERE, "choice_probe.cpp"), "-o", so])
    f = ctypes.CDLL(so).probe_choice
    f.argtypes = [ctypes.c_int, ctypes.c_long, ctypes.c_long, ctypes.c_long] + [ctypes.c_int] * 5 + [ctypes.c_double, ctypes.c_int]
    return f


def _choose(probe, V, G, N, steps, K, rows, uneven, f32, slab, kept):
    return CUTS[probe(V, G, N, steps, K, ROWS[rows], uneven, f32, slab, kept, 0)]


def _sweep(probe):
    with open(os.path.join(ROOT, "profiles", "cut_sweep.csv")) as f:
        for r in csv.DictReader(line for line in f if not line.startswith("#")):
            if int(r["G"]) < 4:
                continue
            times = {c: float(r[c]) for c in CUTS if r[c]}
            cut = _choose(probe, int(r["V"]), int(r["G"]), int(r["N"]), int(r["steps"]), int(r["K"]), r["rows"],
                          int(r["uniform"]) < 0, int(r["f32"]), "slab" in times, float(r["kept"]))
            assert cut in times or (cut == "by_8" and not r["by_8"]), (r, cut)   # (not timed in a part of the sweep)
            if cut in times:
                yield r, times, cut


def test_choice_is_near_the_best_of_every_measured_product(probe):
    """The times are single measurements (2 % apart when repeated), and the best of eight of them is low by that."""
    kinds = {}
    for r, times, cut in _sweep(probe):
        lost = times[cut] / min(times.values())
        for key in ("all", "V %s" % r["V"], r["rows"], "f32" if r["f32"] == "1" else "16 bits"):
            kinds.setdefault(key, []).append(lost)
    for key, lost in kinds.items():
        lost.sort()
        mean = math.exp(sum(map(math.log, lost)) / len(lost))
        high, worst = lost[int(.95 * len(lost))], lost[-1]
        print("%-8s %4d products: %.3f of the best's time, 95 %% within %.3f, all within %.2f" % (key, len(lost), mean, high, worst))
        assert mean < 1.03 and high < 1.18 and worst < 1.6, (key, mean, high, worst)


@pytest.mark.parametrize("V,G,N,steps,K,rows,f32,kept,cuts", [
    # few steps of many groups: a workgroup's own cost decides, not its time per step
    (64, 81, 1728, 81 * 4, 128, "aligned", 0, .25, ["whole_64"]),
    (64, 19, 7032, 19 * 4, 64, "aligned", 0, .25, ["whole_64", "whole_128", "slab"]),   # us: 8.0, 8.0, 8.0; wide_by_2 10.9
    (64, 54, 2560, 54 * 4, 112, "aligned", 0, .4, ["whole_64", "whole_128", "slab"]),   # 6.4, 7.3, 7.3; 9.6
    (16, 360, 180, 360 * 4, 80, "any", 1, .25, ["whole_64", "by_2", "by_4"]),
    (128, 45, 1024, 45 * 16, 856, "aligned", 1, .25, ["by_2"]),
    # two row blocks and more share what a chunk of X holds, too, where most of it is kept
    (64, 128, 16384, 128 * 512, 8192, "aligned", 0, 1., ["slab"]),
    (64, 64, 8192, 64 * 256, 4096, "aligned", 0, 1., ["slab"]),
    (128, 32, 8192, 32 * 256, 4096, "aligned", 0, 1., ["slab"]),
    (64, 32, 14216, 32 * 20, 296, "aligned", 1, 1., ["slab"]),
    (64, 128, 16384, 128 * 128, 8192, "aligned", 0, .25, ["whole_128"]),
    (128, 32, 8192, 32 * 64, 4096, "aligned", 0, .25, ["whole_64"]),
    # finer groups: slab from a quarter (V = 32) or a fifth (16)
    (32, 128, 8192, 128 * 12, 1024, "aligned", 0, .17, ["whole_128"]),
    (32, 128, 8192, 128 * 64, 4096, "aligned", 0, .5, ["slab"]),
    (16, 256, 8192, 256 * 8, 1024, "aligned", 0, .25, ["slab"]),
    # nine column tiles: two of them on one XCD, which takes twice the time of the others
    (32, 207, 1152, 207 * 68, 4152, "aligned", 0, .25, ["whole_64", "whole_128", "wide_by_2", "wide_by_4"]),
])
def test_choice_where_the_cuts_differ_most(probe, V, G, N, steps, K, rows, f32, kept, cuts):
    assert _choose(probe, V, G, N, steps, K, rows, 0, f32, rows == "aligned", kept) in cuts


def test_slab_is_chosen_only_where_it_can_run(probe):
    for r, times, cut in _sweep(probe):
        if cut == "slab":
            assert r["rows"] == "aligned" and int(r["G"]) >= (12 if int(r["V"]) <= 32 else 8 if r["V"] == "64" else 4)


def test_weights_are_shared_where_the_sweep_says_so(probe):
    """Whole tiles of shared weights against such that fetch their own, where there is a workgroup for most CUs: the
    columns whole_64 and whole_128 hold the variant that the rule takes, own_64 and own_128 the other side."""
    ratios = {}
    for r, times, _ in _sweep(probe):
        for what, cut, own in ((1, "whole_64", "own_64"), (2, "whole_128", "own_128")):
            if cut not in times or not probe(int(r["V"]), int(r["G"]), int(r["N"]), int(r["steps"]), 0, 0, 0, 0, 0, 0, what):
                continue
            columns = 64 * what
            if int(r["G"]) * (-(-(-(-int(r["N"]) // columns)) // 4)) >= 200:
                per = int(r["steps"]) // int(r["G"])
                edge = next(e for e in (8, 12, 16, 32, 64, 1 << 20) if per <= e)
                ratios.setdefault((int(r["V"]), columns, edge), []).append(times[cut] / float(r[own]))
    for key, x in sorted(ratios.items()):
        mean = math.exp(sum(map(math.log, x)) / len(x))
        print("V %d, %d columns, up to %d steps: %.3f (%d)" % (key + (mean, len(x))))
        if len(x) >= 10:
            assert mean < 1.03, (key, mean)
