"""Ranges of trial triangles of the batch pair kernels (host rule): their partial
rows stay within 2 GiB (or one range), the ranges cover the triangles, and the
modelled time is within 2 % of the best over all splits, from 20 triangles to
300 000."""
import math
import os
import random
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_split_bounds_scratch_and_time(tmp_path):
    exe = str(tmp_path / "batch_split")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall",
                    "-I", os.path.join(ROOT, "paper_2104_04609_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "batch_split.cpp"), "-o", exe], check=True)
    rng = random.Random(3)
    Ts = [20, 31, 32, 33, 80, 720, 1280, 5120, 12500, 20480, 40500, 163840, 220500, 248000, 272000,
          297680] + [int(math.exp(rng.uniform(math.log(20), math.log(300000)))) for _ in range(80)]
    args = []
    for T in Ts:
        for C in (1, 2, 4):   # 8, 16 and 32 vectors; test triangles per workgroup
            rows = 64 // C
            for slots in (512, 256):
                args.append((T, -(-T // rows), slots, T * 6 * 16 * C * 8))
    out = subprocess.run([exe], input="\n".join(" ".join(map(str, a)) for a in args), text=True,
                         capture_output=True, check=True).stdout.split("\n")
    for (T, tiles, slots, b), line in zip(args, out):
        ns, ln, cost = int(line.split()[0]), int(line.split()[1]), float(line.split()[2])
        assert ln % 32 == 0 and (ns - 1) * ln < T <= ns * ln
        assert ns == 1 or ns * b <= 2 << 30, (T, ns, ns * b)
        nt = -(-T // 32)
        best = min(math.ceil(tiles * n / slots) * (32 * q + 4)
                   for n, q in {-(-nt // q): q for q in range(nt, 0, -1)}.items())
        assert cost <= 1.02 * best, (T, tiles, slots, cost / best)
