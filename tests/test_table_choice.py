"""What the choice of a shared PSF table may return, over a wide grid of problems, against what is compiled.

The choice is plain C++ (csrc/table_choice.cpp), built here with g++. The limits below are those of the
kernels in csrc/table.hip: windows of K = 16, 24 ... 80 samples, 2048 staged weight pairs, half of at most 72
taps on either side of a derivative's band, adjoint workgroups of 4 or 8 waves in 150 KiB of LDS.
"""
import itertools
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
D = 0.5


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("choice") / "table_choice")
    csrc = os.path.join(ROOT, "paper_2406_08703_amd", "csrc")
    cmd = [gxx, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", csrc,
           os.path.join(csrc, "table_choice.cpp"), os.path.join(ROOT, "tests", "native", "table_choice_driver.cpp"),
           "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(problems):
        text = "".join(" ".join(map(repr, p)) + "\n" for p in problems)
        r = subprocess.run([exe], input=text, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        lines = r.stdout.splitlines()
        assert len(lines) == len(problems)
        names = ("h16", "W", "K", "waves", "Nt", "n_reg", "slots", "lds", "pairs", "chunk", "groups", "per_group", "bytes")
        return [dict(zip(names, map(int, l.split()[1:]))) if l[0] == "1" else None for l in lines]
    return run


def problem(n_pupil, n_focal, L, stars, frames, pixel=0.5, q=1, band=(500e-9, 600e-9), bf16x3=0, dither=0):
    """`pixel`: a detector pixel in units of (band centre) / D; q focal samples across it."""
    lo, hi = band if L > 1 else (band[0], band[0])
    return (n_pupil, n_focal, L, stars, frames, n_focal // q, bf16x3, dither, D, pixel * 0.5 * (lo + hi) / D / q, lo, hi)


def check(p, s):
    assert s["K"] % 8 == 0 and 16 <= s["K"] <= 80, (p, s)
    assert s["pairs"] <= 2048 and s["W"] <= 72 and s["W"] + 15 * s["h16"] // 16 < s["K"], (p, s)
    assert s["waves"] in (4, 8) and s["lds"] <= 150 * 1024, (p, s)
    assert s["Nt"] % 64 == 0 and s["n_reg"] % 64 == 0 and s["n_reg"] <= s["Nt"] <= 32064, (p, s)
    assert 1 <= s["chunk"] <= p[4] and s["chunk"] * p[3] <= 65535 and s["bytes"] <= 16 << 30, (p, s)
    assert (s["groups"] - 1) * s["per_group"] < s["chunk"] * p[3] <= s["groups"] * s["per_group"], (p, s)
    assert s["slots"] > 0 and s["slots"] % s["waves"] == 0, (p, s)


def test_every_table_of_a_grid_of_problems_is_compiled(choose):
    ps = []
    for n_pupil, n_det, q, pixel in itertools.product((33, 64, 128, 251, 384, 512, 640, 813, 1024, 1500),
                                                      (16, 61, 128, 284, 512, 768, 1024), (1, 2, 3, 4, 5),
                                                      (0.0489, 0.1, 0.25, 0.4, 0.5, 0.7, 1.0, 1.5)):
        for L, stars, frames in ((1, 1, 40), (2, 3, 64), (8, 1, 16), (16, 1, 16), (32, 2, 64), (29, 8, 4), (90, 24, 1)):
            for band in ((500e-9, 505e-9), (545e-9, 645e-9), (450e-9, 800e-9), (400e-9, 900e-9)):
                if (n_pupil + n_det + L + frames) % 3 == 0:   # a third of the grid, each value with every other
                    ps.append(problem(n_pupil, n_det * q, L, stars, frames, pixel, q, band, dither=int(frames == 1)))
    rng = random.Random(5)
    for _ in range(20000):
        q = rng.choice((1, 1, 2, 3, 4))
        lo = rng.choice((450e-9, 500e-9, 545e-9))
        ps.append(problem(int(32 * 30 ** rng.random()), q * int(16 * 48 ** rng.random()), int(40 ** rng.random()),
                          int(12 ** rng.random()), int(64 ** rng.random()), rng.choice((0.5, rng.uniform(0.05, 1.2))),
                          q, (lo, lo * rng.uniform(1.01, 1.8)), rng.randrange(2), rng.randrange(2)))
    chosen = 0
    for p, s in zip(ps, choose(ps)):
        if s:
            chosen += 1
            check(p, s)
    print(f"{chosen} tables of {len(ps)} problems")
    assert chosen > 3000


@pytest.mark.parametrize("args", [(512, 512, 16, 1, 16), (512, 512, 8, 1, 16, 0.5, 1, (545e-9, 645e-9)),
                                  (640, 512, 16, 1, 16), (813, 284, 28, 1, 43), (480, 496, 29, 8, 4),
                                  (384, 512, 10, 1, 8, 0.5, 1, (545e-9, 645e-9)),
                                  (384, 512, 10, 1, 8, 0.5, 1, (450e-9, 700e-9))])
def test_nyquist_pixels_without_oversampling(choose, args):
    """One sample per Nyquist pixel asks for the longest windows; what is chosen there is compiled."""
    p = problem(*args)
    s = choose([p])[0]
    assert s is None or check(p, s) is None


def test_a_table_that_needs_too_much_memory_is_not_chosen(choose):
    """1500^2 pupils and 40 wavelengths over an octave: the table would take 73 GiB; with few wavelengths
    and a smaller field the same detector has one. A million stars need too much for their weights."""
    big = problem(1500, 1024, 40, 1, 64, band=(450e-9, 900e-9))
    small = problem(600, 512, 8, 1, 64)
    many = problem(128, 128, 24, 2, 500000)
    few = problem(128, 128, 24, 2, 5000)
    got = choose([big, small, many, few])
    assert got[0] is None and got[2] is None
    for s in (got[1], got[3]):
        assert s is not None and s["bytes"] <= 16 << 30
    assert got[3]["bytes"] > 10000 * 16 * got[3]["slots"]   # the stars' own arrays are counted


@pytest.mark.parametrize("args,hi", [((640, 256, 40, 1, 4), 700e-9), ((512, 384, 24, 1, 4), 700e-9),
                                     ((960, 320, 38, 1, 3), 725e-9), ((576, 432, 32, 1, 3), 570e-9),
                                     ((896, 256, 33, 1, 3), 565e-9), ((822, 538, 16, 1, 3), 630e-9)])
def test_split_precision_is_weighed_at_its_own_speed(choose, args, hi):
    """Few frames of large pupils: a table beats FP32 transforms per star, and costs 9 to 28% more than split ones."""
    fp32, split = choose([problem(*args, band=(500e-9, hi), bf16x3=b) for b in (0, 1)])
    assert fp32 is not None and split is None


def test_split_precision_keeps_the_table_where_it_pays(choose):
    """24 stars of 512 pupil and 768 focal samples and 32 wavelengths (10 times faster), and small plans of many frames,
    whose launches cost as much in split precision (half the time and less)."""
    joint = problem(512, 768, 32, 2, 12, q=3, band=(500e-9, 700e-9), bf16x3=1)
    small = [problem(96, 320, 26, 1, 24, q=2, band=(500e-9, 650e-9), bf16x3=1),
             problem(352, 32, 33, 2, 24, pixel=0.25, band=(500e-9, 730e-9), bf16x3=1),
             problem(320, 144, 39, 2, 4, pixel=0.25, q=3, band=(500e-9, 670e-9), bf16x3=1)]
    assert all(s is not None for s in choose([joint, *small]))
