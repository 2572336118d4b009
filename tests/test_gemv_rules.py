"""Short batch-1 launches (see gemv_rules_main.cpp): the ranges of tiles that workgroups get, over drawn launches, and the choice
between the two kernels against measured ones."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# layers, weight bits, int8?, microseconds of the streaming kernel and of the one with ranges of tiles, measured on one MI355X
CHOICES = [
    ("11008x4096", 3, 0, 11.5, 9.1), ("11008x4096*2", 4, 1, 18.3, 16.9), ("4096x4096*3", 3, 0, 11.9, 9.6), ("8192x8192", 4, 0, 15.5, 13.6),
    ("22555x1024", 3, 1, 8.8, 7.0), ("2459x4992*2 5263x640", 3, 0, 12.7, 8.8), ("9296x2432*4", 4, 1, 17.7, 15.7), ("12228x5120", 3, 0, 12.9, 10.8),
    ("9000x14336", 3, 0, 17.0, 20.8), ("17492x11520", 3, 0, 22.8, 25.9), ("4096x4096*4 11008x4096*2 4096x11008", 3, 0, 23.1, 25.8),
    ("7084x9344*3 6653x1664", 4, 0, 30.8, 34.7), ("7091x896*2 8623x11136", 4, 1, 18.9, 21.0), ("4754x12416*3", 4, 0, 27.8, 30.1),
]


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if not cxx:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("rules") / "gemv_rules_main")
    subprocess.run([cxx, "-O1", "-std=c++17", "-o", exe, os.path.join(ROOT, "tests", "gemv_rules_main.cpp")], check=True)
    return lambda lines: subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout.split("\n")[:-1]


def _layers(text):
    got = []
    for part in text.split():
        shape, _, times = part.partition("*")
        got += [tuple(int(v) for v in shape.split("x"))] * int(times or 1)
    return got


def _words(layers):
    return "%d %s" % (len(layers), " ".join("%d %d" % l for l in layers))


def test_choice_follows_the_measurements(ask):
    got = ask(["short %d %d %s" % (bw, int8, _words(_layers(text))) for text, bw, int8, _, _ in CHOICES])
    assert [int(g) for g in got] == [int(short < stream) for _, _, _, stream, short in CHOICES]


def test_ranges_cover_the_launch_and_fit_the_kernel(ask):
    """Every launch that goes there: ranges follow each other, none holds more tiles than LDS has sums for, and the fullest one has
    an equal share and not more than one tile of the deepest layer besides."""
    rng = random.Random(7)
    drawn = []
    for _ in range(4000):
        deep = [128 * int(round(2 ** rng.uniform(0, 7.2))) for _ in range(2)]
        drawn.append([(int(2 ** rng.uniform(4, 17)), rng.choice(deep)) for _ in range(rng.randint(1, 8))])
    taken = [l for l, g in zip(drawn, ask(["short %d %d %s" % (rng.choice([3, 4]), rng.randint(0, 1), _words(l)) for l in drawn])) if g == "1"]
    assert len(taken) > 300
    for layers, line in zip(taken, ask(["cuts " + _words(l) for l in taken])):
        least, most, longest = map(int, line.split())
        share = -(-sum(-(-out // 16) * (inn // 128) for out, inn in layers) // 256)
        deepest = max(inn // 128 for _, inn in layers)
        assert 0 <= least and most <= 64 and longest <= share + deepest and deepest <= 128, (layers, line)
