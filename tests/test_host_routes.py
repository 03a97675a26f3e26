"""Which small-grid contexts step in resident workgroups, against both ways'
measured times."""
import shutil
import subprocess
from pathlib import Path

HERE = Path(__file__).resolve().parent
CSRC = HERE.parent / "paper_2304_03306_amd" / "csrc"

# n64, n128, vorticity source, microseconds of a step with the two passes and
# resident (FP32, then FP64 state; MI355X, untuned, 100-step calls)
TIMES = [
    (0, 72, 0, 18.4, 18.8, 18.7, 18.6), (0, 96, 0, 20.7, 18.8, 21.4, 18.7), (0, 256, 0, 37.8, 21.1, 38.3, 21.6),
    (0, 257, 0, 38.9, 37.0, 39.4, 37.3), (0, 384, 0, 47.5, 38.2, 48.8, 38.4), (0, 513, 0, 58.8, 56.0, 61.3, 56.7),
    (0, 769, 0, 82.0, 74.7, 84.2, 74.2), (0, 1025, 0, 122.5, 93.4, 128.7, 94.2),
    (0, 80, 1, 21.2, 22.6, 21.7, 22.9), (0, 96, 1, 23.7, 22.7, 24.3, 23.1), (0, 256, 1, 43.1, 28.1, 43.2, 28.6),
    (0, 257, 1, 44.2, 48.1, 44.0, 49.3), (0, 288, 1, 47.3, 48.5, 47.7, 50.4), (0, 384, 1, 54.7, 52.3, 55.5, 53.3),
    (0, 512, 1, 67.1, 53.1, 69.9, 54.2), (0, 513, 1, 68.1, 72.8, 70.8, 76.1), (0, 704, 1, 88.4, 78.9, 100.1, 80.5),
    (0, 768, 1, 94.6, 79.4, 106.8, 81.3), (0, 864, 1, 119.6, 101.2, 119.8, 103.3),
    (0, 1025, 1, 138.7, 122.4, 143.9, 128.1),
    (1, 96, 0, 22.9, 25.9, 24.1, 25.8), (1, 128, 0, 28.4, 25.8, 28.7, 25.9), (1, 288, 0, 42.9, 45.5, 43.1, 44.9),
    (1, 512, 0, 60.3, 46.5, 62.8, 47.0), (32, 96, 0, 24.7, 26.1, 25.4, 26.0), (128, 96, 0, 28.7, 26.0, 28.6, 25.9),
    (512, 96, 0, 39.9, 28.0, 39.8, 27.8), (512, 288, 0, 57.4, 47.0, 58.1, 47.0),
    (1, 96, 1, 26.7, 31.1, 27.4, 32.2), (1, 128, 1, 32.8, 33.3, 33.1, 34.4), (1, 192, 1, 39.0, 35.0, 39.1, 35.4),
    (1, 288, 1, 49.1, 57.7, 49.0, 59.5), (1, 512, 1, 72.3, 61.7, 73.9, 62.5), (32, 160, 1, 36.8, 34.8, 36.8, 35.2),
    (32, 320, 1, 53.1, 57.6, 53.2, 59.5), (128, 288, 1, 52.9, 57.3, 53.0, 60.1), (512, 96, 1, 45.6, 33.5, 45.4, 34.1),
]


def _rule(tmp_path, triples):
    exe = tmp_path / "rule"
    r = subprocess.run([shutil.which("g++"), "-std=c++17", "-O1", f"-I{CSRC}", str(HERE / "host" / "resident_rule.cpp"),
                        "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], input="\n".join("%d %d %d" % t for t in triples), capture_output=True, text=True)
    assert r.returncode == 0
    return [v == "1" for v in r.stdout.split()]


def test_the_way_taken_is_the_faster_one(tmp_path):
    """The measured times of either way repeat to 2 %; the way taken costs at
    most that more than the other."""
    taken = _rule(tmp_path, [t[:3] for t in TIMES])
    bad = []
    for t, resident in zip(TIMES, taken):
        for passes, res in (t[3:5], t[5:7]):
            if (res if resident else passes) > 1.02 * (passes if resident else res):
                bad.append((t, resident))
    assert not bad, bad


def test_64_points_always_and_few_of_128_never(tmp_path):
    assert all(_rule(tmp_path, [(n, 0, s) for n in (1, 7, 256, 5000) for s in (0, 1)]))
    assert not any(_rule(tmp_path, [(a, n, s) for a in (0, 1, 5000) for n in (1, 95) for s in (0, 1)]))
