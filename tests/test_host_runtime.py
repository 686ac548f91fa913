"""The host side of the batch without a GPU: what it launches, seen by a stand-in for the HIP runtime (tests/host/runtime.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def scenario(tmp_path_factory):
    """Rows of numbers printed by a scenario of the stand-in."""
    from paper_2208_01260_amd import _lib, build

    if not os.path.exists(_lib.LIB_PATH):
        build.build()
    exe = str(tmp_path_factory.mktemp("host") / "runtime")
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-I" + os.path.join(ROOT, "include"),
                    os.path.join(HERE, "host", "runtime.cpp"), "-o", exe, "-ldl"], check=True)

    def run(*args):
        r = subprocess.run([exe, _lib.LIB_PATH] + [str(a) for a in args], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, (r.returncode, r.stderr)
        return [[int(v) for v in line.split()] for line in r.stdout.splitlines()]

    return run


@pytest.mark.parametrize("fast", [1, 3, 5, 16, 20, 44, 64, 200])
@pytest.mark.parametrize("nx,ny,count", [(64, 64, 5), (57, 49, 24)])
def test_autotune_returns_the_rows_in_use(scenario, nx, ny, count, fast):
    """The rows returned are those that a run then takes, whether timed or from the cache, and the candidate nearest to the
    device's fastest marches."""
    first, cached = scenario("tuned", nx, ny, count, fast)
    assert first == cached
    rows, waves, expected = first
    assert waves == expected
    away = lambda r: max(ny / -(-ny // r) / fast, fast / (ny / -(-ny // r)))  # noqa: E731
    assert rows in (8, 12, 16, 24, 32, 48, 64) and away(rows) == min(away(r) for r in (8, 12, 16, 24, 32, 48, 64))


@pytest.mark.parametrize("lengths", [(300,), (10000,), (255, 1, 1), (200, 200), (1, 256, 17), (256, 5)])
def test_batch_replays_graphs_after_256_steps(scenario, lengths):
    """Every step is launched once (three stages); the first 256 directly, within a call or over several, the rest by replays of
    16 steps and one of the remainder."""
    left = 256
    for n, (direct, graphs, replayed) in zip(lengths, scenario("batch", *lengths)):
        by_hand = min(left, n)
        left -= by_hand
        assert direct == 3 * by_hand and replayed == 3 * (n - by_hand)
        assert graphs == -(-(n - by_hand) // 16)
