"""Which kernel a prefill product takes and in which order, on the CPU: the rules stand in a header of their own, which the launcher
includes, and a host program answers for it."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("gemm_choice") / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(ROOT, "paper_2504_12285_amd", "csrc"), os.path.join(ROOT, "tests", "gemm_choice_driver.cpp"), "-o", exe]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout

    def answers(questions):
        run = subprocess.run([exe], input="\n".join(questions), stdout=subprocess.PIPE, text=True, timeout=120)
        lines = run.stdout.splitlines()
        assert run.returncode == 0 and len(lines) == len(questions)
        return [tuple(int(v) for v in line.split()) for line in lines]
    return answers


def _bytes(along, total, per_line, per_item):
    """Bytes per k of the XCD that reads most, when each takes an eighth of `total` tiles in lines of `along`."""
    share, most = -(-total // 8), 0
    for first in range(0, total, share):
        last = min(total, first + share) - 1
        most = max(most, (last // along - first // along + 1) * per_line + min(along, last - first + 1) * per_item)
    return most


def test_split_k_order(ask):
    """The order is the one that reads less by a quarter, and what the estimate reckons with is that order's bytes."""
    measured = {(3931, 256): 1, (2528, 320): 1, (512, 1024): 1, (408, 925): 1, (452, 891): 1,        # faster across
                (395, 1600): 0, (444, 1600): 0, (329, 1438): 0, (384, 1407): 0, (392, 1280): 0}      # slower across
    for (M, N), (across, _) in zip(measured, ask(["order %d %d" % s for s in measured])):
        assert across == measured[M, N], (M, N)
    rng = random.Random(1)
    shapes = [(rng.randint(1, 4096), rng.randint(1, 14000)) for _ in range(2000)] + [(1, 1), (64, 32), (65, 33), (1 << 24, 1), (1, 1 << 24), (1 << 24, 1 << 24)]
    for (M, N), (across, got) in zip(shapes, ask(["order %d %d" % s for s in shapes])):
        tm, tn = -(-M // 64), -(-N // 32)
        down, over = _bytes(tm, tm * tn, 8, 64), _bytes(tn, tm * tn, 64, 8)
        want, line = (over, 64) if across else (down, 8)
        assert want <= got <= want + line, (M, N)                  # (a share that starts inside a line may be reckoned to touch one more)
        assert not across or 4 * over <= 3 * (down + 8)
        assert across or 4 * (over + 64) > 3 * down


def test_split_k_shapes(ask):
    """The shapes of the GPU test go to the split k loop, in the order that they stand for."""
    import test_gpu_gemm_split_k as t
    for shapes, want in ((t.ACROSS, 1), (t.DOWN, 0)):
        assert [a for a, _ in ask(["order %d %d" % s[:2] for s in shapes])] == [want] * len(shapes)
        for acc in (0, 1):
            assert ask(["plain %d %d %d 0 %d 1" % (M, N, -(-K // 64) * 64, acc) for M, N, K in shapes]) == [(5,)] * len(shapes)


def test_broken_lines_of_few_tokens(ask):
    """fp32 rows that start inside a line: where the split k loop measured 7 - 14 % faster than tiles of 64 x 128.  Whole lines, and int32
    output alone, the other way round."""
    shapes = [(909, 460, 256), (492, 831, 256), (357, 1001, 256), (293, 3082, 448), (772, 975, 448), (1654, 308, 64), (670, 382, 128)]
    assert ask(["plain %d %d %d 0 0 1" % s for s in shapes]) == [(5,)] * len(shapes)
    shapes = [(512, 3840, 2560), (1000, 3840, 2560), (1161, 1914, 64), (242, 4032, 256), (403, 1536, 64), (237, 1856, 64)]
    assert ask(["plain %d %d %d 0 0 1" % s for s in shapes]) == [(4,)] * len(shapes)
    assert ask(["plain 370 2033 256 0 1 0", "plain 242 4032 256 0 1 0"]) == [(4,), (4,)]


def test_stores_of_broken_lines(ask):
    """Outputs of 5 million values and more whose rows start inside a line: plain stores measured 0.66 - 0.90 of the time."""
    shapes = [(4072, 1915), (842, 8443), (713, 10148), (1328, 4641), (585, 10937), (2242, 2986), (2106, 3705), (2443, 3038), (3812, 6613), (4096, 13823)]
    assert ask(["stores %d %d 0" % s for s in shapes]) == [(0,)] * len(shapes)
    shapes = [(422, 4751), (387, 7778), (2077, 1335), (4096, 13824), (2048, 13840)]
    assert ask(["stores %d %d 0" % s for s in shapes]) == [(1,)] * len(shapes)
    assert ask(["stores 422 4751 1", "stores 4096 13824 1"]) == [(0,), (1,)]


def test_tables_of_33_to_48_tokens(ask):
    """Layers (hidden, ffn, count) whose tables measured faster in tiles, and with the tokens in LDS."""
    def layers(hidden, ffn, count):
        shapes = [(hidden + 2 * (hidden // 4), hidden), (hidden, hidden), (2 * ffn, hidden), (hidden, ffn)]
        blocks = [(-(-N // 256), -(-K // 128)) for N, K in shapes]
        return "table %d %d %d" % (count * sum(n for n, _ in blocks), count * sum(n * k for n, k in blocks), max(k for _, k in blocks))
    tiles = [(2560, 6912, 4), (2560, 6912, 30), (4096, 11008, 3), (4096, 8192, 2), (2304, 5760, 3), (1536, 4608, 6), (1024, 2816, 5), (896, 2560, 4)]
    lds = [(2560, 6912, 1), (2560, 6912, 3), (4096, 11008, 1), (2048, 5632, 4), (4096, 8192, 1), (3584, 9472, 1)]
    assert ask([layers(*s) for s in tiles]) == [(1,)] * len(tiles)
    assert ask([layers(*s) for s in lds]) == [(0,)] * len(lds)


def test_gpu_shapes_reach_the_kernels_that_they_stand_for(ask):
    import test_gpu_gemm_pipe as pipe
    import test_gpu_tile_order as order
    for lists in (pipe.TILES, pipe.GUARDED):
        assert sorted(lists) == list(range(6))
        for place, shapes in lists.items():
            assert ask(["plain %d %d %d 0 0 1" % (M, N, -(-K // 64) * 64) for M, N, K in shapes]) == [(place,)] * len(shapes), place
    for what, lists, count in (("residual", pipe.RESIDUAL, 3), ("gate", pipe.GATE, 2)):
        assert sorted(lists) == list(range(count))
        for place, shapes in lists.items():
            assert ask(["%s %d %d %d" % ((what,) + s) for s in shapes]) == [(place,)] * len(shapes), (what, place)
    for what, shapes, count in (("plain", order.PLAIN, 5), ("residual", order.RESIDUAL, 3), ("gate", order.GATE, 2)):
        assert ask(["%s %d %d %d" % ((what,) + s[:3]) + (" 0 0 1" if what == "plain" else "") for s in shapes]) == [(s[3],) for s in shapes]
        assert {s[3] for s in shapes} == set(range(count))


def test_the_order_that_the_gpu_test_reckons_with_is_the_launchers(ask):
    import test_gpu_tile_order as order
    rng = random.Random(2)
    shapes = [(rng.randint(1, 300), rng.randint(1, 300), rng.choice([64, 128]), rng.randint(1, 110) * 64) for _ in range(2000)]
    assert [(gm, band) for gm, band, _ in ask(["tiles %d %d %d %d" % s for s in shapes])] == [order._order(*s) for s in shapes]
