"""Weights fetched ahead, on the CPU: which workgroup reads what, and where the rule has a launch do it, against the times it
rests on.  The header is compiled as it is for the kernels and the launchers (no GPU needed)."""
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("prefetch") / "prefetch")
    subprocess.run(["g++", "-std=c++17", "-O2", "-o", exe, os.path.join(HERE, "prefetch_main.cpp")], check=True)
    return lambda lines: subprocess.run([exe], input="\n".join(lines) + "\n", check=True, capture_output=True, text=True).stdout.splitlines()


def test_every_piece_is_read_by_one_workgroup(ask):
    """Arrays smaller than a thread's loads, ragged, empty, equal to and around what the workgroups read at most, beside
    launches of one and of many workgroups of either size."""
    rng = random.Random(3)
    cases = [(0, 0, 5, 256), (1, 0, 1, 256), (0, 7, 1, 256), (1, 1, 1000, 256), (3072, 0, 1, 256), (3073, 0, 1, 256), (6144, 0, 2, 512),
             (331776, 663552, 3, 256), (331776, 41472, 576, 256), (4800000, 0, 1, 128), (2047, 2049, 1, 128)]
    cases += [(rng.randint(0, 200000), rng.randint(0, 20000), rng.randint(1, 700), rng.choice([128, 256, 512])) for _ in range(30)]
    for c, line in zip(cases, ask(["span %d %d %d %d" % c for c in cases])):
        rows, most, ok = (int(v) for v in line.split())
        assert ok and 1 <= rows <= 1 + 1563, c
        assert (rows == 1) == (c[0] + c[1] == 0), c
        assert most <= 3072 + 2, c   # 48 KB, rounded up in each of the two arrays


# Milliseconds of a step without and with weights fetched ahead: tokens, and the most that a launch would fetch (w_co and w_fc1);
# hidden sizes 1152 (16 and 4 heads of 72), 1536, 3072, 4096 (16 heads of 64)
def _bytes(D, A):
    return 2 * (D * A + 4 * D * D)


TIMES = [(N, _bytes(1152, 1152), a, b) for N, a, b in [
            (64, 5.069, 4.777), (72, 4.705, 4.768), (96, 4.855, 4.831), (128, 5.021, 4.875), (136, 4.775, 4.861), (192, 4.991, 4.906),
            (200, 4.967, 5.106), (256, 5.204, 5.118), (272, 5.342, 5.415), (392, 5.477, 5.535), (512, 6.129, 6.001), (520, 6.012, 6.075),
            (648, 6.232, 6.284), (960, 7.237, 7.016), (1032, 7.350, 7.234), (1200, 8.039, 7.868), (1920, 9.871, 9.467), (2304, 10.694, 10.346)]]
TIMES += [(N, _bytes(1152, 288), a, b) for N, a, b in [(64, 4.576, 4.363), (128, 4.582, 4.392), (336, 4.815, 4.869), (400, 4.857, 4.911),
                                                       (576, 5.553, 5.469), (1200, 6.955, 6.768), (2304, 8.357, 8.141)]]
TIMES += [(N, _bytes(1536, 1536), a, b) for N, a, b in [(64, 2.069, 1.963), (256, 2.374, 2.304), (702, 3.070, 2.977), (2304, 5.324, 5.168)]]
TIMES += [(N, _bytes(3072, 3072), a, b) for N, a, b in [(64, 1.148, 1.197), (256, 1.501, 1.546), (702, 2.266, 2.321), (1200, 2.782, 2.883)]]
TIMES += [(N, _bytes(4096, 1024), a, b) for N, a, b in [(64, 0.913, 0.990), (256, 1.095, 1.218), (702, 1.615, 1.763), (1200, 2.189, 2.339)]]


def test_rule_against_measured_steps(ask):
    """Fetched where a step was measured to gain, left alone where it was measured to lose, and never beyond what was measured."""
    answers = ask(["pays %d %d" % (N, b) for N, b, _, _ in TIMES] + ["pays 3200 1000", "pays 3201 1000"])
    for (N, b, without, with_), pays in zip(TIMES, answers):
        assert int(pays) == (with_ < without), (N, b, without, with_)
    assert answers[-2:] == ["1", "0"]
