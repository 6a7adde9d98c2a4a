"""The split of a 3-D grid's planes over workgroups, on the CPU (tests/chunks3d/main.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def chunks(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("chunks3d") / "chunks3d")
    subprocess.run(["g++", "-std=c++17", "-O1", os.path.join(HERE, "chunks3d", "main.cpp"), "-o", out], check=True)

    def run(cases):
        text = "\n".join(" ".join(str(int(v)) for v in c) for c in cases)
        r = subprocess.run([out], input=text, capture_output=True, text=True, check=True)
        return [int(v) for v in r.stdout.split()]

    return run


def _tiles(nx, ny):
    return -(-nx // 32) * -(-ny // 32)


# (grid, order, gradient, workgroups of the kernel that fit a CU): chunk lengths measured within
# 2.5 % of the fastest of up to 16
MEASURED = [
    ((300, 40, 480), 4, 0, 3, {13}), ((300, 40, 480), 4, 1, 3, {5, 13}),
    ((300, 40, 480), 6, 0, 3, {13}), ((300, 40, 480), 6, 1, 3, {13}),
    ((600, 120, 90), 4, 1, 3, {9}), ((168, 168, 168), 8, 0, 3, {12}), ((168, 168, 168), 8, 1, 3, {12}),
    ((168, 168, 168), 16, 0, 2, {12}), ((168, 168, 168), 16, 1, 2, {12}),
    ((183, 139, 125), 12, 0, 2, {8}), ((183, 139, 125), 12, 1, 2, {8}),
    ((296, 296, 296), 12, 0, 2, {60}), ((296, 296, 296), 12, 1, 2, {60}),
    ((400, 400, 400), 16, 0, 2, {134}), ((400, 400, 400), 16, 1, 2, {134}),
    ((1200, 100, 100), 16, 0, 2, {34}), ((700, 300, 60), 6, 0, 3, {30}), ((64, 64, 64), 8, 0, 3, {1}),
]


def test_near_the_fastest_measured(chunks):
    got = chunks([(_tiles(n[0], n[1]), n[2], order // 2, grad, fit) for n, order, grad, fit, _ in MEASURED])
    for (n, order, grad, _, best), zlen in zip(MEASURED, got):
        assert zlen in best, (n, order, grad, zlen)


def test_lengths_are_of_the_grid(chunks):
    cases = [(t, nz, K, g, fit) for t in (1, 7, 64, 1000, 40000) for nz in (1, 2, 31, 400, 3000) for K in (1, 8)
             for g in (0, 1) for fit in (1, 2, 4)]
    for (t, nz, K, g, fit), zlen in zip(cases, chunks(cases)):
        assert 1 <= zlen <= nz, (t, nz, K, g, fit, zlen)
