"""How much a 2-D program holds, on the CPU (tests/prog2d/sizes.cpp builds them)."""
import os
import subprocess

import pytest

import paper_1810_05268_amd as P

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def sizes(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("prog2d") / "sizes")
    subprocess.run(["hipcc", "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "prog2d", "sizes.cpp"), "-o", out], check=True)

    def run(cases):
        text = []
        for K, T, nt, M, comp in cases:
            a = P.schedule(nt, M, write_min=not comp)
            text += [f"{K} {T} {M} {comp} 1 {len(a)}", " ".join(str(int(v)) for v in a.ravel())]
        r = subprocess.run([out], input="\n".join(text), capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]

    return run


@pytest.mark.parametrize("comp", [0, 1], ids=["plain", "compressed"])
def test_ops_beside_steps_are_bounded_by_the_step_count(sizes, comp):
    """The batched solver's room, 10 nt + 64 ops, holds every op but the steps' at any number of
    slots; with one slot or two the steps alone are more (at nt = 300, order 8, groups of 3)."""
    cases = [(K, T, nt, M, comp) for K, T in ((2, 8), (4, 3), (8, 1)) for nt in (1, 2, 5, 17, 100, 300)
             for M in sorted({1, 2, 3, 5, 9, 20, max(1, nt // 2), max(1, nt - 1), nt}) if M <= nt]
    got = sizes(cases)
    assert len(got) == len(cases)
    for case, (ops, other) in zip(cases, got):
        assert other <= 10 * case[2] + 64, case
    assert got[cases.index((4, 3, 300, 1, comp))][0] > 10 * 300 + 64
