"""The programs of 2-D runs (groups of steps, encodes and decodes) against their schedules, on
the CPU: tests/prog2d/main.cpp executes each one symbolically and checks every level read."""
import os
import subprocess

import pytest

import paper_1810_05268_amd as P

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def binary(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("prog2d") / "prog2d")
    subprocess.run(["hipcc", "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "prog2d", "main.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("comp", [0, 1], ids=["plain", "compressed"])
def test_programs_read_the_levels_their_schedules_mean(binary, comp):
    """Step counts around the group sizes (1..8) and their multiples, slots from one (every
    state recomputed from the first) to one per state, with and without data rows."""
    text, n = [], 0
    for K in (1, 2, 3, 4, 5, 6, 7, 8):
        for nt in (1, 2, 3, 7, 8, 9, 17, 40, 101):
            for M in sorted({1, 2, 3, 5, 9, 20, max(1, nt // 2), max(1, nt - 1), nt}):
                if M > nt:
                    continue
                a = P.schedule(nt, M, write_min=not comp)
                most = 8 if K <= 2 else 2 if K == 8 else 16 // K
                for T in {1, 2, most, (nt + M) % most + 1}:
                    text.append(f"{K} {T} {M} {comp} {(K + M) % 2} {len(a)}")
                    text.append(" ".join(str(int(v)) for v in a.ravel()))
                    n += 1
    r = subprocess.run([binary], input="\n".join(text), capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == f"{n} programs", r.stdout + r.stderr
