"""2-D programs taken op by op, on the CPU (tests/prog2d/stream.cpp): what the solo executor and
the batched solver launch while the program is built."""
import os
import subprocess

import pytest

import paper_1810_05268_amd as P

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.parametrize("comp", [0, 1], ids=["plain", "compressed"])
def test_streamed_ops_are_the_program_and_few_are_held(tmp_path, comp):
    """With one slot a program has nt^2 / (2 T) groups of steps (15,000 for 300 steps by threes);
    an executor that launches them as they come holds those of one action."""
    binary = str(tmp_path / "stream")
    subprocess.run(["hipcc", "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "prog2d", "stream.cpp"), "-o", binary], check=True)
    cases = [(K, T, nt, M) for K, T in ((1, 8), (4, 3), (8, 1)) for nt in (1, 2, 9, 40, 300)
             for M in sorted({1, 2, 5, 20, nt}) if M <= nt]
    text = []
    for K, T, nt, M in cases:
        a = P.schedule(nt, M, write_min=not comp)
        text += [f"{K} {T} {M} {comp} 1 {len(a)}", " ".join(str(int(v)) for v in a.ravel())]
    r = subprocess.run([binary], input="\n".join(text), capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    got = [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]
    assert len(got) == len(cases)
    for case, (ops, held) in zip(cases, got):
        assert held <= 24, case
    assert got[cases.index((4, 3, 300, 1))][0] > 15000
