"""The field arrays that a 2-D run reserves are enough for its programs, and few: every program
is executed symbolically on them, on the CPU (tests/prog2d/rings.cpp)."""
import os
import subprocess

import pytest

import paper_1810_05268_amd as P

HERE = os.path.dirname(os.path.abspath(__file__))
CHUNKS = (1, 75, 5000, 6000, 10000, 20000)   # of a field: 64^2 points to 9051^2


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("prog2d") / "rings")
    subprocess.run(["hipcc", "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "prog2d", "rings.cpp"), "-o", out], check=True)

    def go(lines):
        r = subprocess.run([out], input="\n".join(lines), capture_output=True, text=True)
        assert r.returncode == 0, r.stdout[-200:] + r.stderr
        return [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]

    return go


def _most(K):
    return 8 if K <= 2 else 2 if K == 8 else 16 // K


@pytest.mark.parametrize("comp", [0, 1], ids=["plain", "compressed"])
def test_gradient_programs_fit_the_arrays(run, comp):
    """Group sizes from one step to the order's most, few and many codec chunks, slots from one
    (every state recomputed from the first) to one a state."""
    lines, n = [], 0
    for K in (1, 3, 4, 6, 8):
        for T in sorted({0, 1, 2, _most(K)}):   # 0: steps march
            for chunks in CHUNKS:
                for nt in (1, 2, 9, 40, 101):
                    for M in sorted({1, 2, 5, 20, max(1, nt - 1), nt}):
                        if M > nt or (n + nt) % 3:
                            n += M <= nt
                            continue
                        a = P.schedule(nt, M, write_min=not comp)
                        lines += [f"{K} {T} {chunks} {M} {comp} {len(a)}", " ".join(str(int(v)) for v in a.ravel())]
                        n += 1
    assert len(run(lines)) == len(lines) // 2


def test_forward_programs_and_sizes(run):
    got = run([f"{K} {T} 0 0 0 {nt}" for K in (1, 4, 8) for T in sorted({0, 1, 2, _most(K)}) for nt in (1, 2, 3, 9, 40)])
    assert all(levels <= 4 and decoded == 0 for _, levels, decoded in got)
    # a field that fills the chip alone, one step a launch: two levels, the next, one decoded
    a = P.schedule(40, 5, write_min=False)
    assert run([f"4 1 20000 5 1 {len(a)}", " ".join(str(int(v)) for v in a.ravel())]) == [(1, 3, 1)]


def test_workspace_holds_few_arrays():
    """A 2-D grid at order 4, in groups of four steps: the forward call's two levels before a group
    and two after it, w and zeros; the gradient's 12 levels, 8 decoded, 4 adjoint, one more
    decoded, w, zeros and room to encode eight fields."""
    from tests.test_lib_host import host_problem
    from paper_1810_05268_amd import _binding as B
    pb = host_problem(n=(1500, 1400), nbl=20, space_order=4)
    field = 4 * pb.field_elements()
    assert pb.workspace_bytes(B.OP_FORWARD) <= 6 * field + (1 << 20)
    assert pb.workspace_bytes(B.OP_GRADIENT, 0) <= 36 * field + (1 << 20)
