"""Host-side checks of the single-workgroup coarse cycle's index arithmetic and
sizes: the headers that the kernels are built from, compiled for the host."""
import os
import shutil
import subprocess

import pytest

from paper_1905_08890_amd import build as B


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    """Compiles and runs the body of a main() that has the coarse cycle's headers."""
    hipcc = B.HIPCC if os.path.exists(B.HIPCC) else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("host")

    def run(name, body):
        src = d / f"{name}.hip"
        src.write_text('#include <cstdio>\n#include "coarse_cycle.h"\nusing namespace grmg;\nusing namespace grmg::detail;\n'
                       "int main()\n{\n" + body + "\n}\n")
        exe = d / name
        subprocess.run([hipcc, "-O1", "--offload-host-only", "-std=c++17", "-I", B.INCLUDE, "-I", B.CSRC, str(src), "-o",
                        str(exe)], check=True, capture_output=True, text=True, timeout=300)
        return subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=300).stdout

    return run


def test_pair_index_division_is_exact_on_every_coarsest_side(host):
    """A sweep of a coarsest level of side n decodes its n^2 n/2 x-pairs: t / (n/2) and
    the row's / n.  All coarsest sides up to 1022 (twice an odd number); the quotients just
    below, at and above the last multiples, and a stride through the rest."""
    out = host("division", r"""
    for (int n = 2; n <= 1022; n += 4) {
        const int half = n / 2, tot = n * n * half;
        const SmallDiv dh(half, tot), dn(n);
        for (long t = 0; t < tot; t = t < tot - 100000 ? t + 9973 : t + 1)
            if (dh.div((int)t) != t / half) { printf("side %d pair %ld\n", n, t); break; }
        for (int r = 0; r < n * n; ++r)
            if (dn.div(r) != r / n) { printf("side %d row %d\n", n, r); break; }
    }""")
    assert out == "", out
