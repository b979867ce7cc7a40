"""The transform lengths of csrc/lengths_more.def: together with lengths.def
they cover every 2/3/5-smooth length up to 4096 except those that have no
split with factors of at most 75, every line is a split of its length, and
every factor's register DFT matches the O(N^2) definition (host build)."""
import os
import subprocess

import pytest

from paper_2003_07504_amd.build import lengths

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _smooth(n):
    for q in (2, 3, 5):
        while n % q == 0:
            n //= q
    return n == 1


def test_lengths_cover_the_supported_range_once():
    tuned = [L for L, _, _ in lengths("lengths.def")]
    more = lengths("lengths_more.def")
    assert all(P * Q == L and P <= Q <= 75 for L, P, Q in more)
    every = tuned + [L for L, _, _ in more]
    assert len(set(every)) == len(every)
    assert {n for n in range(2, 4097) if _smooth(n)} - set(every) == {2187, 3125, 3645, 4000}


def test_register_dfts_of_the_further_factors(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "dft_more")
    subprocess.run([HIPCC, "-x", "hip", "-O2", "-std=c++17", "--offload-arch=gfx950",
                    os.path.join(ROOT, "tests", "native", "dft_more_check.cpp"), "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    res = {int(n): (float(a), float(b)) for n, a, b in (ln.split() for ln in out.strip().splitlines())}
    need = {f for _, P, Q in lengths("lengths_more.def") for f in (P, Q)}
    assert need <= set(res)
    for n, (fwd, inv) in res.items():
        assert fwd < 1e-6 and inv < 1e-6, (n, fwd, inv)
