"""The bucket geometry of a gate (csrc/linhash.h), on the CPU: for every order
of bucket bits and gate, a wave's four buckets hold a term's partners and new
terms, and the tiles visit every bucket once."""
import ctypes
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

CSRC = Path(__file__).resolve().parents[1] / "paper_2607_07816_amd" / "csrc"
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

SOURCE = r"""
#include "linhash.h"
extern "C" void directions(unsigned *out) { for (int q = 0; q < 64; ++q) out[q] = lin_dir(q); }
extern "C" void plan(int hb, int m, const int *q, int pm, const int *pq, unsigned *E, int *piv, unsigned long long *cm)
{
    const BktPlan p = bkt_plan(hb, 0, m, q, pm, pq);
    for (int i = 0; i < STS_BKT_DIMS; ++i) { E[i] = p.E[i]; piv[i] = p.piv[i]; }
    cm[0] = p.cm[0];
    cm[1] = p.cm[1];
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not Path(HIPCC).exists():
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("linhash")
    (d / "t.hip").write_text(SOURCE)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}",
                    f"-I{CSRC.parents[1] / 'include'}", str(d / "t.hip"), "-o", str(d / "t.so")],
                   check=True, capture_output=True)
    return ctypes.CDLL(str(d / "t.so"))


def span(vs):
    s = {0}
    for v in vs:
        s |= {x ^ v for x in s}
    return s


@pytest.mark.parametrize("hb", [4, 5, 8, 13, 14])
def test_tiles_and_shares(lib, hb):
    rng = np.random.default_rng(hb)
    dirs = (ctypes.c_uint * 64)()
    lib.directions(dirs)
    for m in (1, 2, 2):
        for pm in (0, 1, 2):
            q = [int(x) for x in rng.choice(64, size=m, replace=False)]
            pq = [int(x) for x in rng.choice(64, size=pm, replace=False)]
            E, piv, cm = (ctypes.c_uint * 4)(), (ctypes.c_int * 4)(), (ctypes.c_ulonglong * 2)()
            lib.plan(hb, m, (ctypes.c_int * 2)(*q), pm, (ctypes.c_int * 2)(*pq), E, piv, cm)
            E = list(E)
            share = span(E[:2])
            assert len(share) == 4 and len(span(E)) == 16
            assert all((dirs[t] >> (32 - hb)) in share for t in q)  # the gate stays in a share
            # the tiles' representatives (all pivot bits zero) meet every coset once
            reps = [b for b in range(1 << hb) if not any(b >> p & 1 for p in piv)]
            assert len(reps) == 1 << (hb - 4)
            assert len({r ^ x for r in reps for x in span(E)}) == 1 << hb
            # a key's coordinates in the share, read by parity, are those of its bucket
            def rest(key):
                b = 0
                for t in range(64):
                    b ^= (dirs[t] >> (32 - hb)) if key >> t & 1 else 0
                for i in range(2):
                    b ^= E[i] if bin(key & int(cm[i])).count("1") & 1 else 0
                return b

            for key in rng.integers(0, 1 << 63, size=20, dtype=np.uint64):
                at = rest(int(key))
                assert len({at ^ x for x in share}) == 4
                assert all(rest(int(key) ^ (1 << t)) == at for t in q)
