"""The walk over the parts of an overfull share (csrc/parts.h), on the CPU:
every term is in exactly one part, no part is larger than a wave's tables, and
a cluster of terms with a long common prefix costs a few parts a bit."""
import ctypes
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

CSRC = Path(__file__).resolve().parents[1] / "paper_2607_07816_amd" / "csrc"
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

SOURCE = r"""
#include "parts.h"
// parts and scans of a share with these hashes; seen[i]: parts that hold term i; returns the parts, -1 if one did not fit
extern "C" long walk(unsigned n, unsigned cap, const unsigned long long *h, unsigned *seen, long *scans, long limit)
{
    PartWalk w;
    w.begin(n, cap);
    long parts = 0;
    *scans = 0;
    auto in = [&](unsigned i) { return !w.depth || (h[i] >> (64 - w.depth)) == w.pre; };
    auto count = [&]() {
        unsigned c = 0;
        for (unsigned i = 0; i < n; ++i) c += in(i);
        ++*scans;
        return c;
    };
    do {
        unsigned c = count();
        while (c > cap && w.depth < 64) {
            w.split();
            c = count();
        }
        if (c > cap) return -1;
        for (unsigned i = 0; i < n; ++i) seen[i] += in(i);
        if (++parts > limit) return parts;
    } while (w.next());
    return parts;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not Path(HIPCC).exists():
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("parts")
    (d / "t.hip").write_text(SOURCE)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}",
                    f"-I{CSRC.parents[1] / 'include'}", str(d / "t.hip"), "-o", str(d / "t.so")],
                   check=True, capture_output=True)
    so = ctypes.CDLL(str(d / "t.so"))
    so.walk.restype = ctypes.c_long
    return so


CAP = 320


def clustered(rng, spread, cluster, bits, at):
    """`spread` random hashes and `cluster` ones that share their top `bits` bits (all zeros, all ones or random)."""
    top = {"low": 0, "high": (1 << bits) - 1, "any": int(rng.integers(0, 1 << 62)) >> (62 - bits) if bits else 0}[at]
    low = [int(x) for x in rng.integers(0, 1 << 62, size=cluster)]
    c = [(top << (64 - bits)) | (x >> (bits - 2) if bits > 2 else x) for x in low]
    return np.concatenate([rng.integers(0, (1 << 64) - 1, size=spread, dtype=np.uint64), np.array(c, dtype=np.uint64)])


@pytest.mark.parametrize("at", ["low", "high", "any"])
@pytest.mark.parametrize("spread,cluster,bits", [(1, 0, 0), (320, 0, 0), (321, 0, 0), (5000, 0, 0), (300, 330, 8),
                                                 (300, 330, 11), (300, 330, 40), (0, 700, 50), (3000, 400, 30)])
def test_every_term_once_in_few_parts(lib, spread, cluster, bits, at):
    rng = np.random.default_rng([spread, cluster, bits])
    h = clustered(rng, spread, cluster, bits, at)
    n = len(h)
    seen, scans = np.zeros(n, dtype=np.uint32), ctypes.c_long(0)
    even = 1
    while n // even > CAP * 3 // 4:
        even *= 2
    # the even parts, a part and a scan more per bit of the cluster's prefix, and its own even parts
    limit = even + bits + max(4 * cluster // CAP, 1) + 16
    parts = lib.walk(n, CAP, h.ctypes.data_as(ctypes.c_void_p), seen.ctypes.data_as(ctypes.c_void_p), ctypes.byref(scans),
                     ctypes.c_long(1 << 20))
    assert 0 < parts <= limit
    assert scans.value <= parts + limit
    assert (seen == 1).all()


BINNED, ROUNDS = 640, 64  # BW_BINNED and WEIGH_ROUNDS of csrc/bucket_impl.h


def rounds_of(sizes):
    return sum(-(-s // 64) + 1 for s in sizes)  # one round more than full ones, for the groups of several members


def part_sizes(h, cap):
    """The parts of the walk, from their definition: halves of what does not fit."""
    even = 0
    while len(h) > cap and len(h) >> even > cap * 3 // 4:
        even += 1
    out, todo = [], [(even, p) for p in range(1 << even)]
    while todo:
        d, p = todo.pop()
        c = sum(1 for x in h if x >> (64 - d) == p)
        if c > cap:
            todo += [(d + 1, 2 * p), (d + 1, 2 * p + 1)]
        else:
            out.append(c)
    return out


@pytest.mark.parametrize("n", [321, 480, 500, BINNED])
def test_rounds_of_usual_shares(lib, n):
    # evenly spread shares of every size that the weighing pass sums stay far below its bound
    for seed in range(5):
        rng = np.random.default_rng([n, seed])
        h = [int(x) for x in rng.integers(0, (1 << 64) - 1, size=n, dtype=np.uint64)]
        assert rounds_of(part_sizes(h, CAP)) <= ROUNDS // 2


def test_the_most_parts_of_a_summed_share(lib):
    # a term beside the cluster at every bit of its prefix: a part a bit, which the bound on the rounds catches
    n = BINNED
    side = [1 << (63 - d) for d in range(50)]
    rng = np.random.default_rng(0)
    h = side + [int(x) for x in rng.permutation(1 << 13)[:n - len(side)]]
    arr = np.array(h, dtype=np.uint64)
    seen, scans = np.zeros(n, dtype=np.uint32), ctypes.c_long(0)
    parts = lib.walk(n, CAP, arr.ctypes.data_as(ctypes.c_void_p), seen.ctypes.data_as(ctypes.c_void_p), ctypes.byref(scans),
                     ctypes.c_long(1 << 20))
    assert parts == len(part_sizes(h, CAP)) <= 66
    assert (seen == 1).all()
    assert rounds_of(part_sizes(h, CAP)) > ROUNDS  # more than a lane's sums are counted on for
