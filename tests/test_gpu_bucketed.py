"""Gate steps at the edges between their paths (needs the GPU).

A step of 1- and 2-qubit gates takes one launch up to 2048 terms (in three
workgroup sizes: up to 512, 1024 and 2048), a selection by one workgroup up to
2^17 (from 2^14 with a window found beforehand), and a chain of launches above;
from 2049 terms on the state stays in the order of a linear hash of its keys.
FP64 sequences are compared with the oracle bit for bit, complex64 steps within
the per-step tolerances of the window tests.
"""
import sys

import numpy as np
import pytest

from oracle import c_oracle as CO
from paper_2607_07816_amd import batch as B
from paper_2607_07816_amd import circuits as C
from tests.helpers import random_state
from tests.test_gpu_window import check

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]

MASK64 = (1 << 64) - 1


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def S():
    from paper_2607_07816_amd import _lib
    return _lib


def gates(rng, n, ms):
    return [(tuple(int(q) for q in rng.choice(n, size=m, replace=False)), C.haar_unitary(rng, 1 << m)) for m in ms]


def oracle(keys, amps, gs, K, p):
    info = None
    for qs, U in gs:
        keys, amps, info = CO.step(keys, amps, qs, U, K, p, True, CO.host_threads())
    return *CO.sorted_terms(keys, amps), info


def run(st, gs):
    for qs, U in gs:
        st.apply_gate(qs, U)
        st.truncate()
    k, a = st.read_terms()
    return k, a, st.stats()


def same(S, keys, amps, n, gs, K, p, cap=None):
    ko, ao, info = oracle(keys, amps, gs, K, p)
    with S.State(n, K=K, p=p, precision="c128", capacity=cap or max(len(keys), K, 1024)) as st:
        st.load_terms(keys, amps)
        kg, ag, stats = run(st, gs)
    check(kg, ag, stats, ko, ao, info, "c128")


EDGES = [1, 2, 511, 513, 1024, 1025, 2047, 2048, 2049, 4097, 1 << 14, (1 << 14) + 1, (1 << 15) - 1,
         (1 << 15) + 1, 1 << 17, (1 << 17) + 1]


@pytest.mark.parametrize("p", [0.0, 0.99])
@pytest.mark.parametrize("N", EDGES)
def test_steps_at_the_edges(S, N, p):
    # gates of 1 and 2 qubits with a sorted step (3 qubits) in between, cut to N terms each time
    rng = np.random.default_rng([N, int(100 * p)])
    keys, amps = random_state(rng, 40, N)
    say(f"N={N} p={p}")
    same(S, keys, amps, 40, gates(rng, 40, [2, 2, 1, 2, 3, 2, 1, 2]), N, p)


@pytest.mark.parametrize("p", [0.5, 0.9])
@pytest.mark.parametrize("N", [1500, 3000, 30011, 70001, 140003])
def test_mass_alone(S, N, p):
    # no top-k: the rule is the mass, in a capacity that does not hold every
    # candidate; a result that does not fit is refused and changes nothing
    rng = np.random.default_rng([N, 3])
    keys, amps = random_state(rng, 40, N)
    refused = 0
    with S.State(40, K=0, p=p, precision="c128", capacity=3 * N) as st:
        st.load_terms(keys, amps)
        for qs, U in gates(rng, 40, [2, 1, 2]):
            ko, ao, info = oracle(keys, amps, [(qs, U)], 0, p)
            st.apply_gate(qs, U)
            if len(ko) > 3 * N:
                with pytest.raises(S.CapacityError):
                    st.truncate()
                refused += 1
            else:
                st.truncate()
                keys, amps = ko, ao
                stats = st.stats()
                assert stats["kept_fraction"] == info["fraction"] and stats["W"] == info["W"]
        kg, ag = st.read_terms()
    say(f"N={N} p={p}: {refused} refused")
    ko, ao = CO.sorted_terms(keys, amps)
    assert np.array_equal(kg, ko)
    assert np.array_equal(ag.view(np.uint64), ao.view(np.uint64))


@pytest.mark.parametrize("N", [700, 2049, 30011, 70001, 140003])
def test_c64_steps(S, N):
    rng = np.random.default_rng(N)
    keys, amps = random_state(rng, 48, N)
    with S.State(48, K=N, p=0.999, precision="c64", capacity=max(N, 1024)) as st:
        st.load_terms(keys, amps)
        for qs, U in gates(rng, 48, [2, 1, 2]):
            k, a = st.read_terms()
            st.apply_gate(qs, U)
            st.truncate()
            kg, ag = st.read_terms()
            ko, ao, info = CO.step(k, a, qs, U, N, 0.999, True, CO.host_threads())
            check(kg, ag, st.stats(), *CO.sorted_terms(ko, ao), info, "c64")


def lin_hash(keys):
    """The bucket hash (linhash.h): the XOR of a fixed word per set key bit."""
    h = np.zeros(len(keys), dtype=np.uint64)
    for q in range(64):
        x = (33 * 64 + q + 0x9e3779b97f4a7c15) & MASK64
        x = ((x ^ (x >> 30)) * 0xbf58476d1ce4e5b9) & MASK64
        x = ((x ^ (x >> 27)) * 0x94d049bb133111eb) & MASK64
        x ^= x >> 31
        h ^= np.where((keys >> np.uint64(q)) & np.uint64(1), np.uint64(x >> 32), np.uint64(0))
    return h


@pytest.mark.parametrize("p", [0.0, 0.9])
@pytest.mark.parametrize("N,bits", [(3000, 4), (20000, 6), (60000, 5), (60000, 9), (200000, 6)])
def test_skewed_buckets(S, N, bits, p):
    # all keys in 2^-bits of the buckets: shares that overflow their tables and slabs
    rng = np.random.default_rng([N, bits])
    keys = rng.integers(0, 1 << 50, size=N << bits, dtype=np.uint64)
    keys = np.unique(keys[lin_hash(keys) >> np.uint64(32 - bits) == 0])[:N]
    amps = rng.standard_normal(len(keys)) + 1j * rng.standard_normal(len(keys))
    amps /= np.linalg.norm(amps)
    same(S, keys, amps, 50, gates(rng, 50, [2, 1, 2]), len(keys), p, cap=4 * N)


@pytest.mark.parametrize("N", [1500, 3000, 20000, 50000, 150000])
def test_ties_across_the_cut(S, N):
    # equal weights throughout (X and a swap keep them): the keys decide
    rng = np.random.default_rng(N)
    keys, _ = random_state(rng, 40, N)
    amps = np.full(len(keys), 1.0 / np.sqrt(1 << 18), dtype=np.complex128)
    X = np.array([[0, 1], [1, 0]], dtype=np.complex128)
    swap = np.eye(4, dtype=np.complex128)[[0, 2, 1, 3]]
    for K in (N, N // 2 + 1):
        same(S, keys, amps, 40, [((3,), X), ((17, 30), swap), ((5,), X)], K, 0.0, cap=N)


@pytest.mark.parametrize("scale", [2.0 ** -9, 2.0 ** 9])
@pytest.mark.parametrize("N", [3000, 20000, 50000, 150000])
def test_missed_window(S, N, scale):
    # a previous cut predicts the next one's exponent; terms on another scale make it miss
    rng = np.random.default_rng(N)
    keys, amps = random_state(rng, 40, N)
    g1, g2 = gates(rng, 40, [2, 2]), gates(rng, 40, [2, 2])
    ko, ao, info = oracle(keys, amps * scale, g2, N, 0.0)
    with S.State(40, K=N, p=0.0, precision="c128", capacity=N) as st:
        st.load_terms(keys, amps)
        run(st, g1)
        st.load_terms(keys, amps * scale)
        kg, ag, stats = run(st, g2)
    check(kg, ag, stats, ko, ao, info, "c128")


@pytest.mark.parametrize("N", [600, 3000, 40000, 140000])
def test_nothing_cut_and_no_truncation(S, N):
    rng = np.random.default_rng(N)
    keys, amps = random_state(rng, 40, N)
    gs = gates(rng, 40, [2, 1])
    same(S, keys, amps, 40, gs, N << 4, 0.0)
    ko, ao = keys, amps
    for qs, U in gs:
        ko, ao, _ = CO.step(ko, ao, qs, U, 0, 0.0, False, CO.host_threads())
    ko, ao = CO.sorted_terms(ko, ao)
    with S.State(40, K=0, p=0.0, precision="c128", capacity=N << 3) as st:
        st.load_terms(keys, amps)
        for qs, U in gs:
            st.apply_gate(qs, U)
        kg, ag = st.read_terms()
    assert np.array_equal(kg, ko)
    assert np.array_equal(ag.view(np.uint64), ao.view(np.uint64))


@pytest.mark.parametrize("N", [1500, 3000, 50000, 150000])
def test_untruncated_gate_beyond_the_capacity(S, N):
    # reported by the next call, the gate discarded; the state goes on from the terms before it
    rng = np.random.default_rng(N)
    keys, amps = random_state(rng, 40, N)
    (q2, U2), (q1, U1) = gates(rng, 40, [2, 1])
    with S.State(40, K=0, p=0.0, precision="c128", capacity=3 * N) as st:
        st.load_terms(keys, amps)
        for _ in range(2):
            st.apply_gate(q2, U2)
            with pytest.raises(S.CapacityError):
                st.num_terms()
            k, a = st.read_terms()
            assert np.array_equal(k, np.sort(keys)) and np.array_equal(a, amps[np.argsort(keys)])
        st.apply_gate(q1, U1)
        kg, ag = st.read_terms()
    ko, ao, _ = CO.step(keys, amps, q1, U1, 0, 0.0, False, CO.host_threads())
    ko, ao = CO.sorted_terms(ko, ao)
    assert np.array_equal(kg, ko)
    assert np.array_equal(ag.view(np.uint64), ao.view(np.uint64))


def test_growth_through_every_size(S):
    # from one term to 2^17 and more: every path in turn, the bucket tables refined on the way
    rng = np.random.default_rng(5)
    perm = [int(q) for q in rng.permutation(30)]
    gs = [(tuple(perm[2 * i: 2 * i + 2]), C.haar_unitary(rng, 4)) for i in range(10)] + gates(rng, 30, [2, 2, 1, 2])
    keys, amps = np.zeros(1, dtype=np.uint64), np.ones(1, dtype=np.complex128)
    same(S, keys, amps, 30, gs, 150000, 0.0)


@pytest.mark.parametrize("K", [700, 1500, 5000, 40000, 135000])
def test_replayed_steps(S, K):
    # the same circuits with their steps captured once and replayed, and launched
    items = [(c, K, 0.0) for c, _ in C.batch_workload(2, 7, n_range=(20, 22), depth_range=(6, 6), logk_range=(9, 9))]
    plain, _ = B.run_batch(items, "c128", 2, 0, want_terms=True)
    for graph in (1, 8):
        res, _ = B.run_batch(items, "c128", 2, graph, want_terms=True)
        for a, b in zip(plain, res):
            assert a["status"] == b["status"] == 0
            assert np.array_equal(a["keys"], b["keys"])
            assert np.array_equal(a["amps"].view(np.uint64), b["amps"].view(np.uint64))


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n,N", [(5, 32), (40, 2500), (64, (1 << 18) + 1)])
def test_terms_to_and_from_the_host(S, n, N, prec):
    rng = np.random.default_rng(N)
    keys, amps = random_state(rng, n, N)
    order = rng.permutation(len(keys))
    want = np.argsort(keys)
    rounded = amps if prec == "c128" else amps.astype(np.complex64).astype(np.complex128)
    with S.State(n, K=0, p=0.0, precision=prec, capacity=max(N, 1024) * 2) as st:
        st.load_terms(keys[order], amps[order])
        for _ in range(2):  # reading leaves the state as it is
            k, a = st.read_terms()
            assert np.array_equal(k, keys[want]) and np.array_equal(a, rounded[want])
        # refused terms change nothing, a pending gate included
        U = np.diag([1.0, 1.0]).astype(np.complex128)
        st.apply_gate((1,), U)
        twice = keys.copy()
        twice[-1] = twice[0]
        nan, inf = amps.copy(), amps.copy()
        nan[len(nan) // 2] = complex(0.0, np.nan)
        inf[-1] = complex(np.inf, 0.0)
        bad = [(twice, amps), (keys, nan), (keys, inf)]
        if n < 64:
            far = keys.copy()
            far[len(far) // 3] = np.uint64(1 << n)
            bad.append((far, amps))
        for k, a in bad:
            with pytest.raises(Exception):
                st.load_terms(k, a)
        k, a = st.read_terms()
        assert np.array_equal(k, keys[want]) and np.array_equal(a, rounded[want])
