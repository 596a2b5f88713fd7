"""Shares that overflow a wave's tables in unkind ways (needs the GPU): many
terms of one share whose mixed masked keys share a long prefix, so that its
parts are many and small. FP64, compared with the oracle bit for bit."""
import functools

import numpy as np
import pytest

from oracle import c_oracle as CO
from paper_2607_07816_amd import circuits as C
from tests.test_gpu_bucketed import MASK64, S, lin_hash, oracle, run, same  # noqa: F401 (S: a fixture)
from tests.test_gpu_window import check

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]


def unmix(h):
    """The inverse of sts_mix64 (common.h), the SplitMix64 finaliser."""
    def unshift(x, s):
        y = x.copy()
        for _ in range(64 // s + 1):
            y = x ^ (y >> np.uint64(s))
        return y
    with np.errstate(over="ignore"):
        x = unshift(h, 31)
        x = x * np.uint64(pow(0x94d049bb133111eb, -1, 1 << 64))
        x = unshift(x, 27)
        x = x * np.uint64(pow(0xbf58476d1ce4e5b9, -1, 1 << 64))
        return unshift(x, 30)


def mix(x):
    with np.errstate(over="ignore"):
        x = (x ^ (x >> np.uint64(30))) * np.uint64(0xbf58476d1ce4e5b9)
        x = (x ^ (x >> np.uint64(27))) * np.uint64(0x94d049bb133111eb)
    return x ^ (x >> np.uint64(31))


@functools.lru_cache(maxsize=None)
def clustered_keys(count, bits, hb, gate):
    """`count` keys of 64 bits, zero on the gate's qubits, in one bucket of
    2^hb, whose mixed keys have `bits` leading bits in common."""
    rng = np.random.default_rng([count, bits, hb])
    mask = np.uint64(MASK64 ^ sum(1 << q for q in gate))
    bucket, out = None, np.zeros(0, dtype=np.uint64)
    prefix = int(rng.integers(0, 1 << 62)) >> (62 - bits)
    while len(out) < count:
        low = rng.integers(0, 1 << (64 - bits), size=1 << 22, dtype=np.uint64)
        k = unmix(np.uint64(prefix << (64 - bits)) | low)
        k = k[k & ~mask == 0]
        b = lin_hash(k) >> np.uint64(32 - hb)
        bucket = b[0] if bucket is None else bucket
        out = np.unique(np.concatenate([out, k[b == bucket]]))
    return rng.permutation(out)[:count]


def span_of_kernel(bits, rng, count):
    """`count` keys of 64 bits whose bucket hash has its top `bits` bits zero."""
    dirs = lin_hash(np.uint64(1) << np.arange(64, dtype=np.uint64)) >> np.uint64(32 - bits)
    rows = [(int(d), 1 << q) for q, d in enumerate(dirs)]  # (hash, key): eliminate the hash bits
    for b in range(bits):
        pivot = next((r for r in rows if r[0] >> b & 1), None)
        if pivot:
            rows.remove(pivot)
            rows = [(h ^ pivot[0], k ^ pivot[1]) if h >> b & 1 else (h, k) for h, k in rows]
    basis = np.array([k for h, k in rows if h == 0], dtype=np.uint64)
    out = np.zeros(0, dtype=np.uint64)
    while len(out) < count:
        pick = rng.integers(0, 2, size=(2 * count, len(basis)), dtype=np.uint64)
        out = np.unique(np.concatenate([out, np.bitwise_xor.reduce(pick * basis[None, :], axis=1)]))
    return rng.permutation(out)[:count]


def test_unmix():
    x = np.random.default_rng(1).integers(0, 1 << 63, size=1000, dtype=np.uint64)
    assert np.array_equal(unmix(mix(x)), x)


@pytest.mark.parametrize("p", [0.0, 0.9])
@pytest.mark.parametrize("N,hb,bits", [(3000, 8, 30), (20000, 11, 30), (150000, 14, 28), (150000, 14, 10)])
def test_clustered_share(S, N, hb, bits, p):
    # one share of 330 clustered terms and the buckets' usual ones, cut by the next gate's truncation
    rng = np.random.default_rng([N, bits])
    gate = (3, 40)
    heavy = clustered_keys(330, bits, hb, gate)
    keys = np.unique(np.concatenate([heavy, rng.integers(0, MASK64, size=N - 330, dtype=np.uint64)]))
    amps = rng.standard_normal(len(keys)) + 1j * rng.standard_normal(len(keys))
    amps /= np.linalg.norm(amps)
    other = tuple(int(q) for q in rng.choice(64, size=2, replace=False))
    gs = [(gate, C.haar_unitary(rng, 4)), (other, C.haar_unitary(rng, 4)), (gate[:1], C.haar_unitary(rng, 2))]
    print(f"N={N} hb={hb} bits={bits} p={p}", flush=True)
    same(S, keys, amps, 64, gs, len(keys), p, cap=2 * len(keys))


@pytest.mark.parametrize("p", [0.0, 0.9])
@pytest.mark.parametrize("N,bits", [(1 << 16, 16), (1 << 16, 12), (60000, 4), (60000, 3), (150000, 4), (150000, 3),
                                    (20000, 3), (1500, 16)])
def test_terms_that_crowd_in_few_buckets(S, N, bits, p):
    # all terms in 2^-bits of the buckets: from some 160 in each on their steps are sorted, those with fewer
    # take their shares in parts. (65536 terms of one bucket took seconds a step bucketed.)
    rng = np.random.default_rng([N, bits])
    keys = span_of_kernel(bits, rng, N)
    amps = rng.standard_normal(N) + 1j * rng.standard_normal(N)
    amps /= np.linalg.norm(amps)
    print(f"N={N} bits={bits} p={p}", flush=True)
    same(S, keys, amps, 64, [((int(a), int(b)), C.haar_unitary(rng, 4)) for a, b in rng.choice(64, size=(3, 2), replace=False)],
         N, p, cap=4 * N)


def test_crowded_terms_and_then_others(S):
    # the order follows the terms that were loaded last; refused terms leave it
    rng = np.random.default_rng(7)
    N = 1 << 14
    crowded, spread = span_of_kernel(14, rng, N), np.unique(rng.integers(0, MASK64, size=N, dtype=np.uint64))
    amps = rng.standard_normal(N) + 1j * rng.standard_normal(N)
    gs = [((5, 50), C.haar_unitary(rng, 4)), ((9,), C.haar_unitary(rng, 2))]
    with S.State(64, K=N, p=0.0, precision="c128", capacity=N) as st:
        for keys in (crowded, spread, crowded):
            st.load_terms(keys, amps[:len(keys)])
            with pytest.raises(Exception):
                st.load_terms(np.concatenate([keys, keys[:1]])[1:], np.full(len(keys), np.nan))
            ko, ao, info = oracle(keys, amps[:len(keys)], gs, N, 0.0)
            kg, ag, stats = run(st, gs)
            check(kg, ag, stats, ko, ao, info, "c128")


@pytest.mark.parametrize("N,bits", [(150000, 3), (60000, 3), (150000, 0)])
def test_untruncated_gates_of_crowded_terms(S, N, bits):
    # the new terms of some shares exceed their slabs: they are computed again for the write
    rng = np.random.default_rng([N, bits, 5])
    keys = span_of_kernel(bits, rng, N) if bits else np.unique(rng.integers(0, MASK64, size=N, dtype=np.uint64))
    amps = rng.standard_normal(N) + 1j * rng.standard_normal(N)
    gs = [((int(a), int(b)), C.haar_unitary(rng, 4)) for a, b in rng.choice(64, size=(2, 2), replace=False)]
    ko, ao = keys, amps
    with S.State(64, K=0, p=0.0, precision="c128", capacity=4 * N) as st:
        st.load_terms(keys, amps)
        for i, (qs, U) in enumerate(gs):
            if i:  # back to N terms
                kg, ag = ko[::4], ao[::4]
                st.load_terms(kg, ag)
                ko, ao = kg, ag
            ko, ao, _ = CO.step(ko, ao, qs, U, 0, 0.0, False, CO.host_threads())
            ko, ao = CO.sorted_terms(ko, ao)
            st.apply_gate(qs, U)
            kg, ag = st.read_terms()
            assert np.array_equal(kg, ko)
            assert np.array_equal(ag.view(np.uint64), ao.view(np.uint64))


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n", [8, 9, 40, 64])
def test_few_terms_to_and_from_the_host(S, n, prec):
    # up to 1,024 terms and 512 per 8 qubits the host orders and checks them, the device more
    line = 1024 + 512 * -(-n // 8)
    rng = np.random.default_rng(n)
    for N in sorted({min(N, 1 << n) for N in (1, 2, 255, 1000, line, line + 1)}):
        ends = np.array([0, (1 << n) - 1], np.uint64)
        keys = np.unique(np.concatenate([ends, rng.integers(0, ends[1], size=4 * N, dtype=np.uint64, endpoint=True)]))
        keys = rng.permutation(keys)[:N]
        amps = rng.standard_normal(len(keys)) + 1j * rng.standard_normal(len(keys))
        want = np.argsort(keys)
        rounded = amps if prec == "c128" else amps.astype(np.complex64).astype(np.complex128)
        with S.State(n, K=0, p=0.0, precision=prec, capacity=8192) as st:
            st.load_terms(keys, amps)
            for bad in ("twice", "range", "nan", "inf"):
                k, a = keys.copy(), amps.copy()
                if bad == "twice":
                    if len(k) < 2:
                        continue
                    k[-1] = k[0]
                elif bad == "range":
                    if n == 64:
                        continue
                    k[len(k) // 2] = np.uint64(1 << n)
                else:
                    a[-1] = complex(0.0, np.nan) if bad == "nan" else complex(np.inf, 0.0)
                with pytest.raises(Exception):
                    st.load_terms(k, a)
            for _ in range(2):
                kg, ag = st.read_terms()
                assert np.array_equal(kg, keys[want]) and np.array_equal(ag, rounded[want])
