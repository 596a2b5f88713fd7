"""Cuts far from where most weights lie, and steps that cut nothing (needs the
GPU): gates close to a permutation, whose cut lies in the tail of the kept
weights, and gates that do not branch, on states around and above 2^17 terms.
FP64, compared with the oracle bit for bit."""
import numpy as np
import pytest

from paper_2607_07816_amd import batch as B
from paper_2607_07816_amd import circuits as C
from tests.helpers import random_state
from tests.test_gpu_bucketed import S, oracle, run  # noqa: F401 (S: a fixture)
from tests.test_gpu_window import check

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]

CZ = np.diag([1, 1, 1, -1]).astype(np.complex128)


def rx(theta):
    c, s = np.cos(theta), np.sin(theta)
    return np.array([[c, -1j * s], [-1j * s, c]])


def pick(rng, n, m):
    return tuple(int(q) for q in rng.choice(n, size=m, replace=False))


def steps(S, keys, amps, n, gs, K, p, cap):
    """Every step of `gs` on one context, each compared with the oracle's."""
    with S.State(n, K=K, p=p, precision="c128", capacity=cap) as st:
        st.load_terms(keys, amps)
        for i, (qs, U) in enumerate(gs):
            keys, amps, info = oracle(keys, amps, [(qs, U)], K, p)
            kg, ag, stats = run(st, [(qs, U)])
            print(f"step {i} {qs}", flush=True)
            if info is None:  # no rule: the oracle weighs nothing
                info = dict(fraction=1.0, W=stats["W"])
            check(kg, ag, stats, keys, amps, info, "c128")


@pytest.mark.parametrize("p", [0.0, 0.99999])
@pytest.mark.parametrize("theta", [1e-2, 1e-3, 1e-4, 1e-7, 1e-12, 1e-40])
@pytest.mark.parametrize("N", [40000, 150000])
def test_gates_close_to_a_permutation(S, N, theta, p):
    rng = np.random.default_rng([N, int(-np.log10(theta))])
    keys, amps = random_state(rng, 40, N)
    gs = [(pick(rng, 40, 2), C.haar_unitary(rng, 4))] + \
         [(pick(rng, 40, 2), CZ @ np.kron(rx(theta), rx(theta))), (pick(rng, 40, 1), rx(theta))] * 2
    steps(S, keys, amps, 40, gs, N, p, N)


@pytest.mark.parametrize("exponents", [(-3, 3), (-60, 60), (-150, 100)])
def test_weights_of_any_size(S, exponents):
    # amplitudes spread over many octaves, on both sides of the cut
    rng = np.random.default_rng(exponents[1])
    N = 150000
    keys, amps = random_state(rng, 40, N)
    amps = amps * 2.0 ** rng.integers(exponents[0], exponents[1], size=N)
    steps(S, keys, amps, 40, [(pick(rng, 40, m), C.haar_unitary(rng, 1 << m)) for m in (2, 1, 2, 2)], N, 0.0, N)


def permutations(rng, n, count):
    """Gates that do not branch."""
    X = np.array([[0, 1], [1, 0]], dtype=np.complex128)
    cx = np.eye(4, dtype=np.complex128)[[0, 3, 2, 1]]
    one = [lambda: np.diag(np.exp(1j * rng.uniform(0, 6, 2))), lambda: X]
    two = [lambda: CZ, lambda: cx]
    return [(pick(rng, n, m), (one if m == 1 else two)[i // 2 % 2]()) for i, m in enumerate((1, 2) * count)][:count]


@pytest.mark.parametrize("K", [0, 1 << 18])
@pytest.mark.parametrize("n,N", [(18, 1 << 18), (18, 140000), (17, 1 << 17)])
def test_every_key_fits(S, n, N, K):
    # K at least every key of the qubits, no p-mass: nothing is ever cut
    rng = np.random.default_rng([n, N])
    keys, amps = random_state(rng, n, N)
    steps(S, keys, amps, n, [(pick(rng, n, m), C.haar_unitary(rng, 1 << m)) for m in (2, 1, 2, 2)], K, 0.0, 1 << 18)


@pytest.mark.parametrize("p", [0.0, 0.9999])
@pytest.mark.parametrize("K", [150000, 150001, 149990, 600000])
def test_gates_that_do_not_branch(S, K, p):
    # as many candidates as K, one fewer, some more; then a gate that branches, and again
    rng = np.random.default_rng(K)
    N = 150000
    keys, amps = random_state(rng, 40, N)
    haar = [(pick(rng, 40, 2), C.haar_unitary(rng, 4))]
    steps(S, keys, amps, 40, permutations(rng, 40, 4) + haar + permutations(rng, 40, 3) + haar + haar, K, p, max(K, N))


@pytest.mark.parametrize("prec", ["c64", "c128"])
def test_uncut_steps_of_shares_beyond_their_slabs(S, prec):
    # growing by four at each gate into the whole capacity, from a state that leaves some slabs too small
    rng = np.random.default_rng(11)
    N = 140000
    keys, amps = random_state(rng, 40, N)
    gs = [(pick(rng, 40, 2), C.haar_unitary(rng, 4)), (pick(rng, 40, 1), C.haar_unitary(rng, 2))]
    with S.State(40, K=8 * N, p=0.0, precision=prec, capacity=8 * N) as st:
        st.load_terms(keys, amps)
        kg, ag, stats = run(st, gs)
    if prec == "c64":
        amps = amps.astype(np.complex64).astype(np.complex128)
    ko, ao, info = oracle(keys, amps, gs, 8 * N, 0.0)
    check(kg, ag, stats, ko, ao, info, prec)


@pytest.mark.parametrize("N,values", [(140000, 1), (300000, 1), (300000, 3)])
def test_cut_among_many_equal_weights(S, N, values):
    # more terms of the cut's weight than the selection's buffer holds (65,536): the keys decide
    rng = np.random.default_rng([N, values])
    keys, _ = random_state(rng, 40, N)
    amps = rng.choice([1.0, 1.5, 1j], size=N)[:N].astype(np.complex128) if values > 1 else np.ones(N, dtype=np.complex128)
    amps = amps * 2.0 ** -9
    H = np.array([[1, 1], [1, -1]], dtype=np.complex128)
    steps(S, keys, amps, 40, permutations(rng, 40, 2) + [(pick(rng, 40, 1), H * 0.5), (pick(rng, 40, 1), H)], N // 2 + 1, 0.0, N)


@pytest.mark.parametrize("N", [40000, 150000])
def test_runs_repeat_bit_for_bit(S, N):
    # complex64 sums of 3-qubit groups follow the state's order, which a p-mass rule's window shapes
    rng = np.random.default_rng(N)
    keys, amps = random_state(rng, 40, N)
    gs = [(pick(rng, 40, m), C.haar_unitary(rng, 1 << m)) for m in (2, 3, 1, 2, 3, 2, 4, 2)]
    out = []
    for _ in range(3):
        with S.State(40, K=N, p=0.97, precision="c64", capacity=2 * N) as st:
            st.load_terms(keys, amps)
            kg, ag, stats = run(st, gs)
            out.append((kg.tobytes(), ag.tobytes(), stats["W"]))
    assert out[0] == out[1] == out[2]


@pytest.mark.parametrize("p", [0.0, 0.9])
@pytest.mark.parametrize("N", [1, 300, 5000])
def test_few_terms_under_a_large_bound(S, N, p):
    # gates that do not branch raise the size bound fourfold each: most shares of the later steps are empty
    rng = np.random.default_rng(N)
    keys, amps = random_state(rng, 40, N)
    cz = [(pick(rng, 40, 2), CZ) for _ in range(9 if N < 1000 else 5)]
    haar = [(pick(rng, 40, m), C.haar_unitary(rng, 1 << m)) for m in (2, 1, 2)]
    # (no read between them: it would tell the host the true size)
    with S.State(40, K=1 << 19, p=p, precision="c128", capacity=1 << 19) as st:
        st.load_terms(keys, amps)
        kg, ag, stats = run(st, cz + haar)
    ko, ao, info = oracle(keys, amps, cz + haar, 1 << 19, p)
    check(kg, ag, stats, ko, ao, info, "c128")


def test_uncut_result_beyond_the_capacity(S):
    # no rule at all: refused as before, and the state goes on from the terms before the gate
    rng = np.random.default_rng(3)
    N = 150000
    keys, amps = random_state(rng, 40, N)
    g2, g1 = (pick(rng, 40, 2), C.haar_unitary(rng, 4)), (pick(rng, 40, 1), C.haar_unitary(rng, 2))
    with S.State(40, K=0, p=0.0, precision="c128", capacity=3 * N) as st:
        st.load_terms(keys, amps)
        for _ in range(2):
            st.apply_gate(*g2)
            with pytest.raises(S.CapacityError):
                st.truncate()
        kg, ag, stats = run(st, [g1])
    ko, ao, info = oracle(keys, amps, [g1], 0, 0.0)
    check(kg, ag, stats, ko, ao, dict(fraction=1.0, W=stats["W"]), "c128")


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_replayed_steps_of_full_states(S, prec):
    # every key held, steps captured once and replayed: the same terms as launched ones, bit for bit
    items = [(c, 1 << 18, 0.0) for c, _ in C.batch_workload(2, 9, n_range=(18, 18), depth_range=(4, 4), logk_range=(9, 9))]
    plain, _ = B.run_batch(items, prec, 2, 0, want_terms=True)
    for graph in (1, 8):
        res, _ = B.run_batch(items, prec, 2, graph, want_terms=True)
        for a, b in zip(plain, res):
            assert a["status"] == b["status"] == 0 and len(a["keys"]) == 1 << 18
            assert np.array_equal(a["keys"], b["keys"]) and np.array_equal(a["amps"], b["amps"])
