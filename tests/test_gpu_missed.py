"""Steps above 2^17 terms whose sampled window is set, weighed and misses the
cut (needs the GPU). The sampling pass takes evenly spaced tiles, so terms whose
weights depend on their tile mislead it: the sampled tiles' are lighter or
heavier than the rest. FP64, compared with the oracle bit for bit; two further
steps would show what a missed window leaves behind."""
import numpy as np
import pytest

from paper_2607_07816_amd import circuits as C
from tests.helpers import random_state
from tests.test_gpu_bucketed import S, lin_hash, oracle, run  # noqa: F401 (S: a fixture)
from tests.test_gpu_window import check

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]


def tile_of(keys, hb, q, before):
    """The tile of each key in the step of a gate on qubits q, the last one
    having been on `before` (bkt_plan, bkt_rep of linhash.h)."""
    direction = [int(d) >> (32 - hb) for d in lin_hash(np.uint64(1) << np.arange(64, dtype=np.uint64))]
    E, pv = [], []
    for v in [direction[t] for t in q] + [direction[t] for t in before] + [1 << i for i in range(hb)]:
        if len(E) == 4:
            break
        for e, p in zip(E, pv):
            v ^= e if v >> p & 1 else 0
        if v:
            E.append(v)
            pv.append(v.bit_length() - 1)
    b = lin_hash(keys) >> np.uint64(32 - hb)
    for e, p in zip(E, pv):
        b ^= np.where(b >> np.uint64(p) & np.uint64(1), np.uint64(e), np.uint64(0))
    for p in sorted(pv, reverse=True):  # drop the pivot bits, all zero now
        b = (b >> np.uint64(p + 1) << np.uint64(p)) | (b & np.uint64((1 << p) - 1))
    return b


def misleading(rng, N, hb, stride, q, before, octaves):
    """A state whose sampled tiles (every stride-th) weigh 2^-octaves of the others."""
    keys, amps = random_state(rng, 40, N)
    sampled = tile_of(keys, hb, q, before) % np.uint64(stride) == 0
    assert abs(sampled.mean() * stride - 1) < 0.1
    return keys, amps * np.where(sampled, 2.0 ** (-octaves / 2), 1.0)


@pytest.mark.parametrize("K,p", [(150000, 0.0), (0, 0.7), (150000, 0.95)])
@pytest.mark.parametrize("octaves,below", [(0.2, 0), (1.0, 0), (2.0, 0), (-0.3, 0), (-1.0, 0), (-2.0, 0), (-1.0, 3), (0.3, 3)])
def test_window_that_misses(S, octaves, below, K, p):
    # 150,000 terms: 2^14 buckets, 1024 tiles, of which 128 are sampled; below: octaves under the previous cut (a cut
    # more than two lower is not in the slabs)
    rng = np.random.default_rng([7, int(10 * octaves + 100), K])
    N, hb, stride = 150000, 14, 8
    first, gate = (3, 17), (8, 29)
    k0, a0 = random_state(rng, 40, N)
    warm = [(first, C.haar_unitary(rng, 4))]
    keys, amps = misleading(rng, N, hb, stride, gate, first, octaves)
    amps = amps * 2.0 ** (-below / 2)
    gs = [(gate, C.haar_unitary(rng, 4)), ((1, 30), C.haar_unitary(rng, 4)), ((12,), C.haar_unitary(rng, 2))]
    with S.State(40, K=K, p=p, precision="c128", capacity=6 * N) as st:
        st.load_terms(k0, a0)
        run(st, warm)  # a previous cut, on which the sample's bins are centred
        st.load_terms(keys, amps)
        st.profile(True)
        st.kernel_times(reset=True)
        for i, g in enumerate(gs):
            keys, amps, info = oracle(keys, amps, [g], K, p)
            kg, ag, stats = run(st, [g])
            if i == 0:  # (a pass that exits at once takes some 5 us)
                t = st.kernel_times()
                print({k: round(1e3 * t[k][0]) for k in ("sample", "group_hist", "side_hist")}, flush=True)
            check(kg, ag, stats, keys, amps, info, "c128")
