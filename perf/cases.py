"""Performance cases of the simulator: what its users have it do, through its
public entry points, from the smallest circuits to the largest states.

Kinds of case (field "kind"):

  circuit   a whole peaked mirror circuit through run_circuit: a new State
            from the ground state, every gate truncated, then the peak, the
            statistics and the final terms.
  layer     steady-state simulation: a State that a circuit has filled to K
            terms, one further layer of gates (random disjoint qubit sets, as
            the random-pair workloads draw them), truncated after each, then
            the peak and the statistics. m = 2 is the plain gate stream,
            m = 3, 4, 5 are circuits fused into blocks. States of up to 2^16
            terms are read back as well; larger ones are not (their users
            read the peak only, and the total mass W, an exact sum over every
            candidate, and the candidate count follow every amplitude).
  static    one gate step on the caller's device arrays (step_static), the
            call for code that cannot allocate. Its order of terms is
            unspecified, so the result is put in ascending key order.
  handover  a state that comes from the host: load_terms, one truncated gate,
            read_terms (the step-by-step check of a trajectory).
  batch     independent uneven circuits through run_batch.
  serve     the same through a resident Server.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2607_07816_amd import _lib, batch, circuits, serve
from paper_2607_07816_amd.run import run_circuit

READ_BACK = 1 << 16  # largest steady state whose terms a layer pass reads back


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

def listed():
    return [
        # the smoke circuit: the smallest calls, launches and latency; FP64,
        # nothing is ever cut
        dict(name="circuit_n10_k1024_c128", kind="circuit", n=10, depth=4, eps=0.05, pairs="brickwork", u3=True,
             K=1024, p=0.0, prec="c128"),
        # one small serving request run alone: p-mass capped at K
        dict(name="circuit_n24_k16k_p99_c64", kind="circuit", n=24, depth=8, eps=0.02, pairs="random", u3=False,
             K=1 << 14, p=0.99, prec="c64"),
        # the allocation-free step near its limit of 65536 terms
        dict(name="static_60000_c64", kind="static", n=40, N=60000, m=2, K=65536, p=0.97, prec="c64"),
        # the batch workload's smallest K in steady state
        dict(name="layer_n20_k4k_c64", kind="layer", n=20, m=2, K=1 << 12, p=0.0, prec="c64"),
        # an odd size between the small and the large ones
        dict(name="layer_n37_k100003_c64", kind="layer", n=37, m=2, K=100003, p=0.999, prec="c64"),
        # the 24-qubit workload (K = 2^20) in FP64
        dict(name="layer_n24_k1m_c128", kind="layer", n=24, m=2, K=1 << 20, p=0.0, prec="c128"),
        # the headline: 48 qubits, K = 2^24, p = 0.99, complex64
        dict(name="layer_n48_k16m_p99_c64", kind="layer", n=48, m=2, K=1 << 24, p=0.99, prec="c64"),
        # circuits fused into blocks of 4 and of 3 qubits
        dict(name="fused4_n24_k1m_c128", kind="layer", n=24, m=4, K=1 << 20, p=0.0, prec="c128"),
        dict(name="fused3_n36_k256k_c64", kind="layer", n=36, m=3, K=1 << 18, p=0.0, prec="c64"),
        # a state handed over from the host, stepped once and read back
        dict(name="handover_n40_300007_c128", kind="handover", n=40, N=300007, m=2, K=300007, p=0.0, prec="c128"),
        # uneven circuits in flight together, and the same mix served
        dict(name="batch8_c64", kind="batch", num=8, n_lo=16, n_hi=40, d_lo=8, d_hi=12, k_lo=12, k_hi=16, p=0.0,
             streams=8, graph=0, prec="c64"),
        dict(name="serve8_c64", kind="serve", num=8, n_lo=20, n_hi=48, d_lo=8, d_hi=10, k_lo=14, k_hi=17, p=0.99,
             streams=4, graph=0, prec="c64"),
    ]


def _log_size(rng, lo, hi):
    """A size in [lo, hi], spread over its logarithm, rarely a round one."""
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    prec = rng.choice(["c64", "c64", "c128"])
    p = rng.choice([0.0, 0.0, 0.99, 0.999])
    kind = rng.choice(["layer"] * 6 + ["circuit", "circuit", "static", "static", "handover", "batch", "serve"])
    if kind == "circuit":
        return dict(kind=kind, n=rng.randint(8, 40), depth=rng.randint(4, 8), eps=round(rng.uniform(0.005, 0.05), 4),
                    pairs=rng.choice(["brickwork", "random"]), u3=rng.random() < 0.3, K=_log_size(rng, 500, 1 << 18),
                    p=p, prec=prec)
    if kind == "static":
        return dict(kind=kind, n=rng.randint(18, 64), N=_log_size(rng, 50, 65536), m=rng.randint(1, 3),
                    K=_log_size(rng, 50, 65536), p=p, prec=prec)
    if kind == "handover":
        size = _log_size(rng, 1000, 1 << 20)
        return dict(kind=kind, n=rng.randint(24, 64), N=size, m=rng.randint(1, 3), K=size, p=p, prec=prec)
    if kind in ("batch", "serve"):
        return dict(kind=kind, num=rng.randint(3, 9), n_lo=16, n_hi=rng.randint(24, 48), d_lo=6, d_hi=rng.randint(8, 12),
                    k_lo=12, k_hi=rng.randint(13, 17), p=p, streams=rng.choice([2, 4, 8]),
                    graph=rng.choice([0, 16]) if kind == "batch" else 0, prec=prec)
    m = rng.choice([1, 2, 2, 2, 2, 2, 2, 3, 4, 5])
    return dict(kind=kind, n=rng.randint(26, 64), m=m, K=_log_size(rng, 1 << 10, 1 << (23 if m <= 2 else 20)), p=p,
                prec=prec)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _layers(rng, n, m, count):
    """`count` layers of Haar gates on random disjoint sets of m qubits."""
    out = []
    for _ in range(count):
        perm = rng.permutation(n)
        out.append([(tuple(int(q) for q in perm[m * i: m * i + m]), circuits.haar_unitary(rng, 1 << m))
                    for i in range(n // m)])
    return out


def _layer_plan(case, seed):
    """Warm-up gates (until the state holds K terms, and two gates more) and
    the layers that passes apply in turn."""
    rng = np.random.default_rng([seed, 11])
    n, m = case["n"], case["m"]
    need = -(-int(case["K"]).bit_length() // m) + 2
    warm = [g for l in _layers(rng, n, m, -(-need * m // (n - n % m)) + 1) for g in l]
    return warm, _layers(rng, n, m, 4)


def _state_terms(case, seed):
    """N distinct keys of n bits with Gaussian amplitudes, normalised (FP64,
    rounded to FP32 for complex64 states)."""
    rng = np.random.default_rng([seed, 12])
    n, N = case["n"], case["N"]
    keys = np.zeros(0, dtype=np.uint64)
    while len(keys) < N:
        more = rng.integers(0, (1 << n) - 1, size=N + N // 4 + 16, dtype=np.uint64, endpoint=True)
        keys = np.unique(np.concatenate([keys, more]))
    keys = rng.permutation(keys)[:N]
    amps = rng.standard_normal(N) + 1j * rng.standard_normal(N)
    amps /= np.linalg.norm(amps)
    if case["prec"] == "c64":
        amps = amps.astype(np.complex64).astype(np.complex128)
    qs = tuple(int(q) for q in rng.choice(n, size=case["m"], replace=False))
    return keys, amps, qs, circuits.haar_unitary(rng, 1 << case["m"])


def _circuit(case, seed):
    return circuits.peaked_circuit(case["n"], case["depth"], case["eps"], seed, pairs=case["pairs"],
                                   u3_layers=case["u3"])


def _items(case, seed):
    rng = np.random.default_rng([seed, 13])
    out = []
    for i in range(case["num"]):
        n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
        d = int(rng.integers(case["d_lo"], case["d_hi"] + 1))
        # sizes stepped evenly over the range, so that every seed's mix costs alike
        logk = case["k_lo"] + (case["k_hi"] - case["k_lo"]) * i // max(case["num"] - 1, 1)
        c = circuits.peaked_circuit(n, d, float(rng.uniform(0.005, 0.05)), int(rng.integers(0, 2**31 - 1)),
                                    pairs="random", u3_layers=False)
        out.append((c, 1 << logk, case["p"] if i % 2 else 0.0))
    return out


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind == "circuit":
        s["circuit"] = _circuit(case, seed)
    elif kind == "layer":
        warm, s["layers"] = _layer_plan(case, seed)
        # 4-qubit blocks run tiled while the state holds at most half the capacity
        cap = 2 * case["K"] if case["m"] >= 4 else case["K"]
        st = _lib.State(case["n"], K=case["K"], p=case["p"], precision=case["prec"], capacity=max(cap, 4096))
        for qs, U in warm:
            st.apply_gate(qs, U)
            st.truncate()
        s["state"], s["next"] = st, 0
    elif kind == "static":
        keys, amps, s["qs"], s["U"] = _state_terms(case, seed)
        dev = torch.device("cuda")
        dt = torch.complex128 if case["prec"] == "c128" else torch.complex64
        s["keys"] = torch.from_numpy(keys.view(np.int64)).to(dev)
        s["amps"] = torch.from_numpy(amps).to(dev).to(dt)
        room = _room(case)
        s["out_keys"] = torch.zeros(room, dtype=torch.int64, device=dev)
        s["out_amps"] = torch.zeros(room, dtype=dt, device=dev)
        s["out_n"] = torch.zeros(1, dtype=torch.int64, device=dev)
        s["stats"] = torch.zeros(2, dtype=torch.float64, device=dev)
    elif kind == "handover":
        s["keys"], s["amps"], s["qs"], s["U"] = _state_terms(case, seed)
        s["state"] = _lib.State(case["n"], K=case["K"], p=case["p"], precision=case["prec"], capacity=case["N"])
    elif kind == "batch":
        s["items"] = _items(case, seed)
        s["packed"] = batch.pack(s["items"], want_terms=True)
    elif kind == "serve":
        s["items"] = _items(case, seed)
        s["server"] = serve.Server(precision=case["prec"], streams=case["streams"], max_active=4, gates_per_turn=8,
                                   hbm_bytes=1 << 30)
    else:
        raise ValueError(kind)
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def _key(k):
    return np.array([k], dtype=np.uint64).view(np.int64)


def _figures(st):
    key, prob = st.peak()
    f = st.stats()
    return dict(peak_key=_key(key), peak_prob=prob, n_terms=st.num_terms(), W=f["W"], kept=f["kept_fraction"],
                log10_cum=f["log10_cum_kept"], candidates=f["candidates"])


def _room(case):
    return min(case["K"], 1 << min(case["n"], 62))


def _terms(keys, amps, room):
    """The terms; where a p-mass cut kept fewer than K, filled up with key -1
    and amplitude 0, so that their number shows in n_terms and not in shapes."""
    keys, short = keys.view(np.int64), room - len(keys)
    if short > 0:
        keys = np.concatenate([keys, np.full(short, -1, dtype=np.int64)])
        amps = np.concatenate([amps, np.zeros(short, dtype=amps.dtype)])
    return dict(keys=keys, amps=amps)


def _result(r, circuit, K):
    return dict(peak_key=_key(r["peak_key"]), peak_prob=r["peak_prob"], n_terms=r["n_terms"],
                log10_cum=r["log10_cum_kept"],
                **_terms(r["keys"], r["amps"], _room(dict(n=circuit.n, K=K))))


def run_circuit_pass(s):
    case = s["case"]
    with run_circuit(s["circuit"], K=case["K"], p=case["p"], precision=case["prec"],
                     capacity=max(case["K"], 4096)) as st:
        out = _figures(st)
        out.update(_terms(*st.read_terms(), _room(case)))
    return out


def run_layer_pass(s):
    st = s["state"]
    for qs, U in s["layers"][s["next"] % len(s["layers"])]:
        st.apply_gate(qs, U)
        st.truncate()
    s["next"] += 1
    out = _figures(st)
    if s["case"]["K"] <= READ_BACK:
        out.update(_terms(*st.read_terms(), _room(s["case"])))
    return out


def run_static_pass(s):
    case = s["case"]
    _lib.step_static(case["n"], case["K"], case["p"], case["prec"], s["qs"], s["U"], s["keys"].data_ptr(),
                     s["amps"].data_ptr(), case["N"], s["out_keys"].data_ptr(), s["out_amps"].data_ptr(),
                     s["out_n"].data_ptr(), s["stats"].data_ptr(), torch.cuda.current_stream().cuda_stream)
    n = int(s["out_n"].item())
    keys, order = torch.sort(s["out_keys"][:n])
    amps = s["out_amps"][:n][order]
    if short := _room(case) - n:
        keys = torch.nn.functional.pad(keys, (0, short), value=-1)
        amps = torch.cat([amps, amps.new_zeros(short)])
    return dict(keys=keys, amps=amps, n_terms=n, stats=s["stats"])


def run_handover_pass(s):
    st = s["state"]
    st.load_terms(s["keys"], s["amps"])
    st.apply_gate(s["qs"], s["U"])
    st.truncate()
    keys, amps = st.read_terms()
    f = st.stats()
    return dict(n_terms=len(keys), W=f["W"], kept=f["kept_fraction"], candidates=f["candidates"],
                **_terms(keys, amps, _room(s["case"])))


def run_batch_pass(s):
    case = s["case"]
    res, _ = batch.run_batch(s["items"], case["prec"], case["streams"], case["graph"], packed=s["packed"])
    return [_result(r, c, K) for r, (c, K, _) in zip(res, s["items"])]


def run_serve_pass(s):
    srv = s["server"]
    tickets = [srv.submit(c, K=K, p=p, want_terms=True) for c, K, p in s["items"]]
    return [_result(srv.wait(t), c, K) for t, (c, K, _) in zip(tickets, s["items"])]


PASS = dict(circuit=run_circuit_pass, layer=run_layer_pass, static=run_static_pass, handover=run_handover_pass,
            batch=run_batch_pass, serve=run_serve_pass)


def run(state):
    return PASS[state["case"]["kind"]](state)


# --------------------------------------------------------------------------
# what a pass cannot do without: every gate step reads the state once and
# writes the new one once, and multiplies each term into its 2^m outputs
# --------------------------------------------------------------------------

def _step_work(n_in, n_out, m, prec):
    term = 24 if prec == "c128" else 16
    return term * (n_in + n_out), 8.0 * (1 << m) * n_in


def _circuit_work(n, gates, K, prec):
    size, by, fl = 1.0, 0.0, 0.0
    for m in gates:
        new = min(size * (1 << m), float(K), 2.0 ** n)
        b, f = _step_work(size, new, m, prec)
        by, fl, size = by + b, fl + f, new
    return by, fl


def work(case):
    kind, prec = case["kind"], case["prec"]
    if kind == "circuit":
        per = 2 * case["depth"]
        gates = ([2] * (case["n"] // 2) + [1] * (case["n"] if case["u3"] else 0)) * per
        by, fl = _circuit_work(case["n"], gates, case["K"], prec)
        by += (32 if prec == "c128" else 24) * min(case["K"], 2.0 ** case["n"])
    elif kind == "layer":
        size = min(case["K"], 2.0 ** case["n"])
        b, f = _step_work(size, size, case["m"], prec)
        g = case["n"] // case["m"]
        by, fl = b * g, f * g
        if case["K"] <= READ_BACK:
            by += (24 + (24 if prec == "c128" else 16)) * size
    elif kind == "static":
        by, fl = _step_work(case["N"], min(case["K"], case["N"] << case["m"]), case["m"], prec)
    elif kind == "handover":
        by, fl = _step_work(case["N"], case["N"], case["m"], prec)
        by += 2 * (24 + (24 if prec == "c128" else 16)) * case["N"]  # to the device and back
    else:
        by = fl = 0.0
        n, d = (case["n_lo"] + case["n_hi"]) // 2, (case["d_lo"] + case["d_hi"]) // 2
        for i in range(case["num"]):
            logk = case["k_lo"] + (case["k_hi"] - case["k_lo"]) * i // max(case["num"] - 1, 1)
            b, f = _circuit_work(n, [2] * (n // 2 * 2 * d), 1 << logk, prec)
            by, fl = by + b, fl + f
    return {"bytes": float(by), "flops": float(fl)}


# --------------------------------------------------------------------------
# the same in plain numpy, FP64: expand every term by its column of U, add up
# equal keys, rank, cut, renormalise
# --------------------------------------------------------------------------

def _np_apply(keys, amps, qs, U):
    m = len(qs)
    one = np.uint64(1)
    pat = np.zeros(len(keys), dtype=np.int64)
    rest = keys.copy()
    for t, q in enumerate(qs):
        pat |= ((keys >> np.uint64(q)) & one).astype(np.int64) << t
        rest &= ~(one << np.uint64(q))
    rests, inv = np.unique(rest, return_inverse=True)
    dense = np.zeros((len(rests), 1 << m), dtype=np.complex128)
    dense[inv, pat] = amps
    new = dense @ np.asarray(U).T
    present = np.ones(new.shape, dtype=bool) & (new != 0)
    dep = np.zeros(1 << m, dtype=np.uint64)
    for i in range(1 << m):
        for t, q in enumerate(qs):
            if (i >> t) & 1:
                dep[i] |= one << np.uint64(q)
    out = rests[:, None] | dep[None, :]
    return out[present], new[present]


def _np_truncate(keys, amps, K, p, trace):
    w = amps.real ** 2 + amps.imag ** 2
    W = float(w.sum())
    order = np.lexsort((keys, -w))
    L = len(order)
    if 0.0 < p < 1.0:
        c = np.cumsum(w[order])
        L = min(L, int(np.searchsorted(c, p * W)) + 1)
    if K:
        L = min(L, K)
    kept = order[:L]
    S = float(w[kept].sum())
    dropped = L < len(order)
    trace.update(W=W, kept=S / W if dropped else 1.0, candidates=len(order))
    trace["log10_cum"] = trace.get("log10_cum", 0.0) + (np.log10(S / W) if dropped else 0.0)
    return keys[kept], amps[kept] / np.sqrt(S) if dropped else amps[kept]


def _np_steps(keys, amps, gates, flags, K, p, trace):
    for (qs, U), cut in zip(gates, flags):
        keys, amps = _np_apply(keys, amps, qs, U)
        if cut:
            keys, amps = _np_truncate(keys, amps, K, p, trace)
    return keys, amps


def _exact_terms(amps, room):
    return dict(keys=None, amps=np.concatenate([amps, np.zeros(max(room - len(amps), 0), dtype=amps.dtype)]))


def _ground():
    return np.zeros(1, dtype=np.uint64), np.ones(1, dtype=np.complex128)


def _np_figures(keys, amps, trace, room):
    w = amps.real ** 2 + amps.imag ** 2
    best = np.lexsort((keys, -w))[0]
    o = np.argsort(keys)
    return dict(peak_key=None, peak_prob=float(w[best] / w.sum()), n_terms=None, W=trace["W"], kept=trace["kept"],
                log10_cum=trace["log10_cum"], candidates=None, **_exact_terms(amps[o], room))


def exact(case, seed):
    """FP64 in plain numpy. complex64 states of several cut steps have none:
    near-ties at a cut fall either way in FP32, and the kept terms differ."""
    kind, K, p, trace = case["kind"], case.get("K"), case["p"], {}
    if kind in ("batch", "serve"):
        return None
    if kind in ("static", "handover"):
        keys, amps, qs, U = _state_terms(case, seed)
        keys, amps = _np_steps(keys, amps, [(qs, U)], [True], _room(case), p, trace)
        if kind == "static":
            out = _exact_terms(amps[np.argsort(keys.view(np.int64))], _room(case))
            return dict(keys=None, amps=torch.from_numpy(out["amps"]), n_terms=None,
                        stats=torch.tensor([trace["W"], trace["kept"]], dtype=torch.float64))
        return dict(n_terms=None, W=trace["W"], kept=trace["kept"], candidates=None,
                    **_exact_terms(amps[np.argsort(keys)], _room(case)))
    if kind == "circuit":
        c = _circuit(case, seed)
        cuts = p > 0 or K < (1 << case["n"])
        if K * len(c.gates) > (1 << 22) or (cuts and case["prec"] == "c64"):
            return None
        keys, amps = _np_steps(*_ground(), c.gates, c.truncate_after, K, p, trace)
        return _np_figures(keys, amps, trace, _room(case))
    warm, layers = _layer_plan(case, seed)
    gates = warm + layers[0]
    if case["prec"] == "c64" or K * len(gates) << case["m"] > (1 << 25):
        return None
    keys, amps = _np_steps(*_ground(), gates, [True] * len(gates), K, p, trace)
    out = _np_figures(keys, amps, trace, _room(case))
    if K > READ_BACK:
        del out["keys"], out["amps"]
    return out
