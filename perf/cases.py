"""The workloads whose speed matters, as calls of the public entry points.

A gate-set-tomography user evaluates the multinomial likelihood of a list of
gate sequences and its gradient, many times, for gate sets that change from
call to call.  The cases below are the forms this takes: fits over structured
lists (fiducial x germ power x fiducial), lists of random words as a fit
service receives them, many requests at once in one batch, one-off calls on
device arrays, an iteration in the CPTP parameterization, and predictions of
repeated gates.  Sizes are those of the named workloads in
``paper_2008_13490_amd.workloads`` or of their parts.

``prepare`` builds what a program has in hand before the call: the resident
request (list, counts, plan) or device arrays, and the gate set.  ``run`` is one
call.  ``exact`` evaluates the same quantities in plain float64 torch.
"""
import math

import numpy as np
import torch

from paper_2008_13490_amd import api
from paper_2008_13490_amd import workloads as W

KIND = {1: "1q", 2: "2q", 3: "3q"}
GATES = {1: 3, 2: 6, 3: 5}
# fiducial alphabets of the structured lists, as in workloads
ALPHABET = {1: (1, 2), 2: (1, 2, 3, 4), 3: (1, 2)}
SHOTS = 1000
PREPS_1Q = ((), (1, 1), (2,), (1,))


def listed():
    return [
        # the one-qubit fit list of 1,044 sequences: a call as small as a fit makes
        dict(name="fit_1q", do="fit", qubits=1, fiducials=6, germs2=0, germs3=1, power=64, probs=False),
        # the two-qubit fit list (13,189 sequences, up to 772 gates), the headline workload
        dict(name="fit_2q", do="fit", qubits=2, fiducials=11, germs2=3, germs3=3, power=256, probs=False),
        # the three-qubit fit list (200,960 sequences, up to 392 gates), the largest fit
        dict(name="fit_3q", do="fit", qubits=3, fiducials=16, germs2=20, germs3=73, power=128, probs=False),
        # sixteen two-qubit fits advanced together (bootstrap samples, several devices)
        dict(name="fits_2q_batch", do="fits", qubits=2, requests=16, fiducials=11, germs2=3, germs3=3, power=256),
        # one iteration in the CPTP mode on a list with powers to 32: parameters to gates, likelihood, chain rule
        dict(name="cptp_2q", do="mode", mode="cptp", qubits=2, fiducials=11, germs2=3, germs3=3, power=32),
        # lists of random words as a fit service receives them, 60 / 30 / 10 % one, two and three qubits
        dict(name="words_1q", do="words", qubits=1, sequences=30000, longest=256, call="eval"),
        dict(name="words_2q", do="words", qubits=2, sequences=30000, longest=256, call="eval"),
        dict(name="words_3q", do="words", qubits=3, sequences=8000, longest=128, call="eval"),
        # the autograd direction on a ragged list: probabilities, then a vector-Jacobian product
        dict(name="vjp_2q", do="words", qubits=2, sequences=3001, longest=100, call="vjp"),
        # many gate sets of uneven size in one batch (70 % one qubit, words to 1,024 gates)
        dict(name="uneven_batch", do="uneven", requests=24, fewest=500, most=20000, longest=1024),
        # a one-off call on device arrays: no request, no plan
        dict(name="plain_2q", do="plain", qubits=2, sequences=2000, longest=64),
        # predictions of r = 0 .. 1000 repetitions of every gate from four states, and their distances
        dict(name="predict_2q", do="predict", qubits=2, repetitions=1000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["fit", "fit", "fits", "mode", "words", "words", "words", "uneven", "plain", "predict"])
    if do in ("fit", "fits", "mode"):
        q = rng.choice([1, 2, 2]) if do != "fit" else rng.choice([1, 2, 3])
        nf = {1: rng.randint(4, 7), 2: rng.randint(6, 13), 3: rng.randint(6, 16)}[q]
        g2 = {1: rng.randint(0, 6), 2: rng.randint(0, 12), 3: rng.randint(0, 20)}[q]
        g3 = {1: rng.randint(0, 12), 2: rng.randint(0, 9), 3: rng.randint(0, 50)}[q]
        case = dict(do=do, qubits=q, fiducials=nf, germs2=g2, germs3=g3,
                    power=2 ** rng.randint(2, {1: 7, 2: 8, 3: 7}[q]))
        if do == "fit":
            case["probs"] = rng.random() < 0.5
        if do == "fits":
            case["requests"] = rng.randint(2, 16)
        if do == "mode":
            case["mode"] = rng.choice(["cptp", "cptp", "tp"])
        return case
    if do == "words":
        q = rng.choice([1, 1, 2, 2, 3])
        return dict(do=do, qubits=q, sequences=_log(rng, 1000, 15000 if q == 3 else 100000),
                    longest=_log(rng, 16, 128 if q == 3 else 256), call=rng.choice(["eval", "eval", "vjp"]))
    if do == "uneven":
        return dict(do=do, requests=rng.randint(4, 24), fewest=rng.randint(100, 1000), most=rng.randint(2000, 20000),
                    longest=_log(rng, 128, 1024))
    if do == "plain":
        return dict(do=do, qubits=rng.choice([1, 2]), sequences=_log(rng, 50, 20000), longest=_log(rng, 8, 256))
    return dict(do=do, qubits=rng.choice([1, 2, 2]), repetitions=_log(rng, 10, 4000))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _rngs(seed, n):
    return [np.random.default_rng(s) for s in np.random.SeedSequence(seed).spawn(n)]


def _structure(case):
    """Fiducials, germs and powers of a structured list: the experiment design, the same for every seed."""
    q = case["qubits"]
    rng = np.random.default_rng(np.random.SeedSequence([2008134901, q, case["germs2"], case["germs3"]]))
    fids = W.shortlex_words(ALPHABET[q], case["fiducials"])
    germs = W.random_germs(GATES[q], [(2, case["germs2"]), (3, case["germs3"])], rng)
    return fids, germs, [2 ** e for e in range(case["power"].bit_length())]


def _structured(case, rotations, counts_rng):
    """CSR list and counts: every F_q F_p, then F_q g^l F_p for each germ, power, p, q (F_p first in time);
    the counts are drawn from a device emulated in Hilbert space."""
    q = case["qubits"]
    truth = W.noisy_gateset(KIND[q], W.LAMBDA, W.SIGMA, rotations)
    fids, germs, powers = _structure(case)
    d, U = 2 ** q, truth.unitaries

    def product(word):
        m = np.eye(d, dtype=np.complex128)
        for k in word:
            m = U[k] @ m
        return m

    after = np.array([product(w)[:, 0] for w in fids]).T           # [d, p]: states after the preparations
    before = np.array([product(w) for w in fids])                  # [q, d, d]: the measurement fiducials
    fb = [bytes(w) for w in fids]
    lengths = np.array([len(w) for w in fids])
    words, lens, probs = [], [], []
    for body, m in [(b"", np.eye(d))] + [(bytes(g) * p, np.linalg.matrix_power(product(g), p))
                                         for g in germs for p in powers]:
        words += [fp + body + fq for fp in fb for fq in fb]
        lens.append((lengths[:, None] + len(body) + lengths[None, :]).ravel())
        probs.append((np.abs(np.einsum("qab,bp->pqa", before, m @ after)) ** 2).reshape(-1, d))
    lens, p = np.concatenate(lens), np.concatenate(probs)
    p = 1.0 / d + (1.0 - truth.lam) ** lens[:, None] * (p - 1.0 / d)
    off = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    return off, np.frombuffer(b"".join(words), np.uint8), W.sample_counts(p, SHOTS, counts_rng)


def _random(q, S, longest, words_rng, counts_rng):
    """CSR list of random words with lengths uniform in 1 .. longest, and uniform counts (workloads.serving_request)."""
    sl = W.random_list(S, GATES[q], 1, longest, words_rng)
    d = 2 ** q
    return sl.offsets, sl.gates, W.sample_counts(np.full((S, d), 1.0 / d), SHOTS, counts_rng)


def _model(q, rng):
    return W.noisy_gateset(KIND[q], W.LAMBDA, W.SIGMA, rng)


def _device(gs):
    return api.DeviceGateSet.from_numpy(gs.n_qubits, gs.rho, gs.effects, gs.gates)


def _host(case, seed):
    """The case's host data: a list of (qubits, offsets, gates, counts, gate set)."""
    if case["do"] in ("fit", "fits", "mode"):
        out = []
        for s in np.random.SeedSequence(seed).generate_state(case.get("requests", 1), np.uint64):
            a, b, c = _rngs(int(s), 3)
            out.append((case["qubits"],) + _structured(case, a, b) + (_model(case["qubits"], c),))
        return out
    if case["do"] == "uneven":
        n = case["requests"]
        mix = np.random.default_rng(np.random.SeedSequence([2008134903, n]))  # which request has which size
        ones = int(round(0.7 * n))
        kinds = np.array([1] * ones + [2] * (n - ones))[mix.permutation(n)]
        sizes = mix.integers(case["fewest"], case["most"] + 1, size=n)
        out = []
        for q, S, s in zip(kinds.tolist(), sizes.tolist(), np.random.SeedSequence(seed).generate_state(n, np.uint64)):
            r = _rngs(int(s), 3)
            out.append((q,) + _random(q, S, case["longest"], r[0], r[1]) + (_model(q, r[2]),))
        return out
    a, b, c = _rngs(seed, 3)
    q = case["qubits"]
    return [(q,) + _random(q, case["sequences"], case["longest"], a, b) + (_model(q, c),)]


def _weights(S, M, seed):
    """The upstream derivatives of a vector-Jacobian product."""
    return np.random.default_rng([seed, 7]).standard_normal((S, M))


def _predict_words(q):
    return list(W.PREDICTION_PREPS_2Q.values()) if q == 2 else list(PREPS_1Q)


def _ideal(q, model):
    return W.GateSet(q, model.names, model.rho, model.effects, W.ideal_targets(KIND[q]))


def prepare(case, seed):
    ctx = api.Context(0)
    if case["do"] == "predict":
        q = case["qubits"]
        model = _model(q, np.random.default_rng(seed))
        pred = api.Predictor(ctx, _predict_words(q), list(range(GATES[q])), case["repetitions"])
        return dict(do="predict", ctx=ctx, pred=pred, gs=_device(model), ideal=pred(_device(_ideal(q, model))))
    data = _host(case, seed)
    state = dict(do=case["do"], ctx=ctx)
    if case["do"] == "plain":
        q, off, gates, counts, model = data[0]
        return dict(state, gs=_device(model), seqs=api.DeviceSeqs.from_numpy(off, gates),
                    counts=torch.as_tensor(counts, device="cuda"))
    reqs = [api.Request(ctx, q, m.K, m.M, off, gates, counts) for q, off, gates, counts, m in data]
    sets = [_device(m) for *_, m in data]
    if case["do"] in ("fits", "uneven"):
        return dict(state, reqs=reqs, batch=api.Batch(ctx, reqs, sets))
    q, off, gates, counts, model = data[0]
    state.update(req=reqs[0], gs=sets[0], probs=case.get("probs", False), call=case.get("call", "eval"))
    if case["do"] == "mode":
        targets = torch.as_tensor(W.ideal_targets(KIND[q]), device="cuda")
        state["par"] = api.Parameterization(ctx, case["mode"], q, model.M, model.K, targets)
        state["theta"] = torch.as_tensor(W.param_point(case["mode"], model, seed), device="cuda")
    if state["call"] == "vjp":
        state["w"] = torch.as_tensor(_weights(len(off) - 1, model.M, seed), device="cuda")
    return state


def run(state):
    do = state["do"]
    if do == "predict":
        p = state["pred"](state["gs"])
        return p, api.tv_distance(state["ctx"], p, state["ideal"])
    if do == "plain":
        return state["ctx"].loglik(state["gs"], state["seqs"], state["counts"], want_probs=True)
    if do in ("fits", "uneven"):
        b = state["batch"]
        b.run()
        return b.obj, b.grad
    if do == "mode":
        gs = state["par"].forward(state["theta"])
        obj, _, g = state["req"].eval(gs)
        return obj, state["par"].backward(state["theta"], g), gs.rho, gs.effects, gs.gates
    if state["call"] == "vjp":
        return state["req"].probs(state["gs"]), state["req"].vjp(state["gs"], state["w"])
    return state["req"].eval(state["gs"], want_probs=state["probs"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    q = case.get("qubits", 2)
    if case["do"] == "predict":
        D, M, K, n = 4 ** q, 2 ** q, GATES[q], case["repetitions"] + 1
        rows = len(_predict_words(q)) * K * n
        return dict(bytes=8.0 * (K * D * D + rows * (2 * M + 1)), flops=rows * (2.0 * D * D + 2 * D * M + 3 * M))

    def one(q, S, steps, index_bytes, backward=True, weights=4):
        """steps: gates that have to be applied (shared prefixes once); 2 D^2 forward, 4 D^2 backward per step."""
        D, M, K = 4 ** q, 2 ** q, GATES[q]
        P = D + M * D + K * D * D
        return (index_bytes + 8 * S + weights * S * M + 8 * P * (2 if backward else 1),
                steps * D * D * (6.0 if backward else 2.0) + S * D * M * (6.0 if backward else 2.0))

    def structured(q):
        # distinct prefixes: per germ and preparation the germ's longest power, and at every
        # power the measurement fiducials (closed under prefixes)
        fids, germs, powers = _structure(case)
        nf = len(fids)
        S = nf * nf * (1 + len(germs) * len(powers))
        steps = nf * (nf - 1) + sum(nf * (len(g) * powers[-1] + len(powers) * (nf - 1)) for g in germs)
        total = sum(2 * nf * sum(map(len, fids)) + nf * nf * n
                    for n in [0] + [len(g) * p for g in germs for p in powers])
        return one(q, S, steps, total)

    if case["do"] in ("fit", "fits", "mode"):
        parts = [structured(q)] * case.get("requests", 1)
        if case["do"] == "fit" and case["probs"]:
            fids, germs, powers = _structure(case)
            S = len(fids) ** 2 * (1 + len(germs) * len(powers))
            parts.append((8.0 * S * 2 ** q, 0.0))
    elif case["do"] == "uneven":
        n, S = case["requests"], (case["fewest"] + case["most"]) / 2
        ones = int(round(0.7 * n))
        steps = S * (case["longest"] + 1) / 2
        parts = [one(1, S, steps, steps)] * ones + [one(2, S, steps, steps)] * (n - ones)
    else:
        S, steps = case["sequences"], case["sequences"] * (case["longest"] + 1) / 2
        if case.get("call") == "vjp":
            parts = [one(q, S, steps, steps, False, 0), one(q, S, steps, steps, True, 8), (8.0 * S * 2 ** q, 0.0)]
        else:
            parts = [one(q, S, steps, steps)]
            if case["do"] == "plain":
                parts.append((8.0 * S * 2 ** q, 0.0))
    return dict(bytes=float(sum(p[0] for p in parts)), flops=float(sum(p[1] for p in parts)))


# ---------------------------------------------------------------------------
# the same quantities in plain float64
# ---------------------------------------------------------------------------
def _reference(rho, E, G, off, gates, counts=None, w=None):
    """(objective, probabilities, gradient) by stepping all sequences together, longest first; the gradient of
    -sum N log p, or of sum w p where `w` is given."""
    dev = G.device
    K, D, _ = G.shape
    off = torch.as_tensor(np.ascontiguousarray(off), device=dev)
    gates = torch.as_tensor(np.array(gates, np.uint8), device=dev).long()
    S = off.numel() - 1
    lens = off[1:] - off[:-1]
    order = torch.argsort(lens, descending=True, stable=True)
    ls, beg = lens[order], off[:-1][order]
    longest = int(ls[0]) if S else 0
    n_at = (ls[None, :] > torch.arange(longest, device=dev)[:, None]).sum(1).tolist() if S * longest < 2 ** 27 else \
        [int((ls > t).sum()) for t in range(longest)]
    f = rho.expand(S, D).clone()
    states, picks = [], []

    def apply(M, k, x):
        if D < 64:
            return (M[k] @ x[:, :, None])[:, :, 0] if x.shape[0] < 64 else (M[k] * x[:, None, :]).sum(-1)
        y = torch.empty_like(x)
        for j in range(K):
            at = (k == j).nonzero()[:, 0]
            y[at] = x[at] @ M[j].T
        return y

    for t in range(longest):
        n = n_at[t]
        k = gates[beg[:n] + t]
        states.append(f[:n].clone())
        picks.append(k)
        f[:n] = apply(G, k, f[:n])
    p = f @ E.T
    if w is None:
        N = counts[order].double()
        objective = -(torch.where(N > 0, N * torch.log(torch.where(N > 0, p, torch.ones_like(p))), 0.0)).sum()
        dp = torch.where(N > 0, -N / p, torch.zeros_like(p))
    else:
        objective, dp = None, w[order]
    dE = dp.T @ f
    b = dp @ E
    GT = G.transpose(1, 2).contiguous()
    dG = torch.zeros_like(G)
    for t in range(longest - 1, -1, -1):
        n, k, s = n_at[t], picks[t], states[t]
        for j in range(K):
            x = torch.where((k == j)[:, None], b[:n], 0.0)
            dG[j] += x.T @ s
        b[:n] = apply(GT, k, b[:n])
        states[t] = None
    probs = torch.empty_like(p)
    probs[order] = p
    return objective, probs, torch.cat([b.sum(0), dE.reshape(-1), dG.reshape(-1)])


def _tensors(model):
    return [torch.as_tensor(np.ascontiguousarray(a), device="cuda", dtype=torch.float64)
            for a in (model.rho, model.effects, model.gates)]


def _generator(x, P, d):
    """Transfer matrix of -i[H, .] + sum_jk C_jk (P_j . P_k - {P_k P_j, .} / 2), H = sum h P / 2, C = T T^dagger,
    for parameters x = [h | diagonal of T | entries of T below it as (re, im)]."""
    D = P.shape[0]
    m = D - 1
    T = torch.diag(x[m:2 * m]).to(torch.complex128)
    low = torch.tril_indices(m, m, -1, device=x.device)
    T = T.index_put((low[0], low[1]), torch.complex(x[2 * m::2], x[2 * m + 1::2]))
    C = T @ T.conj().T
    H = torch.tensordot(x[:m].to(torch.complex128) / 2, P[1:], 1)
    Q = P[1:]
    CQ = torch.tensordot(C, Q, ([1], [0]))                  # [j]: sum_k C_jk P_k
    anti = (CQ @ Q).sum(0) / 2                              # sum_jk C_jk P_k P_j / 2
    image = -1j * (H @ P - P @ H) - (anti @ P + P @ anti)
    image = image + (Q[:, None] @ P[None] @ CQ[:, None]).sum(0)
    return (P[:, None].transpose(-1, -2) * image[None]).sum((-1, -2)).real / d


def _expm(L):
    """Taylor polynomial of L / 16, squared four times."""
    eye = torch.eye(L.shape[0], dtype=L.dtype)
    P = eye
    for k in range(22, 0, -1):
        P = eye + (L / 16) @ P / k
    for _ in range(4):
        P = P @ P
    return P


def _mode_exact(case, seed, q, off, gates, counts, model):
    """Objective and chain rule of the CPTP or TP mode by autograd through the textbook maps."""
    D, M, K, d = 4 ** q, model.M, model.K, 2 ** q
    theta = torch.as_tensor(W.param_point(case["mode"], model, seed)).requires_grad_(True)
    one = torch.zeros(D, dtype=torch.float64)
    one[0] = math.sqrt(d)
    P = torch.as_tensor(np.array(W.pauli_basis(q)))
    n = D if case["mode"] == "cptp" else D - 1
    free = theta[n:n + (M - 1) * D].reshape(M - 1, D)
    E = torch.cat([free, (one - free.sum(0))[None]])
    rest = theta[n + (M - 1) * D:].reshape(K, -1)
    if case["mode"] == "cptp":
        A = torch.diag(theta[:d]).to(torch.complex128)
        rows, cols = zip(*[(j, k) for j in range(d) for k in range(j)])
        A = A.index_put((torch.tensor(rows), torch.tensor(cols)), torch.complex(theta[d:D:2], theta[d + 1:D:2]))
        R = A @ A.conj().T
        R = R / torch.trace(R).real
        rho = (P * R.T[None]).sum((1, 2)).real / math.sqrt(d)
        targets = torch.as_tensor(W.ideal_targets(KIND[q]))
        G = torch.stack([_expm(_generator(rest[k], P, d)) @ targets[k] for k in range(K)])
    else:
        rho = torch.cat([one[:1] / d, theta[:n]])
        top = torch.zeros(K, 1, D, dtype=torch.float64)
        top[:, 0, 0] = 1.0
        G = torch.cat([top, rest.reshape(K, D - 1, D)], 1)
    parts = (rho, E, G)
    objective, _, g = _reference(*[t.detach().cuda().contiguous() for t in parts], off, gates,
                                 torch.as_tensor(counts, device="cuda"))
    grad, = torch.autograd.grad(torch.cat([t.reshape(-1) for t in parts]), theta, g.cpu())
    return [objective.reshape(1), grad] + [t.detach() for t in parts]


def exact(case, seed):
    if case["do"] == "predict":
        q = case["qubits"]
        model = _model(q, np.random.default_rng(seed))

        def predictions(rho, E, G):
            f = []
            for word in _predict_words(q):
                v = rho
                for k in word:
                    v = G[k] @ v
                f.append(v.expand(GATES[q], -1))
            f, out = torch.stack(f), []
            for _ in range(case["repetitions"] + 1):
                out.append(f @ E.T)
                f = (G[None] @ f[..., None])[..., 0]
            return torch.stack(out, 2)

        p = predictions(*_tensors(model))
        ideal = predictions(*_tensors(_ideal(q, model)))
        return p, (p - ideal).abs().sum(-1) / 2
    data = _host(case, seed)
    if case["do"] == "mode":
        return _mode_exact(case, seed, *data[0])
    if case["do"] in ("fits", "uneven"):
        out = [_reference(*_tensors(m), off, gates, torch.as_tensor(c, device="cuda")) for _, off, gates, c, m in data]
        return [o[0].reshape(1) for o in out], [o[2] for o in out]
    q, off, gates, counts, model = data[0]
    if case.get("call") == "vjp":
        w = torch.as_tensor(_weights(len(off) - 1, model.M, seed), device="cuda")
        _, p, g = _reference(*_tensors(model), off, gates, w=w)
        return p, g
    objective, p, g = _reference(*_tensors(model), off, gates, torch.as_tensor(counts, device="cuda"))
    return objective.reshape(1), p if case.get("probs") or case["do"] == "plain" else None, g
