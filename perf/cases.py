"""The work that users of this framework have it do, as cases to be timed.

A case is one call (or one training step) through the public entry points, at
sizes taken from the repository's workloads, its tests and their neighbourhood:

  cumulants  correlators and cumulants of all subsets up to order K
             (click or parity, FP64 or mixed form)
  displaced  the same for a state with first moments
  batched    many covariances of uneven size in one call
  shard      one rank range of one order of a large problem
  fit        one step of fitting transmissions and squeezings to cumulants
             (forward, loss, backward)
  sample     click patterns from parity cumulants (single or double elision)
  estimate   click cumulants estimated from samples, optionally with the Pearson
             coefficient of every order against the ground truth

`listed` holds the named ones, `draw` gives others of the same ranges, `prepare`
makes the inputs, `run` is one pass, `work` the bytes and operations that a pass
cannot do without, and `exact` the same outputs in plain torch, FP64.
"""
import itertools
import math

import numpy as np
import torch

import paper_2511_14923_amd as P

DEV = "cuda"
F64 = torch.float64


# ---------------------------------------------------------------------------
# the cases


def listed():
    return [
        # the smallest call: a 16-mode state, third order; latency and launches count
        {"name": "cumulants_m16_k3", "kind": "cumulants", "M": 16, "K": 3, "parity": False, "mixed": False},
        # a 100-mode state, parity cumulants as the sampler takes them
        {"name": "cumulants_m100_k4", "kind": "cumulants", "M": 100, "K": 4, "parity": True, "mixed": False},
        # the headline problem: the ground truth of a 144-mode state, all orders up to 5
        {"name": "cumulants_m144_k5", "kind": "cumulants", "M": 144, "K": 5, "parity": False, "mixed": False},
        # the mixed form, at a size that is no multiple of anything
        {"name": "mixed_m121_k5", "kind": "cumulants", "M": 121, "K": 5, "parity": False, "mixed": True},
        # a displaced state of medium, odd size
        {"name": "displaced_m87_k5", "kind": "displaced", "M": 87, "K": 5, "parity": False},
        # a sweep: 48 covariances of 40 to 144 modes in one call
        {"name": "batched48_k4", "kind": "batched", "count": 48, "m_lo": 40, "m_hi": 144, "sizes": 25110004,
         "K": 4, "mixed": False},
        # one device's share of a pseudo-photon-number-resolving problem (144 modes
        # on 8 detectors each), a ragged range in the middle of order 5
        {"name": "shard_m1152_k5", "kind": "shard", "M0": 144, "split": 8, "order": 5, "count": 100000007},
        # one step of a fit to third-order click cumulants
        {"name": "fit_m144_k3", "kind": "fit", "M": 144, "K": 3},
        # single-elision samples of a 144-mode state
        {"name": "sample_m144_k3", "kind": "sample", "M": 144, "K": 3, "n": 65536},
        # double-elision samples of a 100-mode state
        {"name": "sample_m100_k5", "kind": "sample", "M": 100, "K": 5, "n": 4096},
        # all click cumulants of a large data set
        {"name": "estimate_m144_k5", "kind": "estimate", "M": 144, "K": 5, "n": 262144, "pearson": False},
        # validation of a medium data set: estimates and Pearson coefficients
        {"name": "validate_m60_k4", "kind": "estimate", "M": 60, "K": 4, "n": 50001, "pearson": True},
    ]


def draw(rng):
    def log_int(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(["cumulants", "cumulants", "displaced", "batched", "shard", "fit", "sample", "sample",
                       "estimate"])
    if kind in ("cumulants", "displaced"):
        K = rng.choice([2, 3, 4, 5])
        M = log_int(6, {2: 400, 3: 300, 4: 180, 5: 140}[K])
        c = {"kind": kind, "M": M, "K": K, "parity": rng.random() < 0.5}
        if kind == "cumulants":
            c["mixed"] = rng.random() < 0.25
        return c
    if kind == "batched":
        lo = rng.randint(6, 60)
        return {"kind": kind, "count": log_int(2, 64), "m_lo": lo, "m_hi": rng.randint(lo + 1, 120),
                "sizes": rng.randrange(1 << 30), "K": rng.choice([3, 4]), "mixed": rng.random() < 0.25}
    if kind == "shard":
        M0, split, order = rng.randint(20, 144), rng.choice([1, 2, 4, 8]), rng.choice([3, 4, 5])
        M = M0 * split
        return {"kind": kind, "M0": M0, "split": split, "order": order,
                "count": log_int(1000, min(80_000_000, math.comb(M, order)))}
    if kind == "fit":
        K = rng.choice([2, 3, 3, 4])
        return {"kind": kind, "M": log_int(6, {2: 160, 3: 140, 4: 48}[K]), "K": K}
    if kind == "sample":
        if rng.random() < 0.5:
            return {"kind": kind, "M": log_int(8, 180), "K": 3, "n": log_int(50, 30000)}
        return {"kind": kind, "M": log_int(8, 90), "K": 5, "n": log_int(50, 4000)}
    K = rng.choice([3, 4, 5])
    return {"kind": kind, "M": log_int(10, {3: 200, 4: 120, 5: 80}[K]), "K": K, "n": log_int(300, 300000),
            "pearson": rng.random() < 0.5}


# ---------------------------------------------------------------------------
# inputs: Haar interferometers with squeezing and loss (xxpp order, vacuum = I/2)


def _haar(M, rng):
    z = (rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))) / math.sqrt(2.0)
    q, r = np.linalg.qr(z)
    d = np.diag(r)
    return q * (d / np.abs(d))[None, :]


def _symplectic(T):
    return torch.from_numpy(np.block([[T.real, -T.imag], [T.imag, T.real]])).to(DEV)


def _covariance(W, r, eta):
    """Input loss eta and squeezing r through the interferometer W (differentiable)."""
    d = torch.cat([0.5 * eta * torch.exp(-2.0 * r) + 0.5 * (1.0 - eta),
                   0.5 * eta * torch.exp(2.0 * r) + 0.5 * (1.0 - eta)])
    s = (W * d.unsqueeze(0)) @ W.T
    return 0.5 * (s + s.T)


def _state(M, rng):
    """(W, r, eta) of one instance: squeezing and transmissions of the 144-mode workload."""
    U = _haar(M, rng)
    r = torch.from_numpy(rng.uniform(0.6, 1.6, M)).to(DEV)
    eta = torch.from_numpy(rng.uniform(0.25, 0.4, M)).to(DEV)
    return U, _symplectic(U), r, eta


def _mean(U, eta, rng):
    M = U.shape[0]
    amp = np.sqrt(rng.uniform(0.05, 0.5, M)) * np.exp(1j * rng.uniform(0.0, 2 * math.pi, M))
    v = torch.from_numpy(math.sqrt(2.0) * np.concatenate([amp.real, amp.imag])).to(DEV)
    return _symplectic(U * np.sqrt(eta.cpu().numpy())[None, :]) @ v


def _split_modes(sigma, k):
    """Every mode split evenly over k detectors (k x k Fourier transform with k - 1 vacua)."""
    M0 = sigma.shape[0] // 2
    M = M0 * k
    s = 0.5 * torch.eye(2 * M, dtype=F64, device=DEV)
    at = torch.arange(M0, device=DEV) * k
    at = torch.cat([at, at + M])
    s[at.unsqueeze(1), at.unsqueeze(0)] = sigma
    F = np.exp(2j * math.pi * np.outer(np.arange(k), np.arange(k)) / k) / math.sqrt(k)
    W = _symplectic(np.kron(np.eye(M0), F))
    s = W @ s @ W.T
    return 0.5 * (s + s.T)


def _shard_start(case):
    """A range in the middle of the order."""
    total = math.comb(case["M0"] * case["split"], case["order"])
    return (total - case["count"]) // 2


def _batch_sizes(case):
    """The instances' modes: part of the case, not of its inputs."""
    rng = np.random.default_rng(case["sizes"])
    return [max(int(m), case["K"]) for m in rng.integers(case["m_lo"], case["m_hi"] + 1, size=case["count"])]


def _padded(n):
    return -(-n // 32) * 32


def _click_bits(n, M, gen):
    """Correlated clicks: a shared factor beside each mode's own, thresholded per mode."""
    out = torch.empty((n, M), dtype=torch.uint8, device=DEV)
    load = 0.2 + 0.3 * torch.rand((3, M), device=DEV, generator=gen)
    thr = 0.3 + 0.6 * torch.rand(M, device=DEV, generator=gen)
    for a in range(0, n, 1 << 18):
        b = min(n, a + (1 << 18))
        z = torch.randn((b - a, 3), device=DEV, generator=gen)
        own = torch.randn((b - a, M), device=DEV, generator=gen)
        out[a:b] = (own + (z.unsqueeze(2) * load.unsqueeze(0)).sum(1) > thr).to(torch.uint8)
    return out


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind in ("cumulants", "displaced", "fit"):
        U, W, r, eta = _state(case["M"], rng)
        st = {"case": case, "sigma": _covariance(W, r, eta).contiguous()}
        if kind == "displaced":
            st["mu"] = _mean(U, eta, rng).contiguous()
        if kind == "fit":
            r2 = torch.from_numpy(rng.uniform(0.6, 1.6, case["M"])).to(DEV)
            e2 = torch.from_numpy(rng.uniform(0.25, 0.4, case["M"])).to(DEV)
            st |= {"W": W, "r": r.requires_grad_(), "eta": eta.requires_grad_(),
                   "target": _plain(_covariance(W, r2, e2), case["K"])[1]}
        return st
    if kind == "batched":
        Ms = _batch_sizes(case)
        # every instance's outputs are slices of one buffer, on 256-byte boundaries
        ns = [sum(math.comb(M, d) for d in range(1, case["K"] + 1)) for M in Ms]
        at = np.cumsum([0] + [_padded(n) for n in ns])
        corr, cum = (torch.zeros(int(at[-1]), dtype=F64, device=DEV) for _ in range(2))
        inst = []
        for M, n, a in zip(Ms, ns, at):
            _, W, r, eta = _state(M, rng)
            inst.append((M, _covariance(W, r, eta).contiguous(), corr[a:a + n], cum[a:a + n]))
        return {"case": case, "inst": inst, "corr": corr, "cum": cum}
    if kind == "shard":
        _, W, r, eta = _state(case["M0"], rng)
        return {"case": case, "sigma": _split_modes(_covariance(W, r, eta), case["split"]).contiguous()}
    if kind == "sample":
        _, W, r, eta = _state(case["M"], rng)
        gen = torch.Generator(device=DEV).manual_seed(int(rng.integers(1 << 40)))
        return {"case": case, "kappa": _plain(_covariance(W, r, eta), case["K"], parity=True)[1],
                "u": torch.rand((case["M"], case["n"]), dtype=F64, device=DEV, generator=gen)}
    gen = torch.Generator(device=DEV).manual_seed(int(rng.integers(1 << 40)))
    st = {"case": case, "bits": _click_bits(case["n"], case["M"], gen)}
    if case["pearson"]:  # the ground truth to compare with
        _, W, r, eta = _state(case["M"], rng)
        st["truth"] = _plain(_covariance(W, r, eta), case["K"])[1]
    return st


# ---------------------------------------------------------------------------
# one pass


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind in ("cumulants", "displaced"):
        flags = P.GBS_PARITY if case["parity"] else P.GBS_CLICK
        if kind == "displaced":
            return P.gbs_cumulants_displaced(case["M"], st["sigma"], st["mu"], case["K"], flags)
        return P.gbs_cumulants(case["M"], st["sigma"], case["K"], flags | (P.GBS_MIXED if case["mixed"] else 0))
    if kind == "batched":
        P.gbs_cumulants_batched(st["inst"], case["K"], P.GBS_MIXED if case["mixed"] else 0)
        return st["corr"], st["cum"]
    if kind == "shard":
        return P.gbs_cumulants_shard(case["M0"] * case["split"], st["sigma"], case["order"], _shard_start(case),
                                     case["count"])
    if kind == "fit":
        st["r"].grad = st["eta"].grad = None
        loss = P.cumulant_matching_loss(st["W"], st["r"], st["eta"], st["target"], case["K"])
        loss.backward()
        return loss.detach(), st["r"].grad, st["eta"].grad
    if kind == "sample":
        bits, prob, _ = P.gbs_sample(case["M"], st["kappa"], case["K"], st["u"])
        return bits, prob
    cum = P.gbs_sample_cumulants(st["bits"], case["K"])
    if not case["pearson"]:
        return cum
    rs, at = [], 0
    for d in range(1, case["K"] + 1):
        n = math.comb(case["M"], d)
        rs.append(P.gbs_pearson(cum[at:at + n], st["truth"][at:at + n]))
        at += n
    return [cum] + rs


# ---------------------------------------------------------------------------
# what a pass cannot do without


def _subset_flops(d):
    """A new mode's block against the shared factors of the rest of the subset, one
    determinant, and the two sums over its 2^(d-1) new probabilities."""
    return 16.0 * (d - 1) + 10.0 + 2.0 * 2.0 ** d


def work(case):
    kind = case["kind"]
    if kind == "batched":
        w = [work({"kind": "cumulants", "M": m, "K": case["K"]}) for m in _batch_sizes(case)]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    if kind == "shard":
        M = case["M0"] * case["split"]
        return {"bytes": 8.0 * M * (2 * M + 1) + 16.0 * case["count"],
                "flops": case["count"] * _subset_flops(case["order"])}
    M, K = case["M"], case["K"]
    outs = [math.comb(M, d) for d in range(1, K + 1)]
    N = sum(outs)
    if kind in ("cumulants", "displaced"):
        return {"bytes": 8.0 * M * (2 * M + 1) + 16.0 * N,
                "flops": sum(c * _subset_flops(d + 1) for d, c in enumerate(outs))}
    if kind == "fit":
        # forward, the target read for the loss, and twice the forward's operations backward
        return {"bytes": 2 * 8.0 * 4 * M * M + 24.0 * N + 64.0 * M,
                "flops": 3 * sum(c * _subset_flops(d + 1) for d, c in enumerate(outs))}
    if kind == "sample":
        # the expansion's terms, and the updates of the marginals
        n = case["n"]
        terms = 2.0 * N + (6.0 * math.comb(M, 4) if K == 5 else 4.0 * math.comb(M, 3))
        return {"bytes": 8.0 * N + n * (9.0 * M + 8.0), "flops": n * terms}
    return {"bytes": 1.0 * case["n"] * M + 8.0 * N + (16.0 * N if case["pearson"] else 0.0),
            "flops": 2.0 * case["n"] * sum(outs[1:])}


# ---------------------------------------------------------------------------
# the same outputs in plain torch, 64 bits


CHUNK = 1 << 22


def _binomials(M, K):
    return torch.tensor([[math.comb(n, k) for n in range(M + 1)] for k in range(K + 1)], dtype=torch.int64, device=DEV)


def _unrank(r, d, binom):
    """Ascending members of the d-subsets of colex ranks r."""
    r, s = r.clone(), [None] * d
    for j in range(d, 0, -1):
        s[j - 1] = torch.searchsorted(binom[j], r, right=True) - 1
        r -= binom[j][s[j - 1]]
    return s


def _vacuum(Q, S, mu=None):
    """p of the subsets with members S (a list of index tensors), by Cholesky."""
    M = Q.shape[0] // 2
    idx = [i for s in S for i in (s, s + M)]
    flat, n = Q.reshape(-1), len(idx)
    L, z, det = [[None] * n for _ in range(n)], [], None
    for i in range(n):
        base = idx[i] * (2 * M)
        for j in range(i + 1):
            v = flat[base + idx[j]]
            for k in range(j):
                v = v - L[i][k] * L[j][k]
            if i == j:
                det = v if det is None else det * v
                L[i][i] = torch.sqrt(v)
            else:
                L[i][j] = v / L[j][j]
        if mu is not None:
            v = mu[idx[i]]
            for k in range(i):
                v = v - L[i][k] * z[k]
            z.append(v / L[i][i])
    p = torch.rsqrt(det)
    return p if mu is None else p * torch.exp(-0.5 * sum(v * v for v in z))


def _partitions(d):
    """Set partitions of range(d) as lists of bit masks."""
    def rec(i, blocks):
        if i == d:
            yield list(blocks)
            return
        for b in range(len(blocks)):
            blocks[b] |= 1 << i
            yield from rec(i + 1, blocks)
            blocks[b] ^= 1 << i
        blocks.append(1 << i)
        yield from rec(i + 1, blocks)
        blocks.pop()
    return list(rec(0, []))


def _moments(p, d, parity):
    """Correlators of every sub-subset (by mask) from the probabilities p[mask] (p[0] = None)."""
    out = [None] * (1 << d)
    for B in range(1, 1 << d):
        size, acc, T = bin(B).count("1"), 0.0, B
        while T:
            t = bin(T).count("1")
            acc = acc + ((-2.0) ** t if parity else (-1.0) ** t) * p[T]
            T = (T - 1) & B
        out[B] = (acc + 1.0) * ((-1.0) ** size if parity else 1.0)
    return out


def _cumulant(m, d):
    acc = 0.0
    for blocks in _partitions(d):
        v = (-1.0) ** (len(blocks) - 1) * math.factorial(len(blocks) - 1)
        for b in blocks:
            v = v * m[b]
        acc = acc + v
    return acc


def _plain(sigma, K, mu=None, parity=False):
    """(correlators, cumulants) of all subsets of orders 1..K, order blocks in colex order."""
    M = sigma.shape[0] // 2
    Q = torch.tril(sigma)
    Q = Q + torch.tril(Q, -1).T + 0.5 * torch.eye(2 * M, dtype=F64, device=DEV)
    binom = _binomials(M, K)
    p, corr, cum = [None], [None], [None]
    for d in range(1, K + 1):
        n = math.comb(M, d)
        parts = []
        for a in range(0, n, CHUNK):
            r = torch.arange(a, min(n, a + CHUNK), device=DEV)
            S = _unrank(r, d, binom)
            new = _vacuum(Q, S, mu)
            full = (1 << d) - 1
            at = [None] * (1 << d)
            for B in range(1, full):
                mem = [S[i] for i in range(d) if B >> i & 1]
                at[B] = sum(binom[j + 1][s] for j, s in enumerate(mem))
            size = [bin(B).count("1") for B in range(1 << d)]
            ps = [None] + [p[size[B]][at[B]] for B in range(1, full)] + [new]
            acc = 1.0
            for B in range(1, 1 << d):
                acc = acc + ((-2.0) ** size[B] if parity else (-1.0) ** size[B]) * ps[B]
            c = acc * ((-1.0) ** d if parity else 1.0)
            m = [None] + [corr[size[B]][at[B]] for B in range(1, full)] + [c]
            parts.append((new, c, _cumulant(m, d)))
        for to, k in ((p, 0), (corr, 1), (cum, 2)):
            to.append(torch.cat([x[k] for x in parts]))
        del parts
    return torch.cat(corr[1:]), torch.cat(cum[1:])


def _plain_range(sigma, d, r0, count):
    M = sigma.shape[0] // 2
    Q = sigma + 0.5 * torch.eye(2 * M, dtype=F64, device=DEV)
    binom = _binomials(M, d)
    out = torch.empty((2, count), dtype=F64, device=DEV)
    for a in range(0, count, CHUNK):
        b = min(count, a + CHUNK)
        S = _unrank(torch.arange(r0 + a, r0 + b, device=DEV), d, binom)
        p = [None] + [_vacuum(Q, [S[i] for i in range(d) if B >> i & 1]) for B in range(1, 1 << d)]
        m = _moments(p, d, False)
        out[0, a:b], out[1, a:b] = m[-1], _cumulant(m, d)
    return out[0], out[1]


def _kappa_blocks(kappa, M, K):
    at, out = 0, [None]
    for d in range(1, K + 1):
        out.append(kappa[at:at + math.comb(M, d)])
        at += math.comb(M, d)
    return out


def _plain_sample(M, K, kappa, u):
    """The chain rule with one (K = 3) or two (K = 5) elided variables, all samples at
    once. Bits are numbered 1..M; p1[a][e], p2[a][e, d] and pp[a][b] (from b to a) hold
    the marginals of the first a bits."""
    N = u.shape[1]
    kap = _kappa_blocks(kappa, M, K)
    C = math.comb
    k2 = lambda i, n: float(k2h[C(n - 1, 2) + i - 1])  # noqa: E731
    k1h, k2h = kap[1].cpu(), kap[2].cpu()
    one = torch.ones(N, dtype=F64, device=DEV)
    p = [one]
    p1 = [torch.zeros((1, N), dtype=F64, device=DEV)]          # p1[a]: rows e = 0..a (row 0 unused)
    pp = [torch.ones((M + 2, N), dtype=F64, device=DEV)]       # pp[a]: row b, 1 where b > a
    p2 = [None]                                                # p2[a]: symmetric (a + 1, a + 1, N)
    chi = torch.ones((M + 1, N), dtype=F64, device=DEV)
    bits = torch.zeros((N, M), dtype=torch.uint8, device=DEV)
    pair = {}

    def pairs(a):  # indices (i, j) of the pairs j < i <= a in colex order
        if a not in pair:
            ij = [(i, j) for i in range(1, a + 1) for j in range(1, i)]
            pair[a] = torch.tensor(ij, device=DEV).reshape(-1, 2).T
        return pair[a]

    for n in range(1, M + 1):
        prev, x = p[n - 1], chi
        c2 = kap[2][C(n - 1, 2):C(n - 1, 2) + n - 1]            # kappa(i, n), i = 1..n-1
        c3 = kap[3][C(n - 1, 3):C(n - 1, 3) + C(n - 1, 2)] if n >= 3 else None  # kappa(i, j, n)
        D = 0.5 * float(k1h[n - 1]) * prev
        if n > 1:
            g2 = c2.unsqueeze(1) * x[1:n]                       # gamma(i, n)
            D = D + 0.25 * (g2 * p1[n - 1][1:n]).sum(0)
        up = [None] + [pp[n - 1][a + 1] for a in range(1, n)]   # p+(n-1 .. a+1)
        if K == 3 and n >= 3:
            for i in range(2, n):
                g = c3[C(i - 1, 2):C(i - 1, 2) + i - 1]
                D = D + 0.125 * x[i] * up[i] * ((g.unsqueeze(1) * x[1:i]) * p1[i - 1][1:i]).sum(0)
        if K == 5 and n >= 3:
            i, j = pairs(n - 1)
            D = D + 0.125 * (c3.unsqueeze(0) @ (x[i] * x[j] * p2[n - 1][i, j]))[0]
            for i in range(3, n):
                q, r = pairs(i - 1)
                at = C(n - 1, 4) + C(i - 1, 3)
                v = kap[4][at:at + C(i - 1, 2)].unsqueeze(0) @ (x[q] * x[r] * p2[i - 1][q, r])
                D = D + x[i] * up[i] * v[0] / 16.0
            for j in range(3, n - 1):
                q, r = pairs(j - 1)
                w = C(j - 1, 2)
                i = torch.arange(j + 1, n, device=DEV)
                at = torch.tensor([C(n - 1, 5) + C(a - 1, 4) + C(j - 1, 3) for a in range(j + 1, n)], device=DEV)
                v = kap[5][at.unsqueeze(1) + torch.arange(w, device=DEV)] @ (x[q] * x[r] * p2[j - 1][q, r])
                mid = torch.stack([pp[a - 1][j + 1] for a in range(j + 1, n)])
                D = D + x[j] * (x[i] * pp[n - 1][i + 1] * mid * v).sum(0) / 32.0
        q = torch.where(prev > 0, (0.5 * prev - D) / prev, 0.5 * one)
        xn = u[n - 1] < q
        bits[:, n - 1] = xn.to(torch.uint8)
        s = torch.where(xn, -one, one)
        chi[n] = s
        p.append(0.5 * prev + s * D)
        h = 0.5 * (1.0 + float(k1h[n - 1]) * s)
        # p+(n .. l): the last elided bit j of each term carries the rest p+(j-1 .. l)
        new = torch.ones((M + 2, N), dtype=F64, device=DEV)
        new[1:n + 1] = h * pp[n - 1][1:n + 1]
        for j in range(1, n):
            c = 0.25 * g2[j - 1] * up[j]
            if K == 5 and j + 1 < n:
                i = torch.arange(j + 1, n, device=DEV)
                k = c3[torch.tensor([C(a - 1, 2) + j - 1 for a in range(j + 1, n)], device=DEV)]
                mid = torch.stack([pp[a - 1][j + 1] for a in range(j + 1, n)])
                c = c + 0.125 * x[j] * (k.unsqueeze(1) * x[i] * pp[n - 1][i + 1] * mid).sum(0)
            new[1:j + 1] += s * c * pp[j - 1][1:j + 1]
        # one elided variable
        one_el = torch.zeros((n + 1, N), dtype=F64, device=DEV)
        one_el[n] = prev
        if n > 1:
            one_el[1:n] = h * p1[n - 1][1:n]
            if K == 3:
                for a in range(2, n):
                    one_el[a] += 0.25 * s * up[a] * (g2[:a - 1] * p1[a - 1][1:a]).sum(0)
                    one_el[1:a] += 0.25 * s * g2[a - 1] * up[a] * p1[a - 1][1:a]
            else:
                one_el[1:n] += 0.25 * s * (g2.unsqueeze(1) * p2[n - 1][1:n, 1:n]).sum(0)
        if K == 5:
            two = torch.zeros((n + 1, n + 1, N), dtype=F64, device=DEV)
            if n > 1:
                two[1:n, 1:n] = h * p2[n - 1][1:n, 1:n]
            for a in range(2, n):
                t = p2[a - 1][1:a, 1:a]
                two[1:a, 1:a] += (0.25 * s * g2[a - 1] * up[a]) * t
                row = 0.25 * s * up[a] * (g2[:a - 1].unsqueeze(1) * t).sum(0)
                two[a, 1:a] += row
                two[1:a, a] += row
                k = c3[C(a - 1, 2):C(a - 1, 2) + a - 1].unsqueeze(1) * x[1:a]
                one_el[1:a] += 0.125 * s * x[a] * up[a] * (k.unsqueeze(1) * t).sum(0)
                if a > 2:
                    i, j = pairs(a - 1)
                    one_el[a] += 0.125 * s * up[a] * (c3[:C(a - 1, 2)].unsqueeze(0) @ (x[i] * x[j] * t[i - 1, j - 1]))[0]
            if n > 1:
                two[n, 1:n] = two[1:n, n] = p1[n - 1][1:n]
            two[torch.arange(n + 1), torch.arange(n + 1)] = 0.0
            p2.append(two)
        pp.append(new)
        p1.append(one_el)
    return bits, p[M]


def _power_sums(bits, K):
    """Samples in which all of S clicked, for all S of orders 1..K (exact: counts below 2^24)."""
    n, M = bits.shape
    x = bits.T.to(torch.float32).contiguous()
    binom = _binomials(M, K).cpu().tolist()
    out = [None, x.sum(1, dtype=F64)]
    for d in range(2, K + 1):
        dl = 1 if d <= 3 else 2
        s = torch.empty(math.comb(M, d), dtype=F64, device=DEV)
        for c in range(dl, M - (d - dl) + 1):
            low = x[:c] if dl == 1 else torch.cat([x[j:j + 1] * x[:j] for j in range(1, c)])
            rest = list(itertools.combinations(range(c + 1, M), d - dl - 1))
            cols = torch.tensor(rest, dtype=torch.int64).reshape(len(rest), -1)
            base = torch.tensor([binom[dl + 1][c] + sum(binom[dl + 2 + q][m] for q, m in enumerate(R)) for R in rest])
            for a in range(0, len(rest), 1024):
                h = x[c].expand(min(1024, len(rest) - a), n)
                for q in range(cols.shape[1]):
                    h = h * x[cols[a:a + 1024, q].to(DEV)]
                v = (low @ h.T).to(F64)
                s[base[a:a + 1024].to(DEV).unsqueeze(0) + torch.arange(v.shape[0], device=DEV).unsqueeze(1)] = v
        out.append(s)
    return out


def _kstat_terms(d, n):
    """{tuple of block masks: coefficient} of the unbiased cumulant in power sums: each
    product of moments averaged over distinct samples."""
    terms = {}
    for pi in _partitions(d):
        k, fall = len(pi), 1.0
        for i in range(k):
            fall *= n - i
        w = (-1.0) ** (k - 1) * math.factorial(k - 1) / fall
        for sg in _partitions(k):
            v = w
            for g in sg:
                c = bin(g).count("1")
                v *= (-1.0) ** (c - 1) * math.factorial(c - 1)
            key = tuple(sorted(sum(pi[i] for i in range(k) if g >> i & 1) for g in sg))
            terms[key] = terms.get(key, 0.0) + v
    return terms


def _plain_estimate(bits, K):
    n, M = bits.shape
    s = _power_sums(bits, K)
    binom = _binomials(M, K)
    out = []
    for d in range(1, K + 1):
        terms = _kstat_terms(d, float(n))
        total = math.comb(M, d)
        val = torch.empty(total, dtype=F64, device=DEV)
        for a in range(0, total, CHUNK):
            b = min(total, a + CHUNK)
            S = _unrank(torch.arange(a, b, device=DEV), d, binom)
            m = [None]
            for B in range(1, 1 << d):
                mem = [S[i] for i in range(d) if B >> i & 1]
                m.append(s[len(mem)][sum(binom[j + 1][v] for j, v in enumerate(mem))] / n)
            acc = 0.0
            for key, c in terms.items():
                v = c * float(n) ** len(key)
                for B in key:
                    v = v * m[B]
                acc = acc + v
            val[a:b] = acc
        out.append(val)
    return torch.cat(out)


def exact(case, seed):
    st = prepare(case, seed)
    kind = case["kind"]
    if kind in ("cumulants", "displaced"):
        return _plain(st["sigma"], case["K"], st.get("mu"), case["parity"])
    if kind == "batched":
        at = 0
        for M, sigma, corr, cum in st["inst"]:
            n = corr.numel()
            st["corr"][at:at + n], st["cum"][at:at + n] = _plain(sigma, case["K"])
            at += _padded(n)
        return st["corr"], st["cum"]
    if kind == "shard":
        return _plain_range(st["sigma"], case["order"], _shard_start(case), case["count"])
    if kind == "fit":
        _, cum = _plain(_covariance(st["W"], st["r"], st["eta"]), case["K"])
        loss = ((cum - st["target"]) ** 2).sum()
        gr, ge = torch.autograd.grad(loss, (st["r"], st["eta"]))
        return loss.detach(), gr, ge
    if kind == "sample":
        return _plain_sample(case["M"], case["K"], st["kappa"], st["u"])
    cum = _plain_estimate(st["bits"], case["K"])
    if not case["pearson"]:
        return cum
    rs, at = [], 0
    for d in range(1, case["K"] + 1):
        n = math.comb(case["M"], d)
        x, y = cum[at:at + n], st["truth"][at:at + n]
        x, y = x - x.mean(), y - y.mean()
        rs.append(((x * y).sum() / torch.sqrt((x * x).sum() * (y * y).sum())).reshape(1))
        at += n
    return [cum] + rs
