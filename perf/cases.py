"""The calls whose speed matters: every query of the library at the sizes it is used at.

A case is one call of a public entry point (``paper_2308_03291_amd.binding``) on inputs that are resident on the
GPU: ``op`` names the query, ``B``, ``N``, ``T`` (and ``K`` for the semi-Markov CRF) its shape, ``dtype`` the storage
type of the potentials, ``min_len`` the shortest sequence of the batch (``N``: all of full length) and ``kind`` and
``scale`` the distribution of the potentials.  Sizes are those of ``paper_2308_03291_amd.workloads`` (the paper's
benchmark shapes among them) where it has one for the query.
"""
from __future__ import annotations

import math

import torch

from paper_2308_03291_amd import binding as crf

DEVICE = "cuda"


def _case(op, B, N, T, *, name=None, K=1, dtype="f32", min_len=None, kind="iid", scale=1.0):
    c = {"op": op, "B": B, "N": N, "T": T, "K": K, "dtype": dtype, "min_len": N if min_len is None else min_len,
         "kind": kind, "scale": scale}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # The smallest call: a handful of short sentences, where launches and host work are all there is.
        _case("marginals", 4, 8, 5, name="marginals_tiny"),
        # Decoding a small ragged batch, the serving case.
        _case("argmax", 32, 64, 32, name="argmax_small", min_len=32),
        # Gradient of a tagger's loss: ragged sentences, 48 tags, emission + transition scores given densely.
        _case("marginals", 128, 128, 48, name="marginals_tagger", min_len=16, kind="tagging", scale=2.0),
        # Gradient over a large tag set, the headline workload: 2.1 GB of potentials streamed from HBM.
        _case("marginals", 64, 512, 128, name="marginals_large"),
        # Very long chains in a tiny batch, peaked potentials stored in half the bytes.
        _case("marginals", 4, 16384, 16, name="marginals_long", dtype="bf16", scale=10.0),
        # Gradient over an odd and very large tag set.
        _case("marginals", 32, 256, 201, name="marginals_wide_odd", dtype="bf16"),
        # The loss of a training or evaluation step, at the size the paper times its linear-chain CRF on.
        _case("log_prob", 128, 256, 32, name="log_prob_paper"),
        # Decoding a tagger from emissions and one transition matrix, an odd tag count (BIO labels), ragged sentences.
        _case("argmax_structured", 256, 100, 45, name="decode_structured_odd", min_len=10, kind="tagging", scale=2.0),
        # Entropy regularisation of the tagger.
        _case("entropy", 128, 128, 48, name="entropy_tagger", min_len=16, kind="tagging", scale=2.0),
        # Distillation: divergence between two chains over the same sentences.
        _case("kl", 64, 256, 64, name="kl_distill", min_len=64),
        # Sampling one path a sequence for a sampled loss.
        _case("sample", 128, 256, 32, name="sample_paper"),
        # Segmentation: the size the paper times its semi-Markov CRF on.
        _case("semi_markov", 1, 64, 32, name="semi_markov_paper", K=8),
    ]


OPS = ("marginals", "marginals", "argmax", "log_prob", "argmax_structured", "entropy", "kl", "sample", "semi_markov")
MAX_STEPS = 512 * 128   # N * T of the headline workload
MAX_POTENTIALS = 1 << 27


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(OPS)
    ragged = rng.random() < 0.5
    dtype = "f32" if op == "argmax_structured" or rng.random() < 0.6 else "bf16"
    if op == "semi_markov":
        K, T = rng.randint(2, 8), _log_int(rng, 8, 64)
        B, N = _log_int(rng, 1, 64), _log_int(rng, 8, 256)
        while B * N * K * T * T > MAX_POTENTIALS:
            B = max(1, B // 2)
        return _case(op, B, N, T, K=K, dtype=dtype, min_len=max(1, N // 2) if ragged else N)
    if rng.random() < 1 / 6:  # long chains in a small batch
        T, B, N = _log_int(rng, 5, 32), rng.randint(1, 8), _log_int(rng, 1024, 16384)
    else:
        T = _log_int(rng, 5, 128 if op == "argmax_structured" else 256)
        B, N = _log_int(rng, 1, 256), _log_int(rng, 8, 512)
        N = min(N, MAX_STEPS // T)
    while B * N * T * T > MAX_POTENTIALS:
        B = max(1, B // 2)
    kind = "tagging" if op == "argmax_structured" or rng.random() < 0.3 else "iid"
    scale = 2.0 if kind == "tagging" else rng.choice((1.0, 1.0, 3.0))
    return _case(op, B, N, T, dtype=dtype, min_len=max(1, N // rng.choice((2, 8))) if ragged else N, kind=kind,
                 scale=scale)


def _potentials(c, g):
    B, N, T = c["B"], c["N"], c["T"]
    shape = (B, N, c["K"], T, T) if c["op"] == "semi_markov" else (B, N, T, T)
    if c["kind"] == "tagging":
        emit, trans = _emit_trans(c, g)
        x = emit[:, :, None, :] + trans
    else:
        x = torch.randn(shape, generator=g, device=DEVICE)
        if c["scale"] != 1.0:
            x.mul_(c["scale"])
    return x.to(torch.bfloat16) if c["dtype"] == "bf16" else x


def _emit_trans(c, g):
    emit = torch.randn(c["B"], c["N"], c["T"], generator=g, device=DEVICE) * c["scale"]
    return emit, torch.randn(c["T"], c["T"], generator=g, device=DEVICE)


def prepare(case, seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    op, B, N, T = case["op"], case["B"], case["N"], case["T"]
    s = {"op": op, "lengths": None}
    if case["min_len"] < N:
        s["lengths"] = torch.randint(case["min_len"], N + 1, (B,), generator=g, device=DEVICE).to(torch.int32)
    if op == "argmax_structured":
        s["emit"], s["trans"] = _emit_trans(case, g)
        return s
    s["phi"] = _potentials(case, g)
    if op == "log_prob":
        s["tags"] = torch.randint(0, T, (B, N), generator=g, device=DEVICE).to(torch.int32)
    elif op == "kl":  # a student half way to its teacher
        q = s["phi"].float()
        s["phi_q"] = (q + 0.5 * torch.randn(q.shape, generator=g, device=DEVICE)).to(s["phi"].dtype)
    elif op == "sample":
        s["seed"] = seed * 2654435761 + 12345
    return s


def run(state):
    op, lengths = state["op"], state["lengths"]
    if op == "marginals":
        return crf.lccrf_marginals(state["phi"], lengths)
    if op == "argmax":
        return crf.lccrf_argmax(state["phi"], lengths)
    if op == "argmax_structured":
        return crf.lccrf_argmax_structured(state["emit"], state["trans"], lengths)
    if op == "log_prob":
        return crf.lccrf_log_prob(state["phi"], state["tags"], lengths)
    if op == "entropy":
        return crf.lccrf_entropy(state["phi"], lengths)
    if op == "kl":
        return crf.lccrf_kl_divergence(state["phi"], state["phi_q"], lengths)
    if op == "sample":
        return crf.lccrf_sample_seeded(state["phi"], state["seed"], lengths)
    return crf.lccrf_semi_markov_log_partition(state["phi"], lengths)


def work(case):
    """Potentials of positions inside the chains read once, results written once; a multiply-add a potential for a
    sum or maximum over the predecessors, as many again for each further one that the query takes."""
    op, B, N, T, K = case["op"], case["B"], case["N"], case["T"], case["K"]
    inside = 0.5 * (case["min_len"] + N) / N
    e = 4 if case["dtype"] == "f32" else 2
    pots = inside * B * N * K * T * T
    if op == "marginals":
        return {"bytes": e * pots + 4.0 * B * N * T * T + 4 * B, "flops": 6.0 * pots}
    if op == "argmax":
        return {"bytes": e * pots + 4.0 * B * N + 4 * B, "flops": 2.0 * pots}
    if op == "argmax_structured":
        return {"bytes": 4.0 * inside * B * N * T + 4 * T * T + 4.0 * B * N + 4 * B, "flops": 2.0 * pots}
    if op == "log_prob":
        return {"bytes": e * pots + 4.0 * B * N + 4 * B, "flops": 2.0 * pots}
    if op == "entropy":
        return {"bytes": e * pots + 4 * B, "flops": 4.0 * pots}
    if op == "kl":
        return {"bytes": 2 * e * pots + 4 * B, "flops": 6.0 * pots}
    if op == "sample":
        return {"bytes": e * pots + 4.0 * B * N, "flops": 2.0 * pots}
    return {"bytes": e * pots + 4 * B, "flops": 2.0 * pots}


def tolerance(case):
    """Measured against 64 bits, times about four: marginals up to 2.4e-6, entropies 2.3e-7, other sums and scores
    1e-7.  Paths: potentials of eight significant bits tie exactly, and any best path is a right answer; otherwise the
    path is the same.  A sampled tag is decided by comparing 32-bit sums (none of 32768 differed from 64 bits)."""
    op = case["op"]
    if op == "marginals":
        return {"rel": 1e-5}
    if op in ("argmax", "argmax_structured"):
        return {"rel": 4e-7, "differ": 0.01 if case["dtype"] == "bf16" else 0.0}
    if op == "sample":
        return {"rel": 0.0, "differ": 1e-3}
    return {"rel": 1e-6}


# ---- the same values in 64 bits, in plain torch ---------------------------------------------------------------

def _lens(state, B, N):
    lens = state["lengths"]
    return torch.full((B,), N, device=DEVICE) if lens is None else lens.long()


def _forward(phi, lens):
    """alpha [N, B, T] (held at its last value past the length)."""
    N, out = phi.shape[1], []
    a = phi[:, 0, 0].double()
    out.append(a)
    for i in range(1, N):
        step = torch.logsumexp(a[:, :, None] + phi[:, i].double(), 1)
        a = torch.where((lens > i)[:, None], step, a)
        out.append(a)
    return torch.stack(out)


def _backward(phi, lens):
    """beta [N, B, T]."""
    B, N, T, _ = phi.shape
    b = torch.zeros(B, T, dtype=torch.float64, device=phi.device)
    out = [b]
    for i in range(N - 1, 0, -1):
        step = torch.logsumexp(phi[:, i].double() + b[:, None, :], 2)
        b = torch.where((lens > i)[:, None], step, b)
        out.append(b)
    return torch.stack(out[::-1])


def _best_score(phi, lens):
    d = phi(0)[:, 0].double()
    for i in range(1, phi.N):
        step = (d[:, :, None] + phi(i).double()).amax(1)
        d = torch.where((lens > i)[:, None], step, d)
    return d.amax(1)


class _Matrices:
    def __init__(self, state, N):
        self.state, self.N = state, N

    def __call__(self, i):
        if "phi" in self.state:
            return self.state["phi"][:, i]
        return self.state["emit"][:, i][:, None, :] + self.state["trans"]


def _edges(phi, lens):
    """logZ [B] and, one position at a time, its edge marginals [B, T, T] in 64 bits (row 0 alone at position 0)."""
    B, N, T, _ = phi.shape
    a, b = _forward(phi, lens), _backward(phi, lens)
    logZ = torch.logsumexp(a[-1], 1)

    def at(i):
        if i == 0:
            mu = torch.zeros(B, T, T, dtype=torch.float64, device=phi.device)
            mu[:, 0] = torch.exp(a[0] + b[0] - logZ[:, None])
            return mu
        mu = torch.exp(a[i - 1][:, :, None] + phi[:, i].double() + b[i][:, None, :] - logZ[:, None, None])
        return mu * (lens > i)[:, None, None]
    return logZ, at


def _semi_markov(phi, lens):
    B, N, K, T, _ = phi.shape
    alphas, last = [], torch.zeros(B, T, dtype=torch.float64, device=phi.device)
    for i in range(N):
        terms = []
        for k in range(min(K, i + 1)):
            x = phi[:, i, k].double()
            terms.append(x[:, 0] if k == i else torch.logsumexp(alphas[i - k - 1][:, :, None] + x, 1))
        alphas.append(torch.logsumexp(torch.stack(terms), 0))
        last = torch.where((lens > i)[:, None], alphas[i], last)
    return torch.logsumexp(last, 1)


def exact(case, seed):
    s = prepare(case, seed)
    op, B, N = case["op"], case["B"], case["N"]
    lens = _lens(s, B, N)
    if op == "sample":
        return None
    if op in ("argmax", "argmax_structured"):
        return _best_score(_Matrices(s, N), lens), None
    phi = s["phi"]
    if op == "semi_markov":
        return _semi_markov(phi, lens)
    if op == "log_prob":
        logZ = torch.logsumexp(_forward(phi, lens)[-1], 1)
        tags = s["tags"].long()
        prev = torch.cat([torch.zeros_like(tags[:, :1]), tags[:, :-1]], 1)
        b, i = torch.arange(B, device=DEVICE)[:, None], torch.arange(N, device=DEVICE)[None, :]
        score = (phi[b, i, prev, tags].double() * (i < lens[:, None])).sum(1)
        return score - logZ
    logZ, edge = _edges(phi, lens)
    if op == "marginals":
        mu = torch.empty(phi.shape, dtype=torch.float64, device=DEVICE)
        for i in range(N):
            mu[:, i] = edge(i)
        return logZ, mu
    if op == "entropy":
        return logZ - sum((edge(i) * phi[:, i].double()).sum((1, 2)) for i in range(N))
    q = s["phi_q"]
    logZ_q = torch.logsumexp(_forward(q, lens)[-1], 1)
    diff = sum((edge(i) * (phi[:, i].double() - q[:, i].double())).sum((1, 2)) for i in range(N))
    return diff - logZ + logZ_q
