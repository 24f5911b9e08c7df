"""Chains of 65 .. 256 tags walked in pieces by several workgroups (the schedule AUTO takes for long chains in small batches), against the
oracle: potentials that forget quickly (every piece matches), one sequence among them that forgets nothing (its pieces do not, and
the rest of its chains is walked again), batches whose potentials are seen to forget slowly (one piece), steps in the log
domain inside a piece, sequences of every short length.  Tolerances as everywhere for these queries (fp32 sums: 1e-5)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2308_03291_amd import workloads
from test_gpu_parity import check_case, crf  # noqa: F401  (crf: the module-scoped binding fixture)
from test_gpu_sample import _check, _check_every_draw

pytestmark = pytest.mark.gpu


UNMATCHED = 2 ** 31 - 1


def _pieces(crf, op, phi, lens=None):
    """What became of the chains of a call: {(b, direction): (plan, [what became of piece 1, 2, ...])}, and how many pieces there may be.  A plan is
    None where the batch was not cut, else whether the chain took no steps in scaled probabilities."""
    B, N, T = phi.shape[:3]
    dt = crf.LCCRF_BF16 if phi.dtype == torch.bfloat16 else crf.LCCRF_F32
    at = ctypes.c_size_t()
    most = crf.load_library().lccrf_first_pass_pieces(op, dt, B, N, T, ctypes.byref(at))
    ws = torch.zeros(crf.workspace_bytes(op, B, N, T, dt), dtype=torch.uint8, device="cuda")
    {crf.OP_LOGZ: crf.lccrf_log_partition, crf.OP_MARGINALS: crf.lccrf_marginals}[op](phi.cuda(), None if lens is None else lens.cuda(), workspace=ws)
    if most == 1:
        return 1, {}
    left = ws[at.value:at.value + 8 * B * most].view(torch.int32).view(2 * B, most).cpu().tolist()
    found = {}
    for b in range(B):
        L = N if lens is None else int(lens[b])
        for direction in range(2 if L > 0 else 0):
            n = L - 1 if op == crf.OP_MARGINALS else L // 2 if direction == 0 else L - 1 - L // 2
            least, rows = left[2 * b + direction][0] >> 1, left[2 * b + direction]
            cut = min(most, max(1, n // least))
            length = -(-n // cut) if n else 1
            found[b, direction] = (None if least >= 1 << 20 else bool(rows[0] & 1), rows[1:-(-n // length)] if n else [])
    return most, found


def _slow(phi, b):
    """Sequence b stays where it is: what a chain started with is still there at its end."""
    phi[b] += (25.0 * torch.eye(phi.shape[-1])).to(phi.dtype)


@pytest.mark.parametrize("T,dtype", [(65, "f32"), (66, "bf16"), (96, "f32"), (101, "bf16"), (128, "f32"), (129, "f32"), (156, "f32"), (201, "bf16"), (256, "f32")])
def test_marginals_and_log_partition(crf, oracle_mod, T, dtype):
    N = 150
    phi, _ = workloads.random_case(9300 + T, 5, N, T, scale=1.0, dtype=dtype)
    _slow(phi, 4)
    phi[1, 31, :, 5] = float("-inf")   # steps that are not accepted, in either chain's pieces
    phi[1, 97, 7, :] = float("-inf")
    phi[2, 50] += 250.0
    phi[2, 103] -= 250.0
    lens = torch.tensor([N, N, N - 1, 83, N], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, what=f"pieces T={T} {dtype}", queries=("logz", "mu"))
    for op in (crf.OP_LOGZ, crf.OP_MARGINALS):
        _, found = _pieces(crf, op, phi, lens)
        for (b, _), (in_log_domain, matched) in found.items():
            assert in_log_domain is False and len(matched) >= (1 if b == 3 else 2), (op, b)
            if b in (0, 3):
                assert UNMATCHED not in matched, (op, b, matched)
            if b == 4:
                assert all(m == UNMATCHED for m in matched), (op, matched)


@pytest.mark.parametrize("T", [72, 144])
def test_every_sequence_forgets_nothing_or_slowly(crf, oracle_mod, T):
    N = 130
    for scale in (3.0, 12.0):
        phi, _ = workloads.random_case(9400 + T, 3, N, T, scale=scale)
        check_case(crf, oracle_mod, phi, None, what=f"slow T={T} scale={scale}", queries=("logz", "mu"))
        most, found = _pieces(crf, crf.OP_MARGINALS, phi)
        assert most > 1 and all(in_log_domain is None for in_log_domain, _ in found.values())
    phi, _ = workloads.random_case(9500 + T, 6, N, T)
    for b in (2, 5):  # (not among the sequences whose matrices are looked at: 0, 1, 3 and 4)
        _slow(phi, b)
    phi[5, :, :, T - 1] = float("-inf")
    check_case(crf, oracle_mod, phi, None, what=f"some slow T={T}", queries=("logz", "mu"))
    _, found = _pieces(crf, crf.OP_MARGINALS, phi)
    for (b, direction), (in_log_domain, matched) in found.items():
        assert in_log_domain is (b == 5 and direction == 0) and len(matched) >= 2, b  # (a tag that cannot be come to can be left)
        assert all((m == UNMATCHED) == (b in (2, 5)) for m in matched), (b, matched)


@pytest.mark.parametrize("T,N", [(68, 120), (200, 120), (68, 260)])
def test_every_short_length(crf, oracle_mod, T, N):
    lengths = [N, 0, 1, 2, 3] + [N // 120 * n for n in (17, 18, 19, 35, 36, 37, 38, 39, 55, 73, 74)]
    phi, _ = workloads.random_case(9600 + T, len(lengths), N, T)
    check_case(crf, oracle_mod, phi, torch.tensor(lengths, dtype=torch.int32), what=f"lengths T={T} N={N}", queries=("logz", "mu"))
    for op in (crf.OP_LOGZ, crf.OP_MARGINALS):
        most, found = _pieces(crf, op, phi, torch.tensor(lengths, dtype=torch.int32))
        if (op, T, N) == (crf.OP_LOGZ, 68, 120):  # (chains too short for it to pay)
            continue
        cut = {len(matched) for _, matched in found.values()}
        assert most > 1 and 0 in cut and len(cut) >= 3, (op, cut)


@pytest.mark.parametrize("T,dtype", [(65, "f32"), (100, "bf16"), (128, "f32"), (200, "f32")])
def test_log_prob(crf, oracle_mod, T, dtype):
    N = 200
    phi, _ = workloads.random_case(9700 + T, 5, N, T, dtype=dtype)
    _slow(phi, 4)
    lens = torch.tensor([N, N, 0, 90, N], dtype=torch.int32)
    tags = torch.randint(0, T, (5, N), generator=torch.Generator().manual_seed(T)).to(torch.int32)
    got = crf.lccrf_log_prob(phi.cuda(), tags.cuda(), lens.cuda()).cpu().numpy()
    want = oracle_mod.log_prob(phi, tags.numpy(), lens.numpy())
    assert np.allclose(got, want, rtol=1e-5, atol=1e-5)
    _, found = _pieces(crf, crf.OP_LOGZ, phi, lens)  # (the same first pass)
    assert UNMATCHED not in found[0, 0][1] and UNMATCHED in found[4, 0][1]


@pytest.mark.parametrize("T", [66, 128, 150])
def test_sampling(crf, oracle_mod, T):
    phi, _ = workloads.random_case(9800 + T, 5, 120, T)
    _slow(phi, 4)
    lens = torch.tensor([120, 119, 40, 2, 120], dtype=torch.int32)
    _check(crf, oracle_mod, phi, lens, 300 + T, f"sample in pieces T={T}", min_exact=0.0)
    _check_every_draw(crf, oracle_mod, phi, lens, 300 + T, f"sample in pieces T={T}")
    assert crf.load_library().lccrf_first_pass_pieces(crf.OP_SAMPLE, crf.LCCRF_F32, 5, 120, T, None) > 1


@pytest.mark.parametrize("T,dtype", [(66, "f32"), (128, "f32"), (136, "f32"), (201, "bf16")])
def test_one_position_forbids_every_edge(crf, oracle_mod, T, dtype):
    """A position whose whole matrix is -inf, at every place of every piece, and two of them in neighbouring pieces: no finite path, so
    logZ = -inf and marginals 0.  (Behind it both the chain and the row it is compared with are zero everywhere, which says nothing.)"""
    N, batch = 240, 16
    base, _ = workloads.random_case(9900 + T, 1, N, T, dtype=dtype)
    want_lz, want_mu = oracle_mod.marginals(base, None)
    want_mu = torch.from_numpy(np.ascontiguousarray(want_mu)).cuda()
    for op in (crf.OP_LOGZ, crf.OP_MARGINALS):
        _, found = _pieces(crf, op, base.repeat(batch, 1, 1, 1))
        assert all(in_log_domain is False and len(matched) >= 4 and UNMATCHED not in matched for in_log_domain, matched in found.values())
    base = base.cuda()
    dead = [(p,) for p in range(1, N)] + [(p, p + d) for d in (17, 23, 41) for p in range(1, N - d, 5)]
    for k in range(0, len(dead), batch - 1):
        places = dead[k:k + batch - 1]
        phi = base.repeat(len(places) + 1, 1, 1, 1)  # (the last one as it is)
        for b, positions in enumerate(places):
            phi[b, list(positions)] = float("-inf")
        lz, mu = crf.lccrf_marginals(phi)
        for got in (crf.lccrf_log_partition(phi), lz):
            got = got.cpu().numpy()
            assert np.all(got[:-1] == -np.inf), (T, [p for p, x in zip(places, got) if x != -np.inf])
            assert np.allclose(got[-1:], want_lz, rtol=1e-5, atol=0)
        assert not mu[:-1].any()
        assert float((mu[-1] - want_mu[0]).abs().max()) <= 1e-5


@pytest.mark.parametrize("T,dtype", [(67, "bf16"), (144, "f32")])
def test_rows_behind_a_match_are_as_exact_as_a_whole_chains(crf, T, dtype):
    """Potentials that forget slowly enough that what is left of a piece's beginning can be followed behind its match: the stored forward vectors
    (the workspace's first [B][N][T] floats, base-2 logarithms) against 64 bits, in pieces (AUTO) and as a whole (SEQUENTIAL; the same
    steps in scaled probabilities at these tag counts).  In pieces a row may be off by as much more as the vector that its piece began with: a
    stored row, rounded by 2^-23 at four bits, turned into a logarithm and back by instructions good to one unit in the last place, 2^-23."""
    B, N = 3, 1500
    g = torch.Generator(device="cuda").manual_seed(T)
    phi = torch.randn(B, N, T, T, generator=g, device="cuda") + 4.0 * torch.eye(T, device="cuda")
    phi = phi.to(torch.bfloat16) if dtype == "bf16" else phi
    half = N // 2 - 2
    a, exact = phi[:, 0, 0].double(), []
    for i in range(1, half):
        a = torch.logsumexp(a[:, :, None] + phi[:, i].double(), 1)
        exact.append(a)
    exact = torch.stack(exact, 1) / np.log(2.0)
    heavy = exact > exact.amax(2, keepdim=True) - 4.0  # (logarithms whose rounding is at most 2^-23)
    error = {}
    for algo in (crf.ALGO_AUTO, crf.ALGO_SEQUENTIAL):
        ws = torch.zeros(crf.workspace_bytes(crf.OP_LOGZ, B, N, T, crf.LCCRF_BF16 if dtype == "bf16" else crf.LCCRF_F32), dtype=torch.uint8, device="cuda")
        crf.lccrf_log_partition(phi, workspace=ws, algo=algo)
        d = ws[:4 * B * N * T].view(torch.float32).view(B, N, T)[:, 1:half].double() - exact
        span = torch.where(heavy, d, -np.inf).amax(2) - torch.where(heavy, d, np.inf).amin(2)  # (a row's common factor is its offset's)
        error[algo] = 0.5 * float(span.max())
    _, found = _pieces(crf, crf.OP_LOGZ, phi.cpu())
    assert all(len(matched) >= 2 for _, matched in found.values())
    assert error[crf.ALGO_AUTO] <= error[crf.ALGO_SEQUENTIAL] + 2.0 ** -22, error


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_marginals_of_128_tags_do_not_drift(crf, dtype):
    """The marginals of a few long chains against 64 bits.  The exponent of a marginal is a sum of four logarithms below sixteen bits, each rounded by
    2^-21, and of two vectors that are themselves off by up to 1.1e-6 bits: 3e-6 in all.  (Half chains in pieces with the paired second pass: 2e-5.)"""
    B, N, T = 3, 400, 128
    assert crf.load_library().lccrf_first_pass_pieces(crf.OP_MARGINALS, 1 if dtype == "bf16" else 0, B, N, T, None) > 1
    phi = 2.0 * torch.randn(B, N, T, T, generator=torch.Generator(device="cuda").manual_seed(128), device="cuda")
    phi = phi.to(torch.bfloat16) if dtype == "bf16" else phi
    a, alpha = phi[:, 0, 0].double(), []
    for i in range(N):
        a = a if i == 0 else torch.logsumexp(a[:, :, None] + phi[:, i].double(), 1)
        alpha.append(a)
    logZ = torch.logsumexp(a, 1)[:, None, None]
    _, mu = crf.lccrf_marginals(phi)
    b, wrong, all_of_it = torch.zeros_like(a), 0.0, 0.0
    for i in range(N - 1, 0, -1):
        want = torch.exp(alpha[i - 1][:, :, None] + phi[:, i].double() + b[:, None, :] - logZ)
        wrong += float(((mu[:, i].double() - want) ** 2).sum())
        all_of_it += float((want ** 2).sum())
        b = torch.logsumexp(phi[:, i].double() + b[:, None, :], 2)
    assert (wrong / all_of_it) ** 0.5 <= 3e-6


def test_paired_second_pass_over_long_chains(crf, oracle_mod):
    """128 tags, N = 512, more sequences than are walked in pieces and few enough for two workgroups a chain, which exchange half vectors 256
    times in each direction: every marginal of three sequences against the oracle, and their copies in the batch the same."""
    phi, _ = workloads.random_case(4501, 3, 512, 128, scale=1.0, dtype="bf16")
    lens = torch.tensor([512, 511, 300], dtype=torch.int32)
    want_lz, want_mu = oracle_mod.marginals(phi, lens.numpy())
    assert crf.load_library().lccrf_first_pass_pieces(crf.OP_MARGINALS, crf.LCCRF_BF16, 54, 512, 128, None) == 1
    lz, mu = crf.lccrf_marginals(phi.cuda().repeat(18, 1, 1, 1), lens.cuda().repeat(18))
    assert np.allclose(lz[:3].cpu().numpy(), want_lz, rtol=1e-5, atol=0)
    assert np.abs(mu[:3].cpu().numpy() - want_mu).max() <= 1e-5
    for k in range(3, 54, 3):
        assert torch.equal(mu[k:k + 3], mu[:3])


@pytest.mark.parametrize("T,B,N", [(116, 8, 660), (128, 8, 600), (112, 6, 1000)])
def test_long_chains_left_to_a_fourth_launch(crf, oracle_mod, T, B, N):
    """Single precision where steps in the log domain are quicker for chains as a whole: a batch that is not cut is walked by a kernel of its own behind
    the launches of the pieces, one that is cut is not walked again; log-partition and samples, ragged, with a chain that forgets nothing among quick ones."""
    phi, _ = workloads.random_case(10100 + T, 2, N, T)
    lens = torch.tensor([N, N - 77], dtype=torch.int32)
    uniforms = torch.rand(2, N, generator=torch.Generator().manual_seed(T))
    for slow in (False, True):
        if slow:
            phi += 25.0 * torch.eye(T)
        want = oracle_mod.log_partition(phi, lens.numpy())
        many, many_lens = phi.cuda().repeat(B // 2, 1, 1, 1), lens.cuda().repeat(B // 2)
        if not slow:
            many[B - 1] += 25.0 * torch.eye(T, device="cuda")  # (not among the sequences whose matrices are looked at, the last of which is 3 B / 4)
        got = crf.lccrf_log_partition(many, many_lens).cpu().numpy()
        ok = slice(0, B if slow else B - 1)
        assert np.allclose(got[ok], np.tile(want, B // 2)[ok], rtol=1e-5, atol=0), slow
        _, found = _pieces(crf, crf.OP_LOGZ, many, many_lens)
        assert all((in_log_domain is None) == slow for in_log_domain, _ in found.values())
        alone = crf.lccrf_sample(phi.cuda(), uniforms.cuda(), lens.cuda())  # (another batch: other pieces or none, the same draws but for rounding)
        drawn = crf.lccrf_sample(many, uniforms.cuda().repeat(B // 2, 1), many_lens)
        for k in range(0, (B if slow else B - 2), 2):
            assert float((drawn[k:k + 2] != alone).float().mean()) <= 0.02
