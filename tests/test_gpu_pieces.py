"""Chains of 65 .. 256 tags walked in pieces by several workgroups (the schedule AUTO takes for long chains in small batches), against the
oracle: potentials that forget quickly (every piece matches), one sequence among them that forgets nothing (its pieces do not, and
the rest of its chains is walked again), batches whose potentials are seen to forget slowly (one piece), steps in the log
domain inside a piece, sequences of every short length.  Tolerances as everywhere for these queries (fp32 sums: 1e-5)."""
import numpy as np
import pytest
import torch

from paper_2308_03291_amd import workloads
from test_gpu_parity import check_case, crf  # noqa: F401  (crf: the module-scoped binding fixture)
from test_gpu_sample import _check, _check_every_draw

pytestmark = pytest.mark.gpu


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


@pytest.mark.parametrize("T", [72, 144])
def test_every_sequence_forgets_nothing_or_slowly(crf, oracle_mod, T):
    N = 130
    for scale in (3.0, 12.0):
        phi, _ = workloads.random_case(9400 + T, 3, N, T, scale=scale)
        check_case(crf, oracle_mod, phi, None, what=f"slow T={T} scale={scale}", queries=("logz", "mu"))
    phi, _ = workloads.random_case(9500 + T, 6, N, T)
    for b in (3, 5):  # (not among the sequences whose matrices are looked at)
        _slow(phi, b)
    phi[5, :, :, T - 1] = float("-inf")
    check_case(crf, oracle_mod, phi, None, what=f"some slow T={T}", queries=("logz", "mu"))


@pytest.mark.parametrize("T", [68, 200])
def test_every_short_length(crf, oracle_mod, T):
    N = 120
    lengths = [N, 0, 1, 2, 3, 17, 18, 19, 35, 36, 37, 38, 39, 55, 73, 74]
    phi, _ = workloads.random_case(9600 + T, len(lengths), N, T)
    check_case(crf, oracle_mod, phi, torch.tensor(lengths, dtype=torch.int32), what=f"lengths T={T}", queries=("logz", "mu"))


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


@pytest.mark.parametrize("T", [66, 128, 150])
def test_sampling(crf, oracle_mod, T):
    phi, _ = workloads.random_case(9800 + T, 5, 120, T)
    _slow(phi, 4)
    lens = torch.tensor([120, 119, 40, 2, 120], dtype=torch.int32)
    _check(crf, oracle_mod, phi, lens, 300 + T, f"sample in pieces T={T}", min_exact=0.0)
    _check_every_draw(crf, oracle_mod, phi, lens, 300 + T, f"sample in pieces T={T}")


@pytest.mark.parametrize("T,dtype", [(66, "f32"), (128, "f32"), (136, "f32"), (201, "bf16")])
def test_one_position_forbids_every_edge(crf, oracle_mod, T, dtype):
    """A position whose whole matrix is -inf, at every place of every piece, and two of them in neighbouring pieces: no finite path, so
    logZ = -inf and marginals 0.  (Behind it both the chain and the row it is compared with are zero everywhere, which says nothing.)"""
    N, batch = 240, 16
    base, _ = workloads.random_case(9900 + T, 1, N, T, dtype=dtype)
    want_lz, want_mu = oracle_mod.marginals(base, None)
    want_mu = torch.from_numpy(np.ascontiguousarray(want_mu)).cuda()
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
    assert error[crf.ALGO_AUTO] <= error[crf.ALGO_SEQUENTIAL] + 2.0 ** -22, error


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_marginals_of_128_tags_do_not_drift(crf, dtype):
    """The marginals of a few long chains against 64 bits.  The exponent of a marginal is a sum of four logarithms below sixteen bits, each rounded by
    2^-21, and of two vectors that are themselves off by up to 1.1e-6 bits: 3e-6 in all.  (Half chains in pieces with the paired second pass: 2e-5.)"""
    B, N, T = 3, 400, 128
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
    assert crf.load_library().lccrf_marginals_by_edges(crf.LCCRF_BF16, 54, 127) == 0
    lz, mu = crf.lccrf_marginals(phi.cuda().repeat(18, 1, 1, 1), lens.cuda().repeat(18))
    assert np.allclose(lz[:3].cpu().numpy(), want_lz, rtol=1e-5, atol=0)
    assert np.abs(mu[:3].cpu().numpy() - want_mu).max() <= 1e-5
    for k in range(3, 54, 3):
        assert torch.equal(mu[k:k + 3], mu[:3])
