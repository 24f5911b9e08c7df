"""GPU parity of the entropy, the cross-entropy and the KL divergence at 33 .. 64 tags, where their chains run in scaled
probabilities until a step leaves the accepted range and in the log domain from there on, against the CPU oracle
(from its fp64 marginals).  Tolerances of the differences as in test_gpu_two_chains.py, 1e-5 of the sizes they are differences of;
the entropy, no such difference, within 1e-5 of itself (of 1 where it is smaller)."""
import numpy as np
import pytest
import torch

from paper_2308_03291_amd import workloads
from test_gpu_parity import crf  # noqa: F401  (fixture)
from test_gpu_two_chains import _check, _pair

pytestmark = pytest.mark.gpu


def _check_all(crf, oracle_mod, p, q, lens, what):
    _check(crf, oracle_mod, p, q, lens, what)
    got = crf.lccrf_entropy(p.cuda(), lens.cuda()).cpu().numpy().astype(np.float64)
    want = oracle_mod.entropy(p, lens.numpy())
    bad = ~(np.isnan(got) & np.isnan(want)) & ~(np.abs(got - want) <= 1e-5 * np.maximum(1.0, np.abs(want)))
    assert not bad.any(), f"{what}: entropy mismatch at {np.nonzero(bad)[0][:6]}: {got[bad][:4]} vs {want[bad][:4]}"


# both numbers of rows a thread holds, the last piece of a row moved back by 0 .. 3 columns, an empty and a full last row group
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [33, 34, 35, 36, 45, 47, 48, 49, 51, 61, 63, 64])
def test_scaled_expectation_chains(crf, oracle_mod, T, dtype):
    N = 23
    p, q, lens = _pair(9100 + T, 9, N, T, dtype=dtype, ragged=True, min_len=0)
    lens[:6] = torch.tensor([N, 1, 2, 3, 4, N], dtype=lens.dtype)
    # the last sequence ends with the tensor: nothing behind it may be read
    _check_all(crf, oracle_mod, p, q, lens, f"T={T} {dtype}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [33, 48, 50, 64])
def test_steps_that_leave_the_scaled_range(crf, oracle_mod, T, dtype):
    """A jump by 2^300 at a position, a tag forbidden from a position on, the first tag forbidden at the start and everywhere, tags
    further apart than single precision's exponents, no path at all, and edges forbidden under q only (infinite results)."""
    N, ninf = 24, float("-inf")
    p, q, lens = _pair(9200 + T, 8, N, T, dtype=dtype, ragged=False, min_len=N)
    lens = torch.full((8,), N, dtype=torch.int32)
    p[0, 5:] += 210.0
    p[1, 6:, :, T // 2] = ninf
    p[2, 0, :, 0] = ninf
    p[3, :, :, 0] = ninf
    p[4, :, :, T - 1] -= 150.0
    p[5, 20] = ninf
    q[6, 7, :, 3] = ninf
    q[7, :, 1, :] -= 200.0
    _check_all(crf, oracle_mod, p, q, lens, f"T={T} {dtype}")


@pytest.mark.parametrize("T", [36, 47, 50, 64])
@pytest.mark.parametrize("N", [5, 6, 7, 8, 9, 10])
def test_a_refused_step_at_every_place_of_a_chain(crf, oracle_mod, T, N):
    """The steps go three a round, the last one or two behind the rounds: every remainder of both half chains, and a step that scaled
    probabilities do not take (entries two hundred bits apart) at every position, once each."""
    p, q, _ = _pair(9250 + 16 * T + N, 2 * N, N, T, dtype="f32", ragged=False, min_len=N)
    lens = torch.full((2 * N,), N, dtype=torch.int32)
    lens[N:] = torch.arange(N) + 1
    for i in range(1, N):
        p[i, i, :, 2] += 90.0
        p[i, i, 1, :] -= 90.0
    _check_all(crf, oracle_mod, p, q, lens, f"T={T} N={N}")


@pytest.mark.parametrize("T,N", [(33, 16), (33, 256), (48, 256), (64, 128), (64, 256)])
def test_entropy_of_nearly_deterministic_chains(crf, oracle_mod, T, N):
    """One path, a random one or one that stays in a tag for long, carries nearly all of the weight: the scaled chains form a small
    entropy from expected scores that are not small.  A position rounds three terms of one or two bits (log alpha, the expected
    score and their products): at most 3e-7 a position, and 1e-5 of the entropy as everywhere."""
    g = torch.Generator().manual_seed(9300 + T + N)
    phi = torch.randn(6, N, T, T, generator=g)
    y = torch.randint(0, T, (6, N), generator=g)
    y[4] = y[4, 0]
    prev = torch.cat([torch.zeros_like(y[:, :1]), y[:, :-1]], 1)
    phi[torch.arange(6)[:, None], torch.arange(N)[None, :], prev, y] += torch.tensor([10., 10., 12., 20., 12., 10.])[:, None]
    lens = torch.tensor([N, N, N, N, N, N - 3], dtype=torch.int32)
    got = crf.lccrf_entropy(phi.cuda(), lens.cuda()).cpu().numpy().astype(np.float64)
    want = oracle_mod.entropy(phi, lens.numpy())
    assert np.all(np.abs(got - want) <= 3e-7 * N + 1e-5 * want), f"T={T} N={N}: {got} vs {want}"
