"""GPU parity of the entropy, the cross-entropy and the KL divergence at 33 .. 64 tags, where their chains run in scaled
probabilities until a step leaves the accepted range and in the log domain from there on, against the CPU oracle
(from its fp64 marginals).  Tolerances as in test_gpu_two_chains.py: 1e-5 of the sizes the results are differences of."""
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
    lz = np.abs(np.nan_to_num(oracle_mod.log_partition(p, lens.numpy()), posinf=0, neginf=0))
    bad = ~(np.isnan(got) & np.isnan(want)) & ~(np.abs(got - want) <= 1e-5 * np.maximum(1.0, lz))
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
