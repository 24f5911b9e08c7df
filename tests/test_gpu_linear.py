"""First passes in scaled probabilities (33 .. 256 tags) and marginals written by a kernel of their own, against the
oracle: the tag counts at the edges of every instantiation (rows a thread holds, pieces off the 16-byte grid), steps that
are not accepted (forbidden tags, jumps of the scale, vectors hundreds of bits apart) in the middle of accepted ones, and
every short length.  Tolerances as everywhere for these queries (fp32 sums of a few hundred terms: 1e-5)."""
import pytest
import torch

from paper_2308_03291_amd import workloads
from test_gpu_parity import check_case, crf  # noqa: F401  (crf: the module-scoped binding fixture)

pytestmark = pytest.mark.gpu

TAGS = [65, 66, 88, 89, 101, 126, 129, 132, 141, 144, 157, 161, 176, 177, 189, 200, 201, 204, 205, 212, 225, 240, 241, 255, 256]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", TAGS)
def test_linear_first_pass_and_edge_marginals(crf, oracle_mod, T, dtype):
    N = 30
    phi, _ = workloads.random_case(7100 + T, 7, N, T, scale=2.0, dtype=dtype)
    phi[1, 11, :, 5] = float("-inf")      # a forbidden tag: a step that is not accepted, among others that are
    phi[2, 7] += 250.0                    # jumps of the scale in either half
    phi[2, 23] -= 250.0
    phi[3, :, :, T - 1] = float("-inf")   # a tag forbidden everywhere: log-domain steps throughout
    lens = torch.tensor([N, N - 1, N, N, 2, 1, 0], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, what=f"linear T={T} {dtype}", queries=("logz", "mu"))


@pytest.mark.parametrize("T", [45, 63, 99, 201])
def test_bfloat16_rows_off_the_grid(crf, oracle_mod, T):
    """The first pass of larger batches (no edge marginals) at odd tag counts, the tensor's last matrix included."""
    phi, _ = workloads.random_case(7300 + T, 130, 9, T, scale=1.5, dtype="bf16")
    check_case(crf, oracle_mod, phi, None, what=f"odd rows T={T}", queries=("logz", "mu"), algo=crf.ALGO_SEQUENTIAL)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [217, 220, 223, 224, 237, 239, 240])
def test_last_matrix_of_full_length_sequences(crf, oracle_mod, T, dtype):
    """Tag counts whose instance holds a row more than they need (217 .. 224, 239, 240), and one that does not; the last
    sequence ends with the tensor.  (That no row past the matrix is taken is asserted on the host: test_abi_host.py.)"""
    phi, _ = workloads.random_case(7200 + T, 3, 12, T, scale=2.0, dtype=dtype)
    check_case(crf, oracle_mod, phi, None, what=f"linear, full length, T={T} {dtype}", queries=("logz", "mu"))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [45, 67, 99, 136, 201])
def test_tags_that_chains_cannot_start_with(crf, oracle_mod, T, dtype):
    """A tag forbidden everywhere (as a successor, as a predecessor too), one that is forbidden at the start only, one whose only way in
    comes from a tag that is itself unreachable, several at once: whether a chain tries scaled steps is decided by such tags."""
    N, ninf = 17, float("-inf")
    phi, _ = workloads.random_case(7600 + T, 7, N, T, dtype=dtype)
    phi[0, :, :, 7] = ninf
    phi[1, :, :, 7] = ninf
    phi[1, 1:, 7, :] = ninf
    phi[2, 0, :, 7:12] = ninf
    phi[3, 0, :, 3:5] = ninf
    phi[3, 1, :, 3] = ninf
    phi[3, 1, 4, 3] = 0.0
    phi[4, :, :, T - 1] = ninf
    phi[4, 0, :, 0] = ninf
    phi[5, :, :, 2:] = ninf
    lens = torch.tensor([N, N, N, N, N - 1, N, 2], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, what=f"no start T={T} {dtype}", queries=("logz", "mu"), algo=crf.ALGO_SEQUENTIAL)


@pytest.mark.parametrize("T,B,dtype", [(152, 49, "f32"), (153, 48, "f32"), (153, 49, "f32"), (180, 49, "f32"), (181, 24, "f32"), (192, 25, "f32"),
                                       (193, 80, "f32"), (212, 81, "f32"), (213, 24, "f32"), (256, 25, "f32"), (213, 64, "bf16"),
                                       (240, 65, "bf16"), (241, 32, "bf16"), (256, 33, "bf16")])
def test_either_side_of_the_batch_that_scaled_steps_pay_for(crf, oracle_mod, T, B, dtype):
    phi, _ = workloads.random_case(7700 + T + B, B, 4, T, scale=1.5, dtype=dtype)
    lens = torch.randint(0, 5, (B,), generator=torch.Generator().manual_seed(T)).to(torch.int32)
    lens[-1] = 4
    check_case(crf, oracle_mod, phi, lens, what=f"batch T={T} B={B} {dtype}", queries=("logz",))


def test_nothing_is_read_past_the_tensor(crf, oracle_mod):
    """NaN right behind the potentials (T odd: rows end anywhere).  A value that is read there and meets an exact zero only
    sends the chain to its log-domain steps: what the kernels may read is asserted on the host (test_abi_host.py)."""
    for T, dtype in ((129, "f32"), (201, "bf16"), (67, "f32"), (99, "bf16")):
        phi, _ = workloads.random_case(7400 + T, 2, 9, T, dtype=dtype)
        flat = torch.full((phi.numel() + 64,), float("nan"), dtype=phi.dtype, device="cuda")
        flat[:phi.numel()] = phi.reshape(-1).cuda()
        check_case(crf, oracle_mod, phi, None, poison=False, what=f"tensor end T={T}", queries=("logz", "mu"),
                   device_phi=flat[:phi.numel()].view(phi.shape))


@pytest.mark.parametrize("T,N", [(65, 96), (129, 128), (201, 128), (256, 64)])
def test_rounding_of_flat_marginals(crf, T, N):
    """Potentials near zero: T^2 edges of nearly the same small probability.  Relative error (2-norm) against 64 bits: alpha, beta and
    the potential enter an exponent of a few bits (three roundings of at most 2^-23, uniform, times ln 2: 7e-8) behind the
    hardware's exponentials and logarithms (1e-7 each at most): 2.5e-7."""
    phi = 0.3 * torch.randn(3, N, T, T, generator=torch.Generator().manual_seed(7500 + T))
    phi = phi.bfloat16().cuda()
    mu = crf.lccrf_marginals(phi)[1]
    x = phi.double()
    a, b = [x[:, 0, 0]], [torch.zeros(3, T, dtype=torch.float64, device="cuda")]
    for i in range(1, N):
        a.append(torch.logsumexp(a[-1][:, :, None] + x[:, i], 1))
        b.append(torch.logsumexp(x[:, N - i] + b[-1][:, None, :], 2))
    b.reverse()
    lz = torch.logsumexp(a[-1], 1)
    num = den = 0.0
    for i in range(1, N):
        want = torch.exp(a[i - 1][:, :, None] + x[:, i] + b[i][:, None, :] - lz[:, None, None])
        num += float(((mu[:, i].double() - want) ** 2).sum())
        den += float((want ** 2).sum())
    assert (num / den) ** 0.5 <= 2.5e-7
