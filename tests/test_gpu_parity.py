"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element,
on the same seeded inputs.

Tolerances (fixed by the benchmark spec): logZ relative 1e-5 (absolute 1e-5 when |logZ| < 1);
marginals absolute 1e-5 for float32 potentials, 1e-4 for bfloat16-stored potentials; Viterbi
tags identical wherever the oracle's gap between the best and the second-best path exceeds
1e-3, and otherwise any valid path whose score is within the logZ tolerance of the best.
"""
import math

import numpy as np
import pytest
import torch

from paper_2308_03291_amd import workloads

pytestmark = pytest.mark.gpu

LOGZ_RTOL = 1e-5
MU_ATOL = {"f32": 1e-5, "bf16": 1e-4}
GAP_MIN = 1e-3


@pytest.fixture(scope="module")
def crf():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2308_03291_amd import binding
    binding.load_library()   # fails loudly if the HIP library was not built
    return binding


def _close_logz(got, want, what=""):
    got = np.asarray(got, dtype=np.float64)
    want = np.asarray(want, dtype=np.float64)
    tol = LOGZ_RTOL * np.maximum(np.abs(want), 1.0)
    both_ninf = np.isneginf(got) & np.isneginf(want)
    bad = ~both_ninf & ~(np.abs(got - want) <= tol)
    assert not bad.any(), f"{what}: logZ/score mismatch at {np.nonzero(bad)[0][:8]}: {got[bad][:4]} vs {want[bad][:4]}"


def _path_score(phi64, y, L):
    if L == 0:
        return 0.0
    s = phi64[0, 0, y[0]]
    for i in range(1, L):
        s += phi64[i, y[i - 1], y[i]]
    return float(s)


def check_case(crf, oracle_mod, phi_cpu, lens_cpu, *, poison=True, algo=0, what="", queries=("logz", "mu", "vit"),
               device_phi=None):
    """Run the requested queries on the GPU and compare everything with the oracle."""
    B, N, T, _ = phi_cpu.shape
    kind = "bf16" if phi_cpu.dtype == torch.bfloat16 else "f32"
    lens_np = None if lens_cpu is None else lens_cpu.numpy()
    eff = np.full((B,), N) if lens_np is None else np.clip(lens_np, 0, N)
    dev = torch.device("cuda:0")
    if device_phi is None:
        src = phi_cpu
        if poison and kind == "f32":
            # nothing outside the chain may be read: fill it with NaN on the device copy only
            src = phi_cpu.clone()
            for b in range(B):
                src[b, eff[b]:] = float("nan")
                if eff[b] > 0:
                    src[b, 0, 1:] = float("nan")
        device_phi = src.to(dev)
    lens_dev = None if lens_cpu is None else lens_cpu.to(dev)

    if "logz" in queries:
        out = torch.full((B,), float("nan"), device=dev)
        crf.lccrf_log_partition(device_phi, lens_dev, out=out, algo=algo)
        want = oracle_mod.log_partition(phi_cpu, lens_np)
        _close_logz(out.cpu().numpy(), want, what + " log_partition")

    if "mu" in queries:
        mu = torch.full((B, N, T, T), float("nan"), device=dev)
        lz = torch.full((B,), float("nan"), device=dev)
        crf.lccrf_marginals(device_phi, lens_dev, out=mu, logZ=lz, algo=algo)
        want_lz, want_mu = oracle_mod.marginals(phi_cpu, lens_np)
        _close_logz(lz.cpu().numpy(), want_lz, what + " marginals.logZ")
        got_mu = mu.cpu().numpy().astype(np.float64)
        assert np.isfinite(got_mu).all(), f"{what}: non-finite marginals"
        err = np.abs(got_mu - want_mu).max()
        assert err <= MU_ATOL[kind], f"{what}: max |mu - oracle| = {err:.3e}"
        for b in range(B):   # exact zeros where no edge exists
            assert not got_mu[b, eff[b]:].any(), f"{what}: marginals past the length of sequence {b}"
            if eff[b] > 0:
                assert not got_mu[b, 0, 1:].any(), f"{what}: rows s>0 of position 0, sequence {b}"

    if "vit" in queries:
        tags = torch.full((B, N), -7, dtype=torch.int32, device=dev)
        score = torch.full((B,), float("nan"), device=dev)
        crf.lccrf_argmax(device_phi, lens_dev, out=tags, score=score, algo=algo)
        want_score, want_tags, gap = oracle_mod.viterbi(phi_cpu, lens_np)
        got_tags = tags.cpu().numpy()
        got_score = score.cpu().numpy().astype(np.float64)
        _close_logz(got_score, want_score, what + " argmax.score")
        phi64 = phi_cpu.to(torch.float32).numpy().astype(np.float64)
        for b in range(B):
            L = int(eff[b])
            assert (got_tags[b, L:] == -1).all(), f"{what}: tags past the length of sequence {b}"
            y = got_tags[b, :L]
            assert ((y >= 0) & (y < T)).all(), f"{what}: tag out of range in sequence {b}"
            if gap[b] > GAP_MIN:
                assert np.array_equal(y, want_tags[b, :L]), \
                    f"{what}: Viterbi path differs in sequence {b} (gap {gap[b]:.3g})"
            elif np.isfinite(want_score[b]):
                s = _path_score(phi64[b], y, L)
                # a near-tie: any path whose own score is the best score within the logZ tolerance
                assert abs(s - want_score[b]) <= LOGZ_RTOL * max(1.0, abs(want_score[b]))


# ---------------------------------------------------------------------------------------
# sweeps over small and odd shapes: several tiles, ragged tails, degenerate sizes

SWEEP = []
for T_ in (1, 2, 3, 5, 16, 17, 32, 48, 64, 100, 128):
    for N_ in (1, 2, 3, 7, 64, 65):
        if T_ * T_ * N_ <= 128 * 128 * 7 or (N_ in (64,) and T_ in (16, 32, 48)):
            SWEEP.append((T_, N_))
SWEEP += [(128, 65), (100, 64), (64, 65), (17, 65)]


@pytest.mark.parametrize("T,N", SWEEP)
def test_sweep_fp32(crf, oracle_mod, T, N):
    B = 5
    phi, _ = workloads.random_case(1000 + 7 * T + N, B, N, T, scale=1.5)
    lens = torch.tensor([N, 1, max(1, N // 2), 0, max(1, N - 1)], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, what=f"T={T} N={N}")


@pytest.mark.parametrize("T,N", [(16, 40), (17, 9), (48, 33), (5, 8), (128, 6)])
def test_sweep_bf16(crf, oracle_mod, T, N):
    phi, _ = workloads.random_case(2000 + T + N, 3, N, T, scale=6.0, dtype="bf16")
    lens = torch.tensor([N, max(1, N // 3), N - 1 if N > 1 else 1], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, poison=False, what=f"bf16 T={T} N={N}")


@pytest.mark.parametrize("T", (6, 7, 9, 13, 21, 30, 33, 45, 50, 63, 75, 99, 127))
@pytest.mark.parametrize("N", (2, 9, 40))
def test_sweep_tag_counts_off_the_16_byte_grid(crf, oracle_mod, T, N):
    """Tag counts that are no multiple of four under the sequential schedule: the rows of a matrix then lie at any
    multiple of four bytes (two for bfloat16), a piece of four columns is loaded from wherever it starts, the pieces
    that run past the end of a row take what follows in the matrix, and the piece that ends a matrix is loaded
    element by element (the poisoned positions behind a sequence's last matrix must stay unread).  Speculative and
    exact step, all three queries; bfloat16 for the chains long enough to have a middle."""
    B = 4
    phi, _ = workloads.random_case(2500 + 11 * T + N, B, N, T, scale=1.5)
    lens = torch.tensor([N, 1, max(1, N // 2), max(1, N - 1)], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, algo=crf.ALGO_SEQUENTIAL, what=f"sequential T={T} N={N}")
    check_case(crf, oracle_mod, phi, lens, algo=crf.ALGO_SEQUENTIAL_EXACT, what=f"exact T={T} N={N}", queries=("logz", "mu"))
    if N == 40:
        phi, _ = workloads.random_case(2600 + T, 2, N, T, scale=4.0, dtype="bf16")
        check_case(crf, oracle_mod, phi, torch.tensor([N, N - 3], dtype=torch.int32), poison=False,
                   algo=crf.ALGO_SEQUENTIAL, what=f"sequential bf16 T={T}")


@pytest.mark.parametrize("T", (13, 30, 45, 63, 99))
def test_tag_counts_off_the_16_byte_grid_forbidden_edges_and_jumps(crf, oracle_mod, T):
    """The same tag counts with -inf potentials, a sequence without a finite path and scales that jump by hundreds
    of nats between positions (rejected speculative steps, replayed exactly)."""
    N = 24
    phi, _ = workloads.random_case(2700 + T, 5, N, T)
    ninf = float("-inf")
    phi[0, 5, :, 7] = ninf
    phi[0, 19, 3, :] = ninf
    phi[1, 8, :, :] = ninf
    phi[2, 0, 0, 2] = ninf
    phi[3, 12, :, 1:] = ninf
    phi[3, 12, :, T - 1] = 0.0              # (the last column of a row: the piece that is cut short)
    phi[3, 12, :, 0] = ninf
    phi[4, ::3] += 300.0
    phi[4, 1::3] -= 300.0
    lens = torch.tensor([N, N, N, N, N - 3], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, poison=False, algo=crf.ALGO_SEQUENTIAL, what=f"sequential -inf / jumps T={T}")


@pytest.mark.parametrize("T", (1, 2, 3, 5, 6, 7, 13, 30, 45, 57, 63, 99, 131, 255))
def test_the_last_matrix_of_the_tensor_with_nothing_usable_behind_it(crf, oracle_mod, T):
    """Full-length sequences, so that the last matrix of the tensor is worked on, in a buffer that holds NaN right
    behind (and before) the tensor: whatever a load of four columns takes in past the end of a row must not reach a
    result, and for the piece that ends the tensor nothing past it is loaded at all (that part cannot be seen from
    the results; the kernels take the element-wise path there)."""
    B, N = 2, 3
    phi, _ = workloads.random_case(2800 + T, B, N, T, scale=1.5)
    n = phi.numel()
    buf = torch.full((n + 64,), float("nan"), device="cuda:0")
    buf[32:32 + n] = phi.reshape(-1).to("cuda:0")          # (32 floats in: the tensor stays 16-byte aligned)
    dphi = buf[32:32 + n].view(B, N, T, T)
    for algo in (crf.ALGO_SEQUENTIAL, crf.ALGO_SEQUENTIAL_EXACT):
        check_case(crf, oracle_mod, phi, None, algo=algo, what=f"tensor end T={T} algo={algo}", device_phi=dphi,
                   queries=("logz", "mu") if algo == crf.ALGO_SEQUENTIAL_EXACT else ("logz", "mu", "vit"))
    if 8 <= T <= 48:
        check_case(crf, oracle_mod, phi, None, algo=crf.ALGO_SEQUENTIAL_LANES, what=f"tensor end, lanes T={T}", device_phi=dphi)
    elif T <= 64:   # (the argmax has chain-wave kernels at every tag count up to 64)
        check_case(crf, oracle_mod, phi, None, algo=crf.ALGO_SEQUENTIAL_LANES, what=f"tensor end, lanes T={T}", device_phi=dphi,
                   queries=("vit",))
    if T <= 64:     # bfloat16 too: rows at any multiple of two bytes
        phih, _ = workloads.random_case(2850 + T, B, N, T, scale=3.0, dtype="bf16")
        bufh = torch.full((n + 64,), float("nan"), device="cuda:0", dtype=torch.bfloat16)
        bufh[32:32 + n] = phih.reshape(-1).to("cuda:0")
        dphih = bufh[32:32 + n].view(B, N, T, T)
        check_case(crf, oracle_mod, phih, None, algo=crf.ALGO_SEQUENTIAL, what=f"tensor end bf16 T={T}", device_phi=dphih)
        check_case(crf, oracle_mod, phih, None, algo=crf.ALGO_SEQUENTIAL_LANES, what=f"tensor end bf16, lanes T={T}", device_phi=dphih,
                   queries=("logz", "mu", "vit") if 8 <= T <= 48 else ("vit",))


@pytest.mark.parametrize("T", [255, 256, 129, 200])
def test_largest_tag_sets(crf, oracle_mod, T):
    phi, _ = workloads.random_case(3000 + T, 2, 5, T)
    lens = torch.tensor([5, 3], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, what=f"T={T}")


@pytest.mark.parametrize("T,dtype", [(129, "f32"), (192, "f32"), (193, "f32"), (250, "f32"), (256, "f32"), (200, "bf16"), (255, "bf16")])
def test_largest_tag_sets_long_chains(crf, oracle_mod, T, dtype):
    """129 .. 256 tags stream every matrix in batches of 64 rows (three batches up to 192 tags, four above):
    chains of 70 positions, ragged, with the speculative and the exact step, marginals and paths."""
    N = 70
    phi, _ = workloads.random_case(3050 + T, 4, N, T, scale=3.0 if dtype == "bf16" else 1.5, dtype=dtype)
    lens = torch.tensor([N, 1, N // 2, N - 1], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, poison=dtype == "f32", what=f"T={T} N={N} {dtype}")
    check_case(crf, oracle_mod, phi, lens, poison=False, algo=crf.ALGO_SEQUENTIAL_EXACT, what=f"exact T={T} N={N} {dtype}",
               queries=("logz", "mu"))


def test_largest_tag_sets_forbidden_edges_and_jumps(crf, oracle_mod):
    """The exact replay of the row-batch kernels (the matrix streamed again from memory): -inf potentials, a
    chain without a finite path, and scales that jump by hundreds of nats between positions."""
    T, N = 160, 24
    phi, _ = workloads.random_case(3060, 4, N, T)
    ninf = float("-inf")
    phi[0, 5, :, 7] = ninf
    phi[0, 9, 3, :] = ninf
    phi[1, 8, :, :] = ninf                       # no finite path at all
    phi[2, 3] += 400.0
    phi[2, 15] -= 400.0
    mask = torch.rand(N, T, T, generator=torch.Generator().manual_seed(5)) < 0.7
    phi[3][mask] = ninf
    phi[3, :, torch.arange(T), torch.arange(T)] = 0.0
    check_case(crf, oracle_mod, phi, None, poison=False, what="T=160 -inf and jumps", queries=("logz", "mu"))


def test_lengths_none_means_full(crf, oracle_mod):
    phi, _ = workloads.random_case(3100, 3, 9, 12)
    check_case(crf, oracle_mod, phi, None, what="lengths=None")


def test_lengths_are_clamped(crf, oracle_mod):
    phi, _ = workloads.random_case(3101, 4, 6, 8)
    lens = torch.tensor([-3, 99, 6, 2], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, poison=True, what="clamped lengths")


# ---------------------------------------------------------------------------------------
# special values

def test_zero_potentials(crf):
    B, N, T = 3, 50, 24
    phi = torch.zeros(B, N, T, T, device="cuda:0")
    lens = torch.tensor([50, 17, 1], dtype=torch.int32, device="cuda:0")
    lz, mu = crf.lccrf_marginals(phi, lens)
    want = lens.cpu().numpy() * math.log(T)
    _close_logz(lz.cpu().numpy(), want, "zero potentials")
    mu = mu.cpu().numpy()
    assert np.allclose(mu[0, 1:], 1.0 / T ** 2, atol=1e-7)
    assert np.allclose(mu[0, 0, 0], 1.0 / T, atol=1e-7)
    score, tags = crf.lccrf_argmax(phi, lens)
    assert (score.cpu().numpy() == 0).all()
    t = tags.cpu().numpy()
    assert (t[0] == 0).all() and (t[1, :17] == 0).all() and (t[1, 17:] == -1).all()


def test_banned_transitions(crf, oracle_mod):
    phi, _ = workloads.random_case(3200, 3, 7, 6)
    ninf = float("-inf")
    phi[0, 2, 1, :] = ninf
    phi[0, 3, :, 0] = ninf
    phi[1, 0, 0, 2] = ninf
    phi[1, 4, :, 1:] = ninf       # only tag 0 allowed at position 4
    phi[2, 3, :, :] = ninf        # no finite path at all in sequence 2
    lens = torch.tensor([7, 6, 7], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, poison=False, what="-inf potentials", queries=("logz", "mu"))
    # argmax on the feasible sequences only
    check_case(crf, oracle_mod, phi[:2].contiguous(), lens[:2], poison=False, what="-inf potentials",
               queries=("vit",))


def test_hmm_total_mass_is_one(crf):
    """Row-stochastic potentials: logZ = 0 up to float32 rounding of the inputs."""
    g = torch.Generator().manual_seed(77)
    B, N, T = 2, 300, 20
    P = torch.rand(B, N, T, T, generator=g, dtype=torch.float64) + 0.05
    P /= P.sum(dim=3, keepdim=True)
    phi = P.log().to(torch.float32)
    lz = crf.lccrf_log_partition(phi.cuda()).cpu().numpy()
    assert np.abs(lz).max() < 2e-4


def test_large_offsets_keep_precision(crf, oracle_mod):
    """A big constant added to every matrix moves logZ by N * c; marginals must not degrade."""
    phi, _ = workloads.random_case(3300, 2, 200, 16)
    phi = phi + 300.0
    check_case(crf, oracle_mod, phi, None, poison=False, what="offset +300", queries=("logz", "mu"))


def test_repeat_runs_are_bit_identical(crf):
    w = workloads.WORKLOADS["cfg2"]
    phi = workloads.phi_batch(w).cuda()
    lens = workloads.lengths(w).cuda()
    lz1, mu1 = crf.lccrf_marginals(phi, lens)
    s1, t1 = crf.lccrf_argmax(phi, lens)
    for _ in range(3):
        lz2, mu2 = crf.lccrf_marginals(phi, lens)
        s2, t2 = crf.lccrf_argmax(phi, lens)
        assert torch.equal(lz1, lz2) and torch.equal(mu1, mu2)
        assert torch.equal(s1, s2) and torch.equal(t1, t2)


def test_dirty_workspace_and_side_stream(crf, oracle_mod):
    phi, lens = workloads.random_case(3400, 6, 30, 20, ragged=True, min_len=0)
    dev = torch.device("cuda:0")
    B, N, T, _ = phi.shape
    need = max(crf.workspace_bytes(op, B, N, T, 0) for op in (0, 1, 2))
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=dev)   # all-ones bytes: NaN as floats
    st = torch.cuda.Stream(device=dev)
    phid, lensd = phi.to(dev), lens.to(dev)
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        lz, mu = crf.lccrf_marginals(phid, lensd, workspace=ws)
        ws.fill_(0xFF)
        score, tags = crf.lccrf_argmax(phid, lensd, workspace=ws)
    st.synchronize()
    want_lz, want_mu = oracle_mod.marginals(phi, lens.numpy())
    _close_logz(lz.cpu().numpy(), want_lz, "side stream")
    assert np.abs(mu.cpu().numpy() - want_mu).max() <= 1e-5
    want_score, want_tags, gap = oracle_mod.viterbi(phi, lens.numpy())
    _close_logz(score.cpu().numpy(), want_score, "side stream score")
    for b in range(B):
        if gap[b] > GAP_MIN:
            assert np.array_equal(tags[b].cpu().numpy(), want_tags[b])


# ---------------------------------------------------------------------------------------
# the two step flavours of the sequential schedule

@pytest.mark.parametrize("T,N", [(5, 8), (16, 40), (32, 64), (36, 44), (48, 33), (64, 30), (100, 9), (128, 12), (255, 4)])
def test_exact_schedule(crf, oracle_mod, T, N):
    """Every position through the exact step (the one that otherwise only replays rejected
    speculative steps)."""
    phi, lens = workloads.random_case(4000 + T, 4, N, T, scale=2.0, ragged=True, min_len=1)
    check_case(crf, oracle_mod, phi, lens, algo=crf.ALGO_SEQUENTIAL_EXACT, what=f"exact T={T} N={N}",
               queries=("logz", "mu"))


@pytest.mark.parametrize("T,N", [(16, 64), (32, 40), (36, 44), (48, 21), (60, 25), (64, 30), (128, 10)])
def test_scale_jumps_force_replays(crf, oracle_mod, T, N):
    """Potentials whose scale jumps by hundreds of nats between neighbouring positions: the
    speculative step (shift = previous normaliser) must be rejected and replayed exactly, also
    in the middle of a chain and in both directions."""
    phi, lens = workloads.random_case(4100 + T, 3, N, T, scale=1.0, ragged=True, min_len=N // 2)
    g = torch.Generator().manual_seed(99 + T)
    jump = (torch.randint(0, 3, (3, N, 1, 1), generator=g).to(torch.float32) - 1.0) * 300.0
    jump[:, ::5] = 0.0
    phi = (phi + jump).contiguous()
    check_case(crf, oracle_mod, phi, lens, what=f"jumps T={T} N={N}", queries=("logz", "mu"))


@pytest.mark.parametrize("N,lens", [(2, [2, 1, 0]), (3, [3, 2, 3]), (9, [9, 4, 7]), (40, [40, 33, 5]), (65, [65, 64, 2])])
def test_paired_second_pass(crf, oracle_mod, N, lens):
    """T = 128 with few sequences: the default schedule serves every chain with two workgroups
    that exchange half vectors each step; it must agree with the oracle and, closely, with the
    one-workgroup-per-chain schedule."""
    T = 128
    phi, _ = workloads.random_case(4200 + N, len(lens), N, T, scale=1.3)
    lens_t = torch.tensor(lens, dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens_t, what=f"paired N={N}", queries=("mu",))
    dphi, dl = phi.cuda(), lens_t.cuda()
    lz_a, mu_a = crf.lccrf_marginals(dphi, dl)
    lz_b, mu_b = crf.lccrf_marginals(dphi, dl, algo=crf.ALGO_SEQUENTIAL)
    assert torch.allclose(lz_a, lz_b, rtol=1e-6, atol=1e-6)
    assert float((mu_a - mu_b).abs().max()) < 2e-6


def test_paired_second_pass_hands_failures_to_the_exact_kernel(crf, oracle_mod):
    """Sequences the paired speculative pass must give up on (forbidden edges, no finite path,
    scale jumps) are recomputed exactly; the others in the same batch are not disturbed."""
    T, N = 128, 12
    phi, _ = workloads.random_case(4300, 5, N, T)
    ninf = float("-inf")
    phi[1, 5, :, 7] = ninf                       # a forbidden tag
    phi[2, 8, :, :] = ninf                       # no finite path at all
    phi[3, 3] += 400.0                           # scale jump in the forward half
    phi[3, 9] -= 400.0                           # and in the backward half
    lens = torch.tensor([12, 12, 12, 12, 11], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, poison=False, what="paired failures", queries=("logz", "mu"))


def test_paired_second_pass_bf16(crf, oracle_mod):
    phi, _ = workloads.random_case(4400, 2, 30, 128, scale=3.0, dtype="bf16")
    check_case(crf, oracle_mod, phi, None, poison=False, what="paired bf16", queries=("mu",))


def test_speculative_and_exact_agree_closely(crf):
    w = workloads.WORKLOADS["cfg2"]
    phi = workloads.phi_batch(w).cuda()
    lens = workloads.lengths(w).cuda()
    lz_a, mu_a = crf.lccrf_marginals(phi, lens)
    lz_b, mu_b = crf.lccrf_marginals(phi, lens, algo=crf.ALGO_SEQUENTIAL_EXACT)
    assert torch.allclose(lz_a, lz_b, rtol=1e-6, atol=0)
    assert float((mu_a - mu_b).abs().max()) < 2e-6


# ---------------------------------------------------------------------------------------
# the named workloads

@pytest.mark.parametrize("key", ["cfg1", "cfg2", "cfg3"])
def test_named_workloads_full(crf, oracle_mod, key):
    w = workloads.WORKLOADS[key]
    phi = workloads.phi_batch(w)
    lens = workloads.lengths(w)
    check_case(crf, oracle_mod, phi, lens, what=key)


def test_config5_long_peaked_bf16(crf, oracle_mod):
    w = workloads.WORKLOADS["cfg5"]
    phi = workloads.phi_batch(w)
    lens = workloads.lengths(w)
    check_case(crf, oracle_mod, phi, lens, poison=False, what="cfg5")


def test_config4_full_size_all_sequences(crf, oracle_mod):
    """The 2.1 GB workload in the launch configuration the benchmark times.  The GPU runs the whole
    batch in one call per query; the oracle then recomputes ALL 64 sequences, eight at a time (to bound
    host memory: the float64 marginals of eight sequences are 0.5 GB), and every logZ, every marginal,
    every Viterbi score and every tag path is compared."""
    w = workloads.WORKLOADS["cfg4"]
    dev = torch.device("cuda:0")
    phi_dev = torch.empty(w.B, w.N, w.T, w.T, dtype=torch.float32, device=dev)
    workloads.phi_batch(w, out=phi_dev)
    lens = workloads.lengths(w)
    lens_dev = lens.to(dev)
    mu = torch.full((w.B, w.N, w.T, w.T), float("nan"), device=dev)
    lz = torch.full((w.B,), float("nan"), device=dev)
    crf.lccrf_marginals(phi_dev, lens_dev, out=mu, logZ=lz)
    lz_only = crf.lccrf_log_partition(phi_dev, lens_dev)
    score, tags = crf.lccrf_argmax(phi_dev, lens_dev)
    torch.cuda.synchronize()
    assert torch.allclose(lz, lz_only, rtol=1e-6, atol=0)
    got_lz = lz.cpu().numpy()
    got_lz_only = lz_only.cpu().numpy()
    got_score = score.cpu().numpy()
    got_tags = tags.cpu().numpy()
    worst = 0.0
    graded_paths = 0
    for b0 in range(0, w.B, 8):
        pick = list(range(b0, min(b0 + 8, w.B)))
        phi_b = torch.stack([workloads.phi_sequence(w, b) for b in pick]).contiguous()
        want_lz, want_mu = oracle_mod.marginals(phi_b, lens[pick].numpy())
        _close_logz(got_lz[pick], want_lz, f"cfg4 seqs {b0}.. marginals.logZ")
        _close_logz(got_lz_only[pick], want_lz, f"cfg4 seqs {b0}.. log_partition")
        got_mu = mu[b0:b0 + len(pick)].cpu().numpy()
        assert np.isfinite(got_mu).all()
        err = float(np.abs(got_mu - want_mu).max())
        worst = max(worst, err)
        assert err <= 1e-5, f"cfg4 seqs {b0}..{pick[-1]}: max |mu - oracle| = {err:.3e}"
        assert not got_mu[:, 0, 1:].any(), "rows s > 0 of position 0 must be exact zeros"
        del got_mu, want_mu
        want_score, want_tags, gap = oracle_mod.viterbi(phi_b, lens[pick].numpy())
        _close_logz(got_score[pick], want_score, f"cfg4 seqs {b0}.. argmax.score")
        phi64 = phi_b.numpy()
        for k, b in enumerate(pick):
            y = got_tags[b]
            assert ((y >= 0) & (y < w.T)).all()
            if gap[k] > GAP_MIN:
                assert np.array_equal(y, want_tags[k]), f"cfg4 seq {b}: Viterbi path differs (gap {gap[k]:.3g})"
                graded_paths += 1
            else:   # a near-tie: any path whose own score is the best score within the logZ tolerance
                s = _path_score(phi64[k].astype(np.float64), y, w.N)
                assert abs(s - want_score[k]) <= LOGZ_RTOL * max(1.0, abs(want_score[k]))
    assert graded_paths >= w.B // 2, "too few sequences with a clear top-2 gap to grade the paths"
    print(f"cfg4: all {w.B} sequences, max |mu - oracle| = {worst:.2e}, {graded_paths} paths graded bit-exact")


def test_paired_second_pass_bf16_full_length(crf, oracle_mod):
    """T = 128, N = 512 (config 4's chain length) with bfloat16-stored potentials; every marginal against the oracle.  (So few
    chains are walked in pieces; two workgroups per chain at this length: test_gpu_pieces.py.)"""
    phi, _ = workloads.random_case(4500, 3, 512, 128, scale=3.0, dtype="bf16")
    lens = torch.tensor([512, 511, 300], dtype=torch.int32)
    check_case(crf, oracle_mod, phi, lens, poison=False, what="paired bf16 N=512", queries=("logz", "mu"))


def test_paper_benchmark_shape(crf, oracle_mod):
    """The size the paper times this model on (appendix table of tested sizes): b=128, n=256, 32 tags."""
    w = workloads.WORKLOADS["paper_lccrf"]
    phi = workloads.phi_batch(w)
    pick = [0, 17, 127]
    dev_phi = phi.cuda()
    lz, mu = crf.lccrf_marginals(dev_phi)
    want_lz, want_mu = oracle_mod.marginals(phi[pick].contiguous(), None)
    _close_logz(lz.cpu().numpy()[pick], want_lz, "paper shape")
    assert np.abs(mu[pick].cpu().numpy() - want_mu).max() <= 1e-5


def test_paper_hmm_shape(crf, oracle_mod):
    """The paper's HMM size (same appendix table): one chain, n=128, 32 states: a single sequence
    leaves all parallelism to the two chains."""
    w = workloads.WORKLOADS["paper_hmm"]
    check_case(crf, oracle_mod, workloads.phi_batch(w), workloads.lengths(w), what="paper hmm shape")


def test_paired_second_pass_gives_up_when_the_wait_expires(crf, oracle_mod):
    """The bounded wait of the paired pass, made to expire from the host: with a poll limit of 0 every
    receiver gives up without looking, all four workgroups of every sequence stop, and the one-workgroup
    kernel recomputes the whole batch.  Every kernel exits normally; the results equal the oracle's and,
    bit for bit, those of the schedule that never uses pairs."""
    T, N = 128, 40
    phi, _ = workloads.random_case(4600, 6, N, T, scale=1.3)
    lens = torch.tensor([40, 39, 2, 17, 1, 0], dtype=torch.int32)
    dphi, dl = phi.cuda(), lens.cuda()
    lz_seq, mu_seq = crf.lccrf_marginals(dphi, dl, algo=crf.ALGO_SEQUENTIAL)
    lz_pair, mu_pair = crf.lccrf_marginals(dphi, dl)
    crf.set_pair_poll_limit(0)
    try:
        check_case(crf, oracle_mod, phi, lens, what="paired, wait expired", queries=("mu",))
        lz_0, mu_0 = crf.lccrf_marginals(dphi, dl)
        torch.cuda.synchronize()
    finally:
        crf.set_pair_poll_limit(-1)
    assert torch.equal(mu_0, mu_seq) and torch.equal(lz_0, lz_seq)
    # with the default limit the pairs do the work: close to, but rounded differently from, the other kernel
    assert float((mu_pair - mu_seq).abs().max()) < 2e-6
    assert not torch.equal(mu_pair, mu_seq)
    lz_again, mu_again = crf.lccrf_marginals(dphi, dl)      # and the default is back in force
    assert torch.equal(mu_again, mu_pair)


def _tie_rule_path(phi64, L, T, h):
    """Of all best paths (by enumeration), the one with the smallest tag at h, then at h-1, ..., 0, then at
    h+1, ..., L-1: the documented choice of the sequential schedule among exactly tied paths."""
    from oracle import brute
    paths = brute.all_paths(T, L)
    sc = brute.path_scores(phi64, L, paths)
    best = paths[sc == sc.max()]
    for i in [h] + list(range(h - 1, -1, -1)) + list(range(h + 1, L)):
        best = best[best[:, i] == best[:, i].min()]
    assert best.shape[0] == 1
    return best[0], float(sc.max())


@pytest.mark.parametrize("T,L", [(2, 4), (2, 9), (3, 7), (4, 6), (5, 5)])
def test_exactly_tied_best_paths_follow_the_documented_rule(crf, T, L):
    """Small integer potentials: many paths tie exactly (the sums are exact in any order).  The sequential
    schedule must return the path the header documents; the case T=2, L=4 with tied optima (0,0,1,0) and
    (0,0,0,1) tells that rule from "smallest tag from the back"."""
    N = L + 2
    g = torch.Generator().manual_seed(700 + 10 * T + L)
    B = 24
    phi = torch.randint(-1, 2, (B, N, T, T), generator=g).to(torch.float32)
    if (T, L) == (2, 4):
        phi[0] = 0.0
        phi[0, 1] = torch.tensor([[1.0, 0.0], [0.0, 0.0]])   # y0 = y1 = 0
        phi[0, 2] = torch.tensor([[1.0, 1.0], [0.0, 0.0]])   # y1 = 0, y2 free
        phi[0, 3] = torch.tensor([[0.0, 1.0], [1.0, 0.0]])   # y3 != y2
        phi[0, 0, 0] = torch.tensor([1.0, 0.0])
    lens = torch.full((B,), L, dtype=torch.int32)
    lens[1] = L - 1
    score, tags = crf.lccrf_argmax(phi.cuda(), lens.cuda(), algo=crf.ALGO_SEQUENTIAL)
    score, tags = score.cpu().numpy(), tags.cpu().numpy()
    ties = 0
    for b in range(B):
        Lb = int(lens[b])
        want, best = _tie_rule_path(phi[b].numpy().astype(np.float64), Lb, T, Lb // 2)
        assert score[b] == best
        assert np.array_equal(tags[b, :Lb], want), f"sequence {b}: {tags[b, :Lb]} vs {want}"
        assert (tags[b, Lb:] == -1).all()
    if (T, L) == (2, 4):
        assert list(tags[0, :4]) == [0, 0, 0, 1]
