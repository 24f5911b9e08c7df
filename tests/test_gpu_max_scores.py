"""Best paths at 65 .. 256 tags whose scores run along the chains alone and whose pointers are found afterwards: tags and scores are
those of the sequential schedule bit for bit (the same additions in double precision, the first of equals) at the edges of
every instantiation, rows off the 16-byte grid, exact ties, forbidden transitions, a tag and a position without any path, NaN,
every short length; the call without room for the scores takes the other schedule and gives the same."""
import pytest
import torch

from test_gpu_parity import crf  # noqa: F401  (the module-scoped binding fixture)

pytestmark = pytest.mark.gpu


def _potentials(gen, *shape, special):
    x = torch.randint(0, 4, shape, generator=gen).to(torch.float32)  # (ties everywhere)
    if special:
        x[torch.rand(shape, generator=gen) < 0.5] = float("-inf")
        x[torch.rand(shape, generator=gen) < 0.01] = float("nan")
    return x


def _lengths(N):
    return torch.tensor([N, N - 1, 1, 0, 2, 3, (N + 1) // 2], dtype=torch.int32)


def _score_bytes(B, N, T):
    return (B * N * T * 8 + 255) // 256 * 256


@pytest.mark.parametrize("special", (False, True))
@pytest.mark.parametrize("dtype", (torch.float32, torch.bfloat16))
@pytest.mark.parametrize("T", (65, 68, 95, 96, 97, 127, 128, 129, 160, 161, 207, 208, 209, 255, 256))
def test_scores_then_pointers(crf, T, dtype, special):
    B, N = 7, 33
    g = torch.Generator().manual_seed(9100 + T)
    phi = _potentials(g, B, N, T, T, special=special)
    phi[5, 1, :, T // 2] = phi[6, 2, T - 1, :] = float("-inf")
    phi[1, N // 2] = float("-inf")
    phi, lens = phi.to(dtype).cuda(), _lengths(N).cuda()
    s, y = crf.lccrf_argmax(phi, lens)
    s_seq, y_seq = crf.lccrf_argmax(phi, lens, algo=crf.ALGO_SEQUENTIAL)
    assert torch.equal(y, y_seq) and torch.equal(s.view(torch.int32), s_seq.view(torch.int32))
    dt = crf.LCCRF_F32 if dtype == torch.float32 else crf.LCCRF_BF16
    small = torch.empty(crf.workspace_bytes(crf.OP_ARGMAX, B, N, T, dt) - _score_bytes(B, N, T), dtype=torch.uint8, device="cuda")
    s_b, y_b = crf.lccrf_argmax(phi, lens, workspace=small)
    assert torch.equal(y, y_b) and torch.equal(s.view(torch.int32), s_b.view(torch.int32))
    with pytest.raises(crf.LccrfError):
        crf.lccrf_argmax(phi, lens, workspace=small[:-256])


@pytest.mark.parametrize("special", (False, True))
@pytest.mark.parametrize("N", (6, 7, 40))
@pytest.mark.parametrize("T", (65, 96, 97, 111, 128))
def test_structured_scores_then_pointers(crf, T, N, special):
    B = 7
    g = torch.Generator().manual_seed(9200 + 3 * T + N)
    emit, trans = _potentials(g, B, N, T, special=special), _potentials(g, T, T, special=special)
    trans[:, T // 2] = float("-inf")
    emit[1, N // 2] = float("-inf")
    phi = (emit[:, :, None, :] + trans[None, None]).contiguous().cuda()
    emit, trans, lens = emit.cuda(), trans.cuda(), _lengths(N).cuda()
    s, y = crf.lccrf_argmax_structured(emit, trans, lens)
    s_seq, y_seq = crf.lccrf_argmax(phi, lens, algo=crf.ALGO_SEQUENTIAL)
    assert torch.equal(y, y_seq) and torch.equal(s.view(torch.int32), s_seq.view(torch.int32))
    small = torch.empty(crf.workspace_bytes(crf.OP_ARGMAX, B, N, T, crf.LCCRF_F32) - _score_bytes(B, N, T), dtype=torch.uint8, device="cuda")
    s_b, y_b = crf.lccrf_argmax_structured(emit, trans, lens, workspace=small)
    assert torch.equal(y, y_b) and torch.equal(s.view(torch.int32), s_b.view(torch.int32))


@pytest.mark.parametrize("B,N,T", [(300, 43, 65), (128, 96, 96), (128, 97, 97), (450, 600, 65)])
def test_positions_are_searched_in_large_padded_batches(crf, B, N, T):
    """More positions than get a workgroup each (12288, and more than a workgroup looks at in one go, 64 of every 4096), nearly all of them
    padding, a few sequences of full length among them: the kernels that carry the tags along give the same."""
    g = torch.Generator().manual_seed(9300 + T)
    emit, trans = _potentials(g, B, N, T, special=False).cuda(), _potentials(g, T, T, special=False).cuda()
    lens = torch.randint(0, 9, (B,), generator=g).to(torch.int32)
    lens[::37] = N
    lens = lens.cuda()
    room = crf.workspace_bytes(crf.OP_ARGMAX, B, N, T, crf.LCCRF_F32)
    small = torch.empty(room - _score_bytes(B, N, T), dtype=torch.uint8, device="cuda")
    for ln in (lens, None):
        full = torch.empty(room, dtype=torch.uint8, device="cuda").fill_(255)
        s, y = crf.lccrf_argmax_structured(emit, trans, ln, workspace=full)
        s_b, y_b = crf.lccrf_argmax_structured(emit, trans, ln, workspace=small)
        assert torch.equal(y, y_b) and torch.equal(s.view(torch.int32), s_b.view(torch.int32))


@pytest.mark.parametrize("dtype,T,B,N", [(torch.float32, 130, 17, 400), (torch.bfloat16, 209, 24, 300), (torch.bfloat16, 73, 70, 180)])
def test_positions_are_searched_dense(crf, dtype, T, B, N):
    """The same over dense potentials, two workgroups a position from 129 tags on."""
    g = torch.Generator(device="cuda").manual_seed(9400 + T)
    phi = torch.randint(0, 4, (B, N, T, T), generator=g, device="cuda").to(dtype)
    lens = torch.randint(0, 9, (B,), generator=g, device="cuda").to(torch.int32)
    lens[::7] = N
    for ln in (lens, None):
        s, y = crf.lccrf_argmax(phi, ln)
        s_seq, y_seq = crf.lccrf_argmax(phi, ln, algo=crf.ALGO_SEQUENTIAL)
        assert torch.equal(y, y_seq) and torch.equal(s.view(torch.int32), s_seq.view(torch.int32))
