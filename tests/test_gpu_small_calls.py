"""GPU parity of the kernels that small calls take, at the edges of their tiles: against plain
float64 on the same inputs."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def fr():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2609_36932_amd as m
    return m


def _problem(T, d, V, seed, dtype=torch.bfloat16):
    g = torch.Generator().manual_seed(seed)
    H = torch.randn(T, d, generator=g).to(dtype)
    W = (torch.randn(V, d, generator=g) / d ** 0.5).to(dtype)
    y = torch.randint(0, V, (T,), generator=g, dtype=torch.int32)
    z = H.double() @ W.double().T
    lse = torch.logsumexp(z, 1)
    logp = z.gather(1, y.long()[:, None])[:, 0] - lse
    old = (logp + 0.05 * torch.randn(T, generator=g)).float()
    return H, W, y, z, lse, logp, old


def _reference(H, W, y, z, lse, logp, old, off, adv):
    """GRPO (seq-mean, eps 0.2): loss, dhidden, dW in float64."""
    T, S = len(y), len(off) - 1
    L = torch.from_numpy(np.diff(off))
    seq = torch.repeat_interleave(torch.arange(S), L)
    A, w = adv.double()[seq], 1.0 / (S * L.double()[seq])
    lo, hi = 1.0 - float(np.float32(0.2)), 1.0 + float(np.float32(0.2))
    rho = torch.exp(logp - old.double())
    inside = ((A >= 0) & (rho <= hi)) | ((A < 0) & (rho >= lo))
    loss = -(w * torch.minimum(rho * A, rho.clamp(lo, hi) * A)).sum()
    g = -w * inside * rho * A
    dZ = -g[:, None] * torch.exp(z - lse[:, None])
    dZ[torch.arange(T), y.long()] += g
    return loss, dZ @ W.double(), dZ.T @ H.double()


def _rel(a, b):
    return float((a.double().cpu() - b).norm() / b.norm())


@pytest.mark.parametrize("T, d, V, need_dW, dh_dtype", [
    (1, 8, 512, True, torch.float32),         # one row, one chunk of columns
    (255, 264, 513, True, torch.bfloat16),    # a row short of a tile, ragged columns and vocabulary
    (257, 248, 640, False, torch.float32),    # a row over a tile, dhidden alone
    (40, 520, 63, True, torch.float32),       # fewer vocabulary rows than one K step: one part
    (300, 1000, 20011, True, torch.bfloat16),  # many parts
    (130, 264, 20480, False, torch.bfloat16),
])
def test_direct_dhidden(fr, T, d, V, need_dW, dh_dtype):
    """dhidden read from W itself with its K in parts.  1e-2 is the bar of bf16 gradients
    (operands of 2^-9 relative rounding)."""
    H, W, y, z, lse, logp, old = _problem(T, d, V, T + d)
    off = np.asarray(sorted({0, T // 3, T // 3 + T // 2, T}), dtype=np.int64)
    adv = torch.linspace(-1.0, 1.5, len(off) - 1)
    loss, dH, dW = _reference(H, W, y, z, lse, logp, old, off, adv)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    call = fr.policy_loss_fwd_bwd(
        H.to(DEV), W.to(DEV), y.to(DEV), old.to(DEV), torch.from_numpy(off).to(DEV),
        torch.from_numpy(off), adv.to(DEV), need_dW=need_dW, dhidden_dtype=dh_dtype, status=st)
    torch.cuda.synchronize()
    assert st.item() == 0
    assert abs(call.loss.item() - loss.item()) <= 1e-4 * abs(loss.item()) + 1e-6
    assert _rel(call.dhidden, dH) < 1e-2
    if need_dW:
        assert _rel(call.dW, dW) < 1e-2


def test_direct_dhidden_unaligned_output_and_repeat(fr):
    """A dhidden array that is aligned to its elements only is written like any other, and a
    second call gives the same bits (the parts are added in a fixed order)."""
    T, d, V = 70, 264, 20011
    H, W, y, z, lse, logp, old = _problem(T, d, V, 5)
    off = np.asarray([0, 30, T], dtype=np.int64)
    adv = torch.tensor([1.0, -0.5])
    _, dH, _ = _reference(H, W, y, z, lse, logp, old, off, adv)
    args = (H.to(DEV), W.to(DEV), y.to(DEV), old.to(DEV), torch.from_numpy(off).to(DEV),
            torch.from_numpy(off), adv.to(DEV))
    for dt in (torch.float32, torch.bfloat16):
        a = fr.policy_loss_fwd_bwd(*args, dhidden_dtype=dt)
        b = fr.LossCall(*args, dhidden_dtype=dt)
        flat = torch.empty(T * d + 1, dtype=dt, device=DEV)
        b.args.dhidden = flat.data_ptr() + flat.element_size()
        b.run()
        torch.cuda.synchronize()
        assert torch.equal(flat[1:].view(T, d), a.dhidden) and torch.equal(a.dW, b.dW)
        assert _rel(a.dhidden, dH) < 1e-2


@pytest.mark.parametrize("T, d, V, accumulate, dh_dtype", [
    (1, 8, 1, False, torch.float32),          # one of everything
    (65, 72, 257, True, torch.float32),       # a token, some columns and a vocabulary row over a tile
    (63, 40, 31, False, torch.bfloat16),      # fewer vocabulary rows than one K step
    (200, 136, 3001, True, torch.float32),    # dhidden in parts, a partial last K step everywhere
    (8200, 1024, 300, False, torch.float32),  # 128 x 128 dhidden tiles
    (130, 512, 16400, True, torch.float32),   # 128 x 128 dW tiles
])
def test_float32_tiles(fr, T, d, V, accumulate, dh_dtype):
    """float32 GEMM tiles: log-probs and gradients to float32 accuracy (1e-5: the sums' terms are
    of mixed sign, and up to 16400 of them follow each other; bf16 dhidden to its rounding)."""
    H, W, y, z, lse, logp, old = _problem(T, d, V, T + d, torch.float32)
    off = np.asarray(sorted({0, T // 3, T // 3 + T // 2, T}), dtype=np.int64)
    adv = torch.linspace(-1.0, 1.5, len(off) - 1)
    loss, dH, dW = _reference(H, W, y, z, lse, logp, old, off, adv)
    base = 1e-3 * torch.randn(V, d, generator=torch.Generator().manual_seed(1))
    rows = torch.arange(T - 1, -1, -1, dtype=torch.int32)  # gathered: stored in reverse order
    call = fr.policy_loss_fwd_bwd(
        H.flip(0).contiguous().to(DEV), W.to(DEV), y.flip(0).contiguous().to(DEV),
        old.flip(0).contiguous().to(DEV), torch.from_numpy(off).to(DEV), torch.from_numpy(off),
        adv.to(DEV), row_index=rows.to(DEV), dhidden_dtype=dh_dtype, need_entropy=True,
        dW=base.to(DEV) if accumulate else None, dW_accumulate=accumulate, T=T)
    torch.cuda.synchronize()
    assert (call.logp.double().cpu() - logp).abs().max() < 2e-5
    ent = lse - (torch.exp(z - lse[:, None]) * z).sum(1)
    assert (call.entropy.double().cpu() - ent).abs().max() < 2e-5
    if V > 1:  # (one class: every gradient is exactly a difference of equal numbers)
        assert _rel(call.dhidden, dH) < (1e-5 if dh_dtype == torch.float32 else 4e-3)
        assert _rel(call.dW, dW + base.double() * accumulate) < 1e-5


@pytest.mark.parametrize("T, d, V", [
    (1, 8, 1), (64, 40, 257), (65, 72, 700), (128, 264, 255), (129, 200, 511), (192, 64, 256),
    (193, 64, 20000),    # whole tiles, the last 79 cut in two
    (256, 64, 9000),     # 36 whole tiles, each cut in four
    (300, 136, 3000),    # a narrow column among the others
    (3200, 64, 5200),    # a narrow column after 12 whole ones
    (4096, 72, 5200),    # 16 whole columns of 21: the last 80 tiles cut in two
])
def test_logits_tiles(fr, T, d, V):
    """Logits tiles of every width: token_logprob (partials only) and the loss call (exp-logits
    stored, gradients from them) on gathered rows.  2e-5 absolute for the log-probs: float32 sums
    of values around 1 (bf16 inputs are exact in both)."""
    H, W, y, z, lse, logp, old = _problem(T, d, V, T + V)
    rows = torch.arange(T - 1, -1, -1, dtype=torch.int32).to(DEV)
    Hr, yr = H.flip(0).contiguous().to(DEV), y.flip(0).contiguous().to(DEV)
    lp, ls = fr.token_logprob(Hr, W.to(DEV), yr, row_index=rows)
    torch.cuda.synchronize()
    assert (lp.double().cpu() - logp).abs().max() < 2e-5
    assert (ls.double().cpu() - lse).abs().max() < 2e-5
    if V == 1:
        return
    off = np.asarray(sorted({0, T // 3, T // 3 + T // 2, T}), dtype=np.int64)
    adv = torch.linspace(-1.0, 1.5, len(off) - 1)
    loss, dH, dW = _reference(H, W, y, z, lse, logp, old, off, adv)
    call = fr.policy_loss_fwd_bwd(
        Hr, W.to(DEV), yr, old.flip(0).contiguous().to(DEV), torch.from_numpy(off).to(DEV),
        torch.from_numpy(off), adv.to(DEV), row_index=rows, T=T)
    torch.cuda.synchronize()
    assert (call.logp.double().cpu() - logp).abs().max() < 2e-5
    assert _rel(call.dhidden, dH) < 1e-2 and _rel(call.dW, dW) < 1e-2


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("T, big, offs", [
    (600, range(260, 301), (0, 130, 290, 600)),       # one of three 256-token blocks
    (600, range(512, 600), (0, 200, 512, 530, 600)),  # the narrow last column's, and only those
    (300, range(0, 300, 7), (0, 1, 33, 300)),         # some rows of every block
    (70, range(70), (0, 70)),                         # every row
])
def test_shifted_rows_in_one_slab(fr, dtype, T, big, offs):
    """Rows whose logits leave exp's range, in some 256-token blocks of one slab: exactly those rows
    are evaluated again with a shift, and every output matches float64, their neighbours' too.
    Log-probs: float32 values of up to ~300 (half an ulp 1.5e-5) summed over d = 72 and rounded a few
    times; gradients: bf16 operands, or that error in an exponent."""
    d, V = 72, 1300
    H, W, y, *_ = _problem(T, d, V, T + len(big), dtype)
    H[list(big)] *= 64.0
    z = H.double() @ W.double().T
    top = z.max(1).values
    assert not ((top.abs() > 55) & (top.abs() < 65)).any()
    lse = torch.logsumexp(z, 1)
    logp = z.gather(1, y.long()[:, None])[:, 0] - lse
    old = (logp + 0.05 * torch.randn(T, generator=torch.Generator().manual_seed(3))).float()
    off = np.asarray(offs, dtype=np.int64)
    adv = torch.linspace(-1.0, 1.5, len(off) - 1) if len(off) > 2 else torch.ones(1)
    loss, dH, dW = _reference(H, W, y, z, lse, logp, old, off, adv)
    rows = torch.arange(T - 1, -1, -1, dtype=torch.int32)
    call = fr.policy_loss_fwd_bwd(
        H.flip(0).contiguous().to(DEV), W.to(DEV), y.flip(0).contiguous().to(DEV),
        old.flip(0).contiguous().to(DEV), torch.from_numpy(off).to(DEV), torch.from_numpy(off),
        adv.to(DEV), row_index=rows.to(DEV), need_entropy=True, T=T)
    torch.cuda.synchronize()
    assert int(call.stats[1].item()) == int((top.abs() >= 60).sum()) == len(big)
    assert (call.lse.double().cpu() - lse).abs().max() < 2e-4
    assert (call.logp.double().cpu() - logp).abs().max() < 2e-4
    ent = lse - (torch.exp(z - lse[:, None]) * z).sum(1)
    assert (call.entropy.double().cpu() - ent).abs().max() < 2e-3
    assert abs(call.loss.item() - loss.item()) <= 1e-3 * abs(loss.item())
    tol = 1e-2 if dtype == torch.bfloat16 else 1e-3
    assert _rel(call.dhidden, dH) < tol and _rel(call.dW, dW) < tol


def test_launches_follow_the_current_stream(fr):
    """The handle passed to the library is torch's current stream, on the default one and inside a
    stream context."""
    assert fr._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert fr._stream() == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert fr._stream() == torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("T, need_dW", [(6144, True), (6145, True), (20480, False), (20481, False)])
def test_dhidden_on_both_sides_of_the_transposed_copy(fr, T, need_dW):
    """The last call that reads W itself and the first that transposes it, beside dW and alone (1e-2:
    the bar of bf16 gradients)."""
    d, V = 40, 330
    H, W, y, z, lse, logp, old = _problem(T, d, V, T)
    off = np.asarray([0, T // 3, T // 3 + T // 2, T], dtype=np.int64)
    adv = torch.linspace(-1.0, 1.5, 3)
    _, dH, dW = _reference(H, W, y, z, lse, logp, old, off, adv)
    call = fr.policy_loss_fwd_bwd(
        H.to(DEV), W.to(DEV), y.to(DEV), old.to(DEV), torch.from_numpy(off).to(DEV),
        torch.from_numpy(off), adv.to(DEV), need_dW=need_dW)
    torch.cuda.synchronize()
    assert _rel(call.dhidden, dH) < 1e-2
    if need_dW:
        assert _rel(call.dW, dW) < 1e-2


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("V", [300, 20011])  # 2 vocabulary blocks (30 of the merge's slices empty); 79
def test_rows_that_are_not_finite_or_very_negative(fr, dtype, V):
    """NaN and infinite hidden rows give NaN or infinite log-probs and leave their neighbours alone, in
    token_logprob and in a loss call with entropy and dhidden; logits around -3e4 over whole vocabulary
    blocks count for nothing.  Tolerances as in test_logits_tiles."""
    T, d = 40, 72
    H, W, y, *_ = _problem(T, d, V, V, dtype)
    H[:, 0] = 1.0
    W[:, 0] = 0.0
    W[256:290, 0] = -3e4                    # the second block's rows (all of it but a few at V = 300)
    if V > 512:
        W[256:512, 0] = -3e4
        W[-1, 0] = -3e4
    y[:] = torch.arange(T, dtype=torch.int32) * 6
    z = H.double() @ W.double().T
    lse = torch.logsumexp(z, 1)
    logp = z.gather(1, y.long()[:, None])[:, 0] - lse
    old = (logp + 0.01).float()
    off = np.asarray([0, 10, T], dtype=np.int64)
    adv = torch.tensor([1.0, -0.5])
    _, dH, _ = _reference(H, W, y, z, lse, logp, old, off, adv)
    ent = lse - (torch.exp(z - lse[:, None]) * z).sum(1)
    bad = torch.zeros(T, dtype=torch.bool)
    bad[[3, 11, 39]] = True
    H[3, 5] = float("nan")
    H[11, 7] = float("inf")
    H[39, 9] = -float("inf")
    args = (H.to(DEV), W.to(DEV), y.to(DEV))
    lp, ls = fr.token_logprob(*args)
    call = fr.policy_loss_fwd_bwd(*args, old.to(DEV), torch.from_numpy(off).to(DEV),
                                  torch.from_numpy(off), adv.to(DEV), need_dW=False,
                                  need_entropy=True)
    torch.cuda.synchronize()
    for got, want in ((lp, logp), (call.logp, logp), (ls, lse), (call.lse, lse), (call.entropy, ent)):
        got = got.double().cpu()
        assert not torch.isfinite(got[bad]).any()
        assert (got[~bad] - want[~bad]).abs().max() < 2e-5
    assert _rel(call.dhidden[~bad.to(DEV)], dH[~bad]) < 1e-2


@pytest.mark.parametrize("lens", [
    (512, 3, 0, 255, 256, 257),       # 256 threads a sequence, up to two tokens a thread
    (513, 3, 0, 1024, 1025),          # 1024 threads
    (900,) + (2,) * 600,              # many short ones and a long one: 256
])
@pytest.mark.parametrize("algo", ["grpo", "gspo"])
def test_loss_of_long_and_short_sequences(fr, lens, algo):
    """The loss kernel's block sizes: loss, clip count and the log-probs' gradient through dhidden for
    sequences around them (loss: float64 sums of float32 log-probs; dhidden: float32 GEMM)."""
    d, V = 16, 40
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    T, S = int(off[-1]), len(lens)
    H, W, y, z, lse, logp, _ = _problem(T, d, V, T, torch.float32)
    old = (logp + 0.2 * torch.randn(T, generator=torch.Generator().manual_seed(7))).float()
    adv = torch.linspace(-1.0, 1.5, S)
    eps = float(np.float32(0.2))
    loss, g, info = oracle.policy_loss(logp.numpy(), old.double().numpy(), None, off,
                                       adv.double().numpy(), algo=algo, eps_low=eps, eps_high=eps)
    dZ = -torch.from_numpy(g)[:, None] * torch.exp(z - lse[:, None])
    dZ[torch.arange(T), y.long()] += torch.from_numpy(g)
    call = fr.policy_loss_fwd_bwd(
        H.to(DEV), W.to(DEV), y.to(DEV), old.to(DEV), torch.from_numpy(off).to(DEV),
        torch.from_numpy(off), adv.to(DEV), algo=algo, need_dW=False)
    torch.cuda.synchronize()
    assert abs(call.loss.item() - loss) <= 1e-5  # (terms of order 1 and of both signs)
    assert int(call.stats[0].item()) == info["clipped_tokens"]
    assert _rel(call.dhidden, dZ @ W.double()) < 1e-5


@pytest.mark.parametrize("V", [16384, 16385])  # 64 vocabulary blocks, 65: 8 slices, 32
@pytest.mark.parametrize("T", [31, 33])        # around a block's 32 tokens
def test_merge_slices(fr, V, T):
    """Log-probs and entropy through both forms of the merge (2e-5: as in test_logits_tiles)."""
    d = 24
    H, W, y, z, lse, logp, old = _problem(T, d, V, V + T, torch.float32)
    lp, ls = fr.token_logprob(H.to(DEV), W.to(DEV), y.to(DEV))
    off = torch.tensor([0, T])
    call = fr.policy_loss_fwd_bwd(
        H.to(DEV), W.to(DEV), y.to(DEV), old.to(DEV), off.to(DEV), off, torch.ones(1, device=DEV),
        need_dW=False, need_entropy=True)
    torch.cuda.synchronize()
    ent = lse - (torch.exp(z - lse[:, None]) * z).sum(1)
    for got, want in ((lp, logp), (call.logp, logp), (ls, lse), (call.lse, lse), (call.entropy, ent)):
        assert (got.double().cpu() - want).abs().max() < 2e-5
