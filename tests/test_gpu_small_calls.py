"""GPU parity of the kernels that small calls take, at the edges of their tiles: against plain
float64 on the same inputs."""
import numpy as np
import pytest
import torch

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
