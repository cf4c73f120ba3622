"""GPU calls whose kernels need more threads than one launch can hold (2^32) at the tile and block
sizes in use, against float64 on the few distinct rows that they gather."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def fr():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2609_36932_amd as m
    yield m
    torch.cuda.empty_cache()


def _rows(R, T):
    """row of token t: 0, 1, .., R - 1, 0, .. and the last rows once more at the end"""
    return (torch.arange(T, dtype=torch.int64, device=DEV) * 7 % R).int()


def test_float32_logits_tiles(fr):
    """8196 vocabulary blocks x 1024 columns of 64 tokens: 2^23 + 4096 blocks of 512 threads.  2e-5:
    float32 sums of 8 products and of exps around 1."""
    T, R, d, V = 65536, 64, 8, (1 << 21) + 900
    g = torch.Generator(device=DEV).manual_seed(1)
    H = torch.randn(R, d, device=DEV, generator=g)
    W = torch.randn(V, d, device=DEV, generator=g) / d ** 0.5
    y = torch.randint(0, V, (R,), device=DEV, dtype=torch.int32, generator=g)
    rows = _rows(R, T)
    print(f"[large] float32 logits T={T} V={V}", flush=True)
    lp, ls = fr.token_logprob(H, W, y, row_index=rows)
    torch.cuda.synchronize()
    z = H.double() @ W.double().T
    lse = torch.logsumexp(z, 1)
    logp = z.gather(1, y.long()[:, None])[:, 0] - lse
    assert (ls.double() - lse[rows.long()]).abs().max() < 2e-5
    assert (lp.double() - logp[rows.long()]).abs().max() < 2e-5


def test_merge_of_a_large_slab(fr):
    """One slab of 2^27 + 2^13 tokens (loss alone, no gradient): 2^22 + 2^8 merge blocks of 1024
    threads.  Log-probs to float32 sums of a few terms (2e-5)."""
    S, L, R, d, V = 128, (1 << 20) + 64, 61, 8, 40
    T = S * L
    g = torch.Generator(device=DEV).manual_seed(2)
    H = torch.randn(R, d, device=DEV, generator=g)
    W = torch.randn(V, d, device=DEV, generator=g) / d ** 0.5
    y = torch.randint(0, V, (R,), device=DEV, dtype=torch.int32, generator=g)
    z = H.double() @ W.double().T
    lse = torch.logsumexp(z, 1)
    logp = z.gather(1, y.long()[:, None])[:, 0] - lse
    old = (logp + 0.02 * torch.randn(R, device=DEV, generator=g)).float()
    rows = _rows(R, T)
    off = torch.arange(S + 1, dtype=torch.int64) * L
    adv = torch.linspace(-1.0, 1.5, S, device=DEV)
    print(f"[large] merge T={T}", flush=True)
    call = fr.policy_loss_fwd_bwd(H, W, y, old, off.to(DEV), off, adv, row_index=rows, T=T,
                                  need_dhidden=False, need_dW=False, slab_tokens=T)
    assert len(call.slab_plan()[0]) == 2
    torch.cuda.synchronize()
    for name, got, want in (("lse", call.lse, lse), ("logp", call.logp, logp)):
        for a in range(0, T, 1 << 25):
            b = min(T, a + (1 << 25))
            err = (got[a:b] - want.float()[rows[a:b].long()]).abs().max()
            assert err < 2e-5, (name, a, float(err))


def test_float32_dW_of_long_rows(fr):
    """Hidden rows of 2^20 elements, 16416 tokens: the scaled rows are 2^32 + 2^23 pieces of 16 bytes,
    and each of them reaches dW.  1e-3: a logit sums 2^20 float32 products of which the partial sums
    are around 1 (2^20 roundings of 2^-25, as a random walk 3e-5), and exp turns that into a relative
    error."""
    T, R, d, V = 16416, 32, 1 << 20, 8
    g = torch.Generator(device=DEV).manual_seed(3)
    H = torch.randn(R, d, device=DEV, generator=g)
    W = torch.randn(V, d, device=DEV, generator=g) / d ** 0.5
    y = torch.randint(0, V, (R,), device=DEV, dtype=torch.int32, generator=g)
    z = H.double() @ W.double().T
    lse = torch.logsumexp(z, 1)
    logp = z.gather(1, y.long()[:, None])[:, 0] - lse
    rows = _rows(R, T)
    off = torch.tensor([0, T // 2, T])
    adv = torch.tensor([1.0, -0.5], device=DEV)
    print(f"[large] float32 dW T={T} d={d}", flush=True)
    call = fr.policy_loss_fwd_bwd(H, W, y, logp.float(), off.to(DEV), off, adv, row_index=rows, T=T,
                                  need_dhidden=False)
    torch.cuda.synchronize()
    # old = current: every ratio is 1 (inside the clip range), g_t = -A / (2 L)
    gt = torch.where(torch.arange(T, device=DEV) < T // 2, adv[0], adv[1]).double() * (-1.0 / T)
    gr = torch.zeros(R, dtype=torch.float64, device=DEV).index_add_(0, rows.long(), gt)
    dZ = -gr[:, None] * torch.exp(z - lse[:, None])
    dZ[torch.arange(R, device=DEV), y.long()] += gr
    for a in range(0, d, 1 << 17):
        want = dZ.T @ H[:, a:a + (1 << 17)].double()
        assert (call.dW[:, a:a + (1 << 17)].double() - want).norm() < 1e-3 * want.norm(), a
