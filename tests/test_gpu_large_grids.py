"""GPU calls past the limits of 32 bits: kernels that need more threads than one launch can hold (2^32)
at the tile and block sizes in use, and bf16 rows of more than 2^28 elements; against float64 on the few
distinct rows or entries that they hold."""
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


def _sparse(rows, n, seed, value):
    """bf16 [rows, n], zero but for the same ~400 columns in every row: some of each end and middle"""
    g = torch.Generator(device=DEV).manual_seed(seed)
    cols = torch.unique(torch.cat([torch.arange(72, device=DEV), n - 1 - torch.arange(72, device=DEV),
                                   torch.randint(0, n, (256,), device=DEV, generator=g)]))
    x = torch.zeros((rows, n), dtype=torch.bfloat16, device=DEV)
    part = (value * torch.randn(rows, len(cols), device=DEV, generator=g)).bfloat16()
    x[:, cols] = part
    return x, cols, part


def test_bf16_long_rows(fr):
    """d = 320 M: the eighth row of a load starts past 32 bits of bytes.  The logits' few nonzero terms
    sum to float32 accuracy (2e-5 at values around 1)."""
    d, V, T = 320_000_000, 9, 3
    print(f"[large] bf16 d={d}", flush=True)
    W, cols, wp = _sparse(V, d, 4, 0.05)
    H, hcols, hp = _sparse(T, d, 4, 1.0)
    assert torch.equal(cols, hcols)
    y = torch.tensor([8, 0, 7], dtype=torch.int32, device=DEV)
    lp, ls = fr.token_logprob(H, W, y)
    torch.cuda.synchronize()
    z = hp.double() @ wp.double().T
    lse = torch.logsumexp(z, 1)
    assert (ls.double() - lse).abs().max() < 2e-5
    assert (lp.double() - (z.gather(1, y.long()[:, None])[:, 0] - lse)).abs().max() < 2e-5


def test_bf16_backward_over_long_rows(fr):
    """V = 307 M: the exp-logit rows that dhidden reads, ten of them, start past 32 bits of bytes within
    a load, and dW spans 2^20 vocabulary blocks.  W is zero but for 96 rows, so that the oracle is short.
    1e-2 is the bar of bf16 gradients."""
    d, V, T = 8, 307_000_000, 10
    torch.cuda.empty_cache()  # (what earlier tests of the process left)
    if torch.cuda.mem_get_info()[0] < 220 << 30:
        pytest.skip("needs 190 GB")
    print(f"[large] bf16 V={V}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(5)
    rows = torch.unique(torch.cat([torch.arange(16, device=DEV), V - 1 - torch.arange(16, device=DEV),
                                   torch.randint(0, V, (64,), device=DEV, generator=g)]))
    W = torch.zeros((V, d), dtype=torch.bfloat16, device=DEV)
    wp = torch.randn(len(rows), d, device=DEV, generator=g).bfloat16()
    W[rows] = wp
    H = torch.randn(T, d, device=DEV, generator=g).bfloat16()
    pick = torch.randint(0, len(rows), (T,), device=DEV, generator=g)
    pick[0], pick[T - 1] = 0, len(rows) - 1
    y = rows[pick].int()
    z = H.double() @ wp.double().T
    lse = torch.log((V - len(rows)) + torch.exp(z).sum(1))
    logp = z.gather(1, pick[:, None])[:, 0] - lse
    off = torch.tensor([0, 4, T])
    adv = torch.tensor([1.0, -0.5], device=DEV)
    call = fr.policy_loss_fwd_bwd(H, W, y, logp.float(), off.to(DEV), off, adv)
    torch.cuda.synchronize()
    assert (call.logp.double() - logp).abs().max() < 2e-5
    seq = (torch.arange(T, device=DEV) >= 4).long()
    gt = -adv.double()[seq] / (2.0 * torch.tensor([4.0, 6.0], device=DEV).double()[seq])
    dZ = -gt[:, None] * torch.exp(z - lse[:, None])
    dZ[torch.arange(T, device=DEV), pick] += gt
    dH, dWp = dZ @ wp.double(), dZ.T @ H.double()
    assert (call.dhidden.double() - dH).norm() < 1e-2 * dH.norm()
    assert (call.dW[rows].double() - dWp).norm() < 1e-2 * dWp.norm()
    rest = (-(gt * torch.exp(-lse))[:, None] * H.double()).sum(0)  # every row whose logits are 0
    call.dW[rows] = rest.float()
    for a in range(0, V, 1 << 24):
        err = (call.dW[a:a + (1 << 24)] - rest.float()).abs().max()
        assert err < 1e-2 * rest.abs().max(), (a, float(err))
