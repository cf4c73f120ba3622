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
