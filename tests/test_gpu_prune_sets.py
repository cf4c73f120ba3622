"""GPU pruning through the hash sets and both compaction launches, at the edges of their sizes, bit
for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from synth import CONFIGS, make_rollouts, plant_duplicates
from tests._parity import to_dev

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def fr():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2609_36932_amd as m
    return m


@pytest.mark.parametrize("Q, G, lens, V, n", [
    (1024, 4, (1, 12), 40, 1),      # 4096 trajectories: the last size that scans in the fill
    (1366, 3, (0, 12), 40, 2),      # 4098: the scan launch
    (3, 64, (30, 33), 40, 1),       # one full conflict word; ids past one word of bits
    (2, 70, (1, 260), 9, 3),        # two words; trigrams over 9 ids, more keys than a block
    (4, 8, (510, 514), 1 << 19, 1),  # a key per thread and one more; the largest bit set
    (4, 8, (255, 258), (1 << 19) + 1, 1),  # unigrams in the hash set
    (3, 8, (14, 20), 50, 2),        # 13-19 bigrams around the smallest hash set
    (3, 8, (1022, 1028), 90, 2),    # around the last set with four slots a key
    (3, 8, (2046, 2052), 90, 2),    # around the last of 32 KB
    (1366, 3, (508, 518), 700, 2),  # 4098 rollouts of up to 518: blocks of 256
    (1366, 3, (505, 512), 700, 3),  # and of up to 512: blocks of 128
    (4, 8, (1000, 1300), 3, 1),     # at most 3 distinct ids: every insert but three is a repeat
])
@pytest.mark.parametrize("keep", [0.0, 0.5])
def test_prune_sets(fr, Q, G, lens, V, n, keep):
    ro = make_rollouts(CONFIGS[3], Q=Q, len_range=lens, G=(G,), V=V, seed=40 + Q)
    plant_duplicates(ro, p_copy=0.6, p_mutate=0.1, seed=Q)
    ref = oracle.hot_path_step(ro.rewards, ro.group_off, ro.token_ids, ro.traj_tok_off,
                               lmhead=False, ngram_n=n, keep_ratio=keep)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    out = fr.prune(to_dev(ro.token_ids, DEV), to_dev(ro.traj_tok_off, DEV),
                   to_dev(ro.rewards, DEV), to_dev(ro.group_off, DEV), to_dev(ref["class_id"], DEV),
                   to_dev(ref["group_valid"], DEV), V=V, max_group=G,
                   max_len=int(ro.lengths.max()), ngram_n=n, keep_ratio=keep, status=st)
    torch.cuda.synchronize()
    assert st.item() == 0, fr.status_names(st.item())
    nk, tk = out["counts"].cpu().tolist()
    assert np.array_equal(out["keep_mask"].cpu().numpy(), ref["keep_mask"])
    assert np.array_equal(out["mdap_count"].cpu().numpy(), ref["mdap_count"])
    assert nk == len(ref["kept_traj"]) and tk == len(ref["tok_src"])
    assert np.array_equal(out["kept_traj"][:nk].cpu().numpy(), ref["kept_traj"])
    assert np.array_equal(out["kept_tok_off"][:nk + 1].cpu().numpy(), ref["kept_tok_off"])
    assert np.array_equal(out["tok_src"][:tk].cpu().numpy(), ref["tok_src"])


def _run(fr, ro, ref, max_group, st, **kw):
    return fr.prune(to_dev(ro.token_ids, DEV), to_dev(ro.traj_tok_off, DEV),
                    to_dev(ro.rewards, DEV), to_dev(ro.group_off, DEV), to_dev(ref["class_id"], DEV),
                    to_dev(ref["group_valid"], DEV), max_group=max_group, status=st, **kw)


@pytest.mark.parametrize("n", [1, 2])
def test_prune_many_questions_under_the_largest_bounds(fr, n):
    """More questions times max_group than one launch of a block for each slot could hold (2^23
    blocks of 512 threads): groups of 1-3 under max_group = 256 and max_len = 16384."""
    Q = 33000
    ro = make_rollouts(CONFIGS[3], Q=Q, len_range=(1, 4), G=(1, 2, 3), V=6, seed=11)
    plant_duplicates(ro, p_copy=0.5, p_mutate=0.2, seed=12)
    ref = oracle.hot_path_step(ro.rewards, ro.group_off, ro.token_ids, ro.traj_tok_off,
                               lmhead=False, ngram_n=n, keep_ratio=0.0)
    assert 0 < ref["keep_mask"].sum() < ro.N
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    print(f"[prune] Q={Q} N={ro.N} n={n}", flush=True)
    out = _run(fr, ro, ref, 256, st, V=6, max_len=16384, ngram_n=n)
    torch.cuda.synchronize()
    assert st.item() == 0, fr.status_names(st.item())
    assert np.array_equal(out["keep_mask"].cpu().numpy(), ref["keep_mask"])
    assert np.array_equal(out["mdap_count"].cpu().numpy(), ref["mdap_count"])
    assert np.array_equal(out["tok_src"][:len(ref["tok_src"])].cpu().numpy(), ref["tok_src"])


def test_prune_skips_a_question_of_bad_offsets(fr):
    """Questions whose offsets leave [0, N] or are not monotone are flagged and skipped; the others
    are pruned as if alone, also where rollouts belong to no question."""
    ro = make_rollouts(CONFIGS[3], Q=5, len_range=(4, 20), G=(8,), V=12, seed=21)
    plant_duplicates(ro, p_copy=0.6, p_mutate=0.1, seed=22)
    ref = oracle.hot_path_step(ro.rewards, ro.group_off, ro.token_ids, ro.traj_tok_off,
                               lmhead=False, keep_ratio=0.0)
    off = ro.group_off.copy()
    off[2] = ro.N + 5  # question 1 ends, and question 2 begins, past the last rollout
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    out = fr.prune(to_dev(ro.token_ids, DEV), to_dev(ro.traj_tok_off, DEV),
                   to_dev(ro.rewards, DEV), to_dev(off, DEV), to_dev(ref["class_id"], DEV),
                   to_dev(ref["group_valid"], DEV), V=12, max_group=8, max_len=20, status=st)
    torch.cuda.synchronize()
    assert fr.status_names(st.item()) == ["BAD_OFFSETS"]
    keep, count = out["keep_mask"].cpu().numpy(), out["mdap_count"].cpu().numpy()
    assert count.tolist() == [c if q not in (1, 2) else 0 for q, c in enumerate(ref["mdap_count"])]
    for q in (0, 3, 4):
        a, b = ro.group_off[q], ro.group_off[q + 1]
        assert np.array_equal(keep[a:b], ref["keep_mask"][a:b])
