"""GPU parity of budget matching (Appendix Eq. lambda2_budget_matching_appendix):
occam_match_lambda against the oracle's match_lambda on the same score vectors.

The count decision is taken in float32 on both sides: the expected ratios are the
float32 quotients s(v) / s(r) (register scores are chosen dyadic, so s(r) is exact in
float32 whatever the summation order), and the oracle picks the level from them.  The
returned lambda and the mean kept count must then agree bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_29657_amd import occam

pytestmark = pytest.mark.gpu


def make_scores(N, R, seed, ties=0, zeros=0):
    rng = np.random.default_rng(seed)
    N = np.asarray(N, dtype=np.int64)
    k_off = np.concatenate([[0], np.cumsum(N + R)]).astype(np.int64)
    sc = np.empty(int(k_off[-1]), dtype=np.float32)
    for b in range(len(N)):
        kb = int(k_off[b])
        sc[kb:kb + R] = rng.integers(16, 257, R) / 256.0            # dyadic register scores
        v = np.exp(rng.standard_normal(int(N[b])) * 1.5) * 0.02
        if ties and N[b]:
            v = np.round(v * ties) / ties                            # many equal ratios
        if zeros and N[b]:
            v[rng.integers(0, N[b], zeros)] = 0.0
        sc[kb + R:kb + R + N[b]] = v.astype(np.float32)
    return sc, k_off


def expected(sc, k_off, R, reduce, k_target):
    sr = oracle.register_reference(sc.astype(np.float64), k_off, R, reduce)
    assert np.array_equal(sr, sr.astype(np.float32))                 # exact in float32
    rat = [(sc[k_off[b] + R:k_off[b + 1]] / np.float32(sr[b])).astype(np.float64)
           for b in range(len(k_off) - 1)]
    lam = oracle.match_lambda(rat, np.float64(np.float32(k_target)))
    kept = sum(int(np.count_nonzero(r >= lam)) for r in rat)
    return np.float32(lam), np.float32(kept / (len(k_off) - 1)), rat


def run_case(N, R, k_target, reduce=oracle.REG_MEAN, seed=0, ties=0, zeros=0, ragged=True,
             ws=None):
    print("case: B=%d N=%s R=%d k=%s reduce=%d seed=%d ties=%d zeros=%d" % (
        len(N), list(N)[:6], R, k_target, reduce, seed, ties, zeros), flush=True)
    sc, k_off = make_scores(N, R, seed, ties, zeros)
    B = len(N)
    if ragged:
        p = occam.Problem(B, 16, 16, 64, R, key_offsets=torch.tensor(k_off.astype(np.int32),
                                                                      device="cuda"),
                          max_cands=max(1, int(max(N))))
    else:
        p = occam.Problem(B, 16, 16, 64, R, cands=int(N[0]))
    d_sc = torch.from_numpy(sc).cuda()
    if ws is None:
        ws = occam.workspace(p)
    assert ws.numel() >= occam.workspace_size(p)
    out = torch.full((2,), -7.0, dtype=torch.float32, device="cuda")
    occam.match_lambda(p, d_sc, k_target, out[0:1], ws, mean_kept=out[1:2], reduce=reduce)
    torch.cuda.synchronize()
    got_lam, got_mk = out.cpu().numpy()
    want_lam, want_mk, rat = expected(sc, k_off, R, reduce, k_target)
    assert got_lam.view(np.uint32) == want_lam.view(np.uint32), (got_lam, want_lam)
    assert got_mk == want_mk, (got_mk, want_mk)
    # The float32 lambda keeps exactly the matched count.
    kept = sum(int(np.count_nonzero(r >= np.float64(got_lam))) for r in rat)
    assert np.float32(kept / B) == want_mk
    return got_lam, got_mk


def test_ragged_with_an_empty_sample():
    run_case([300, 0, 577, 1, 64], R=4, k_target=50.0, seed=1)


@pytest.mark.parametrize("k_target", [0.0, 0.4, 1.0, 17.25, 99.5, 250.0, 1e6])
def test_targets_from_none_to_all(k_target):
    run_case([200, 131, 256], R=2, k_target=k_target, seed=2)


@pytest.mark.parametrize("reduce", [oracle.REG_MEAN, oracle.REG_MAX, oracle.REG_SUM])
def test_register_reductions(reduce):
    run_case([576] * 6, R=8 if reduce == oracle.REG_MEAN else 3, k_target=64.0, reduce=reduce,
             seed=3, ragged=False)


def test_many_equal_ratios_and_zeros():
    # Few distinct levels: the matched count is a level, not the target itself.
    lam, mk = run_case([1000, 999, 17], R=1, k_target=333.3, seed=4, ties=64, zeros=40)
    assert lam > 0


def test_half_way_target_takes_the_smaller_count():
    # Two samples, distinct ratios: 2 * 4.25 = 8.5 kept over the batch lies half way
    # between the levels of 8 and 9, and the tie goes to 8 (the larger lambda).
    run_case([40, 40], R=1, k_target=4.25, seed=5)


def test_all_ratios_zero_or_equal():
    run_case([50, 50], R=1, k_target=10.0, seed=6, ties=1)   # ratios in {0, 1/256 multiples}


def test_no_candidates_gives_one():
    lam, mk = run_case([0, 0, 0], R=2, k_target=5.0, seed=7)
    assert lam == 1.0 and mk == 0.0


def test_full_size_batch():
    # 64 samples of 2880 candidates: about 184k ratios through all four radix passes.
    run_case([2880] * 64, R=4, k_target=576.0, seed=8, ragged=False)


def test_many_small_samples():
    # 1000 samples of 0..50 candidates: one chunk each, many workgroups per pass.
    N = np.random.default_rng(9).integers(0, 51, 1000)
    run_case(list(N), R=2, k_target=12.5, seed=9)


def test_repeated_calls_reuse_the_workspace():
    # The selection state lives in the workspace and is cleared by every call.
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    for seed, k, N in ((10, 3.0, [700, 300, 1500]), (11, 40.0, [1500, 2]), (12, 0.0, [5])):
        run_case(N, R=4, k_target=k, seed=seed, ws=ws)


@pytest.mark.parametrize("N", [4095, 4096, 4097, 16384])
def test_samples_of_several_chunks(N):
    # A workgroup takes 4096 ratios: one chunk full, one of a single ratio, four full ones.
    run_case([N] * 3, R=2, k_target=N / 7.0, seed=N, ragged=False)


@pytest.mark.parametrize("ties", [0, 32])
def test_ragged_samples_of_several_chunks(ties):
    # Chunks wholly past a short or empty sample; equal ratios on both sides of a chunk's edge.
    run_case([16384, 0, 17, 4097, 8192, 12289], R=4, k_target=901.5, seed=20 + ties, ties=ties,
             zeros=30 if ties else 0)


def test_candidate_mean_over_several_chunks():
    # Every workgroup forms the mean over the whole sample.  Constant samples: their mean, and
    # with it every ratio, is exact in float32 whatever the order of the sum.
    N, R, level = [9000, 4096, 5], 2, [0.5, 0.25, 2.0]
    k_off = np.concatenate([[0], np.cumsum(np.asarray(N) + R)]).astype(np.int64)
    sc = np.full(int(k_off[-1]), 0.125, dtype=np.float32)
    for b, n in enumerate(N):
        sc[k_off[b] + R:k_off[b] + R + n] = level[b]
        sc[k_off[b] + R] += level[b] / 2                    # one ratio above 1 per sample,
        sc[k_off[b] + R + n - 1] -= level[b] / 2            # one below, the mean kept
    p = occam.Problem(3, 16, 16, 64, R, max_cands=max(N),
                      key_offsets=torch.tensor(k_off.astype(np.int32), device="cuda"))
    ws = occam.workspace(p)
    for target, count in ((1.0, 3), (4000.0, sum(N) - 3), (5000.0, sum(N))):
        out = torch.zeros(2, device="cuda")
        occam.match_lambda(p, torch.from_numpy(sc).cuda(), target, out[0:1], ws,
                           mean_kept=out[1:2], reduce=occam.REF_CAND_MEAN)
        lam, mk = out.cpu().numpy()
        # Levels: 3 ratios of 1.5, all but 3 of at least 1, all; lambda the geometric midpoint.
        want = {3: np.sqrt(1.5), sum(N) - 3: np.sqrt(0.5), sum(N): 0.25}[count]
        assert mk == np.float32(count / 3) and abs(lam - want) < 1e-6, (target, lam, mk)
