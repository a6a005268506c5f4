"""GPU parity where a launch rule of the multi-row kernels changes form: the edges of the
scoring kernel's forms (64-row blocks of four waves; 128-row blocks of eight, from d = 120, or
of four waves with the keys in registers, up to d = 112), and the dealing of the statistics tasks to the XCDs on ragged batches (unit counts with and without
a remainder, below and above the rule's line)."""
import pytest

from parity import custom_stage
from test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [2, 32, 33, 63, 64, 65, 127, 129])
def test_narrow_scoring_form(T):
    # Keys one below, at and one past a 128-key chunk, and less than a wave's 32.
    sb = custom_stage(B=4, R=2, H=4, Hkv=2, d=72 if T % 2 else 128, T=[T] * 4,
                      N=[125, 126, 127, 9], seed=100 + T)
    run_and_check(sb, 1.0)


@pytest.mark.parametrize("d,Hkv,N", [(64, 1, 8189), (40, 2, 8190), (128, 2, 8191)])
def test_wide_scoring_form(d, Hkv, N):
    # 4 x 33 x 2 or 4 x 32 x 2 wide workgroups (256 or more); the last chunk full, one short
    # or one key.  (d = 40 and 64: the tall form, twice as many workgroups.)
    sb = custom_stage(B=4, R=2, H=2, Hkv=Hkv, d=d, T=[256] * 4, N=[N] * 4, seed=200 + d)
    run_and_check(sb, 1.0)


@pytest.mark.parametrize("d,H,Hkv,T", [(8, 3, 3, 128), (40, 1, 1, 256), (56, 5, 5, 128),
                                       (64, 4, 2, 256), (72, 4, 4, 128), (80, 6, 3, 128),
                                       (96, 2, 2, 256), (104, 3, 1, 128), (112, 2, 1, 256)])
def test_tall_scoring_form(d, H, Hkv, T):
    # Key counts around a 128-key chunk and a wave's 32, odd and even head counts (the head
    # loop takes two steps at a time).  From d = 64 the form needs 512 tasks by the bound.
    bound = 16384 if d >= 64 and T == 256 else 32766 if d >= 64 else 400
    N = [125, 126, 127, 9, 0, 400]
    sb = custom_stage(B=6, R=2, H=H, Hkv=Hkv, d=d, T=[T] * 6, N=N, seed=500 + d)
    run_and_check(sb, 1.0, ragged=True, row_offsets=False, max_cands=bound)


@pytest.mark.parametrize("d", [48, 96])
def test_tall_scoring_form_uniform(d):
    # 256 tasks: 4 samples x 32 chunks x 2 row blocks; the last chunk ends one key early.
    sb = custom_stage(B=4, R=2, H=3, Hkv=3, d=d, T=[256] * 4, N=[4093] * 4, seed=550 + d)
    run_and_check(sb, 1.0)


@pytest.mark.parametrize("d,T", [(128, 65), (96, 80), (128, 97), (128, 127), (128, 225), (120, 330), (64, 100), (72, 255),
                                 (40, 449)])
def test_row_blocks_not_quite_full(d, T):
    # The 128-row forms with rows past T in the last block: 5 x 28 wide tasks or more.
    sb = custom_stage(B=5, R=2, H=2, Hkv=1, d=d, T=[T] * 5, N=[7000] * 5, seed=700 + T)
    run_and_check(sb, 1.0)


@pytest.mark.parametrize("T", [128, 256])
def test_wide_scoring_form_with_key_offsets(T):
    # Ragged keys, uniform rows: 330 or 333 wide tasks by the bound, decoded from the offsets
    # in a 512-thread workgroup; a full sample, a chunk of one key, less than a wave's keys,
    # and none.
    B = 5 if T == 256 else 9
    N = [8190 if T == 256 else 9300, 30, 0, 255, 4000, 511, 0, 64, 1][:B]
    sb = custom_stage(B=B, R=2, H=2, Hkv=1, d=128, T=[T] * B, N=N, seed=250 + T)
    run_and_check(sb, 1.0, ragged=True, row_offsets=False)


@pytest.mark.parametrize("stage", ["txt", "mut"])
@pytest.mark.parametrize("B,H,Hkv", [(9, 7, 7), (8, 8, 8), (11, 12, 6)])
def test_statistics_units(stage, B, H, Hkv):
    # 63 units, 64, and 66 with two query heads each (at this head dim and length contiguous
    # ranges).
    N = [(37 * b * b + 5) % 300 for b in range(B)]
    N[3] = 0
    T = [n + 2 for n in N] if stage == "mut" else [(53 * b + 2) % 290 + 2 for b in range(B)]
    sb = custom_stage(B=B, R=2, H=H, Hkv=Hkv, d=72, T=T, N=N, seed=300 + B, stage=stage)
    run_and_check(sb, 1.0)


@pytest.mark.parametrize("stage", ["txt", "mut"])
@pytest.mark.parametrize("B,H,Hkv,d,T,longest", [
    (9, 7, 7, 64, 290, 300), (8, 8, 8, 64, 290, 300), (11, 12, 6, 64, 290, 300),   # 63, 64, 66
    (16, 4, 4, 128, 100, 300), (17, 4, 4, 128, 100, 300),      # one workgroup per unit
    (17, 8, 4, 64, 100, 300),                                  # two (query heads)
    (8, 8, 8, 72, 290, 379), (8, 8, 8, 72, 290, 380)])         # 383 and 384 keys
def test_statistics_units_dealt(stage, B, H, Hkv, d, T, longest):
    # Both sides of the lines of the dealing rule; an empty sample among them.
    N = [(37 * b * b + 5) % 300 for b in range(B)]
    N[3], N[5] = 0, longest
    rows = [n + 4 for n in N] if stage == "mut" else [(53 * b + 2) % T + 2 for b in range(B)]
    sb = custom_stage(B=B, R=4, H=H, Hkv=Hkv, d=d, T=rows, N=N, seed=600 + B, stage=stage)
    run_and_check(sb, 1.0)


@pytest.mark.parametrize("stage", ["txt", "mut"])
@pytest.mark.parametrize("B,H,T", [(5, 30, 700), (4, 28, 700), (3, 32, 520), (7, 10, 650),
                                   (8, 7, 2049), (8, 8, 1150)])
def test_statistics_row_blocks(stage, B, H, T):
    # One or two row blocks per workgroup, uniform: even and odd counts of them on both sides of
    # 448 workgroups (450, 336, 240, 210, 504, 320).
    N = [T - 2 if stage == "mut" else 90] * B
    if stage == "mut":
        H = max(1, H // 4)
    sb = custom_stage(B=B, R=2, H=H, Hkv=H, d=40, T=[T] * B, N=N, seed=800 + T, stage=stage)
    run_and_check(sb, 1.0)


@pytest.mark.parametrize("H,d", [(12, 64), (20, 64), (16, 80)])
@pytest.mark.parametrize("B,lo", [(3, 0), (40, 500)])
def test_contiguous_run_one_row_form(H, d, B, lo):
    # (16 x 80 takes the padded form: the other side of the rule.)
    # Key counts around the wave's run of rows and the workgroup's chunk (16 keys for three
    # samples, 128 for forty), an empty sample among them.
    N = [0, 1, 127, 126, 3][:B] + [lo + 13 * b for b in range(B - 5)]
    sb = custom_stage(B=B, R=2, H=H, Hkv=H, d=d, T=[1] * B, N=N, seed=400 + H + B)
    run_and_check(sb, 1.0)


@pytest.mark.parametrize("N", [1, 63, 1024, 12287, 12288, 12289])
@pytest.mark.parametrize("values", [0, 1, 7])
def test_topk_edges(N, values):
    # Around a wave's group, the workgroup and the LDS limit; all scores distinct, all equal,
    # or seven levels.  Whole numbers: compared exactly with a stable sort.
    import numpy as np
    import torch
    from paper_2605_29657_amd import occam
    rng = np.random.default_rng(N + values)
    s = rng.permutation(N).astype(np.float32) + 1 if values == 0 else (
        rng.integers(0, values, N).astype(np.float32))
    p = occam.Problem(1, 1, 1, 64, 1, rows=1, cands=N, dtype="f32")
    ws = occam.workspace(p)
    scores = torch.from_numpy(np.concatenate([[0.5], s]).astype(np.float32)).cuda()
    for K in sorted({0, 1, N // 2, N}):
        kept = torch.zeros(max(N, 1), dtype=torch.int32, device="cuda")
        cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
        offs = torch.zeros(2, dtype=torch.int32, device="cuda")
        occam.select_topk(p, scores, K, kept, cnt, offs, ws)
        want = np.sort(np.argsort(-s, kind="stable")[:K])
        assert int(cnt[0]) == K and offs.tolist() == [0, K]
        assert np.array_equal(kept[:K].cpu().numpy(), want)


def fused_against_unfused(T, N, d, own_lse, seed, H=4, Hkv=2, R=3, ragged=False):
    """The fused prune's scores, thresholds and survivors against the unfused calls', bit for
    bit, on samples of N[b] keys and T[b] rows (uniform unless ragged)."""
    import numpy as np
    import torch
    from paper_2605_29657_amd import occam
    print("case: T=%s N=%s d=%d lse=%s ragged=%s" % (T, N, d, own_lse, ragged), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    i32 = lambda x: torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32,
                                 device="cuda")
    B, keys, total = len(N), sum(N) + R * len(N), sum(N)
    q = torch.randn(sum(T), H, d, generator=gen, device="cuda").bfloat16()
    k = torch.randn(keys, Hkv, d, generator=gen, device="cuda").bfloat16()
    lse = 7.0 + torch.rand(sum(T), H, generator=gen, device="cuda") if own_lse else None
    p = occam.Problem(B, H, Hkv, d, R, rows=T[0], cands=N[0],
                      q_offsets=i32(T) if ragged else None,
                      key_offsets=i32([n + R for n in N]) if ragged else None,
                      max_rows=max(T), max_cands=max(N))
    ws = occam.workspace(p)
    first = torch.zeros(keys, device="cuda")
    occam.score(p, q, k, first, ws, row_lse=lse)
    f, ratios, o = first.cpu().numpy(), [], 0
    for n in N:
        ratios.append(f[o + R:o + R + n] / f[o:o + R].mean())
        o += R + n
    lam = float(np.median(np.concatenate(ratios)))
    got = []
    for fused in (True, False):
        s, tau = torch.zeros(keys, device="cuda"), torch.zeros(B, device="cuda")
        idx = torch.zeros(total, dtype=torch.int32, device="cuda")
        cnt = torch.zeros(B, dtype=torch.int32, device="cuda")
        off = torch.zeros(B + 1, dtype=torch.int32, device="cuda")
        if fused:
            occam.prune(p, q, k, lam, idx, cnt, off, ws, scores=s, tau=tau, row_lse=lse)
        else:
            occam.score(p, q, k, s, ws, row_lse=lse)
            occam.threshold(p, s, lam, occam.REG_MEAN, tau)
            occam.select(p, s, tau, idx, cnt, off, ws)
        got.append([x.cpu().numpy() for x in (s, tau, idx, cnt, off)])
    assert 0 < got[0][3].sum() < total
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("own_lse", [False, True])
@pytest.mark.parametrize("T,N,d,ragged", [
    ([300, 40, 129], [2044, 0, 1633], 64, True),       # 5 blocks: 10235 partials
    ([160, 2, 65], [2727, 0, 9], 64, True),            # 3 blocks: 8190 partials
    ([160, 2, 65], [2728, 0, 9], 64, True),            # 8193
    ([65] * 2, [4093] * 2, 128, False),                # 2 blocks: 8192
    ([65] * 2, [4094] * 2, 128, False),                # 8194
    ([256] * 5, [8189] * 5, 128, False),               # two wide blocks
    ([100] * 2, [9000] * 2, 40, False),                # one block, scores in a launch of their own
])
def test_row_blocks_and_select_placement(T, N, d, ragged, own_lse):
    # Both sides of the lines for where the row blocks are combined and the survivors selected.
    fused_against_unfused(T, N, d, own_lse, sum(N), ragged=ragged)


@pytest.mark.parametrize("T", [64, 65, 128, 300])
def test_caller_normaliser_blocks_combined_in_the_select(T):
    # With a caller normaliser the fused prune combines the row blocks in its select: the
    # unfused calls' scores, thresholds and survivors bit for bit.
    import numpy as np
    import torch
    from paper_2605_29657_amd import occam
    gen = torch.Generator(device="cuda").manual_seed(T)
    B, H, Hkv, d, R, N = 3, 4, 2, 64, 3, 700
    keys = B * (R + N)
    q = torch.randn(B * T, H, d, generator=gen, device="cuda").bfloat16()
    k = torch.randn(keys, Hkv, d, generator=gen, device="cuda").bfloat16()
    lse = 7.0 + torch.rand(B * T, H, generator=gen, device="cuda")
    p = occam.Problem(B, H, Hkv, d, R, rows=T, cands=N)
    ws = occam.workspace(p)
    first = torch.zeros(keys, device="cuda")
    occam.score(p, q, k, first, ws, row_lse=lse)
    f = first.cpu().numpy().reshape(B, R + N)
    lam = float(np.median(f[:, R:] / f[:, :R].mean(1, keepdims=True)))
    got = []
    for fused in (True, False):
        s, tau = torch.zeros(keys, device="cuda"), torch.zeros(B, device="cuda")
        idx = torch.zeros(B * N, dtype=torch.int32, device="cuda")
        cnt = torch.zeros(B, dtype=torch.int32, device="cuda")
        off = torch.zeros(B + 1, dtype=torch.int32, device="cuda")
        if fused:
            occam.prune(p, q, k, lam, idx, cnt, off, ws, scores=s, tau=tau, row_lse=lse)
        else:
            occam.score(p, q, k, s, ws, row_lse=lse)
            occam.threshold(p, s, lam, occam.REG_MEAN, tau)
            occam.select(p, s, tau, idx, cnt, off, ws)
        got.append([x.cpu().numpy() for x in (s, tau, idx, cnt, off)])
    assert 0 < got[0][3].sum() < B * N
    for a, b in zip(*got):
        assert np.array_equal(a, b)
