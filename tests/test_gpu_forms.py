"""GPU parity where a launch rule of the multi-row kernels changes form: the edges of the
scoring kernel's two forms (64-row blocks of four waves; 128-row blocks of eight), and the
dealing of the statistics tasks to the XCDs on ragged batches (unit counts with and without
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
    # or one key.
    sb = custom_stage(B=4, R=2, H=2, Hkv=Hkv, d=d, T=[256] * 4, N=[N] * 4, seed=200 + d)
    run_and_check(sb, 1.0)


@pytest.mark.parametrize("stage", ["txt", "mut"])
@pytest.mark.parametrize("B,H,Hkv", [(9, 7, 7), (8, 8, 8), (11, 12, 6)])
def test_statistics_units(stage, B, H, Hkv):
    # 63 units (contiguous ranges), 64, and 66 with two query heads each.
    N = [(37 * b * b + 5) % 300 for b in range(B)]
    N[3] = 0
    T = [n + 2 for n in N] if stage == "mut" else [(53 * b + 2) % 290 + 2 for b in range(B)]
    sb = custom_stage(B=B, R=2, H=H, Hkv=Hkv, d=72, T=T, N=N, seed=300 + B, stage=stage)
    run_and_check(sb, 1.0)
