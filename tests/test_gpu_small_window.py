"""Block scores whose launch reduces the window itself, at the edges of that rule, and the selection's early end."""
import numpy as np
import pytest
import torch

from oracle import slim_oracle as so
from tests.helpers import f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slim():
    import paper_2508_06447_amd as slim
    slim.load_library()
    return slim


def rand(shape, dtype, seed):
    return torch.from_numpy(np.random.default_rng(seed).standard_normal(shape).astype(np.float32)).to(dtype)


# 64 KB of Query states is the limit: 8 tokens of 32 heads of 128 in bf16, 4 in float; 1024 elements of the window query; 512 blocks of 8 units for
# the scores from unit keys
@pytest.mark.parametrize("N,block,unit,w,Hq,Hkv,d,dtype", [
    (700, 64, 8, 8, 32, 8, 128, torch.bfloat16), (700, 64, 8, 9, 32, 8, 128, torch.bfloat16), (700, 64, 8, 1, 32, 8, 128, torch.bfloat16),
    (700, 64, 8, 4, 32, 8, 128, torch.float32), (700, 64, 8, 5, 32, 8, 128, torch.float32),
    (300, 16, 8, 32, 4, 2, 64, torch.float32), (45, 16, 16, 7, 6, 2, 32, torch.float32), (130, 128, 3, 5, 28, 4, 128, torch.bfloat16),
    (200, 16, 4, 3, 16, 16, 64, torch.bfloat16), (200, 16, 4, 3, 9, 9, 128, torch.bfloat16), (90, 8, 1, 2, 2, 1, 8, torch.bfloat16),
    (32768, 64, 8, 4, 32, 8, 128, torch.bfloat16), (32769, 64, 8, 4, 32, 8, 128, torch.bfloat16),
])
def test_scores_with_a_small_window(slim, N, block, unit, w, Hq, Hkv, d, dtype):
    print(f"N={N} block={block} unit={unit} w={w} heads={Hq}/{Hkv} d={d} {dtype}", flush=True)
    q, k = rand((w, Hq, d), dtype, N + w), rand((N, Hkv, d), dtype, N)
    want = so.block_scores(f64(q), f64(k), block, unit)
    # a score is the mean product of two vectors of E normal elements, one of them a mean over w and Hq / Hkv: every sum is of at most E terms
    # in float32, whose rounding grows with their root: a few 2^-24 of the largest score
    tol = 16 * 2.0 ** -24 * np.abs(want).max()
    units = slim.slim_unit_keys(k.cuda(), block, unit)
    for name, got in (("keys", slim.slim_score_blocks(q.cuda(), k.cuda(), block, unit)),
                      ("unit keys", slim.slim_score_blocks_from_unit_keys(q.cuda(), units, N, Hkv, block, unit))):
        err = np.abs(f64(got) - want).max()
        print(f"  {name}: max-abs {err:.2e} (bound {tol:.2e})", flush=True)
        assert err <= tol


@pytest.mark.parametrize("nb", [5, 256, 1000, 1024, 1025, 4096])
@pytest.mark.parametrize("kind", ["first digit", "second digit", "last digit", "equal"])
def test_selection_ends_at_any_digit(slim, nb, kind):
    """The digit at which every candidate from the threshold up is taken: the sign and exponent, further ones, the last, or never (ties)."""
    g = np.random.default_rng(nb)
    bits = {"first digit": np.where(np.arange(nb) % 3 == 0, 0x42000000, 0x3f800000), "second digit": 0x3f800000 + (g.permutation(nb) % 64 << 16),
            "last digit": 0x3f800000 + g.permutation(nb), "equal": np.full(nb, 0x3f800000)}[kind]
    scores = bits.astype(np.uint32).view(np.float32)
    for n_keep in sorted({2, max(2, (nb + 2) // 3), nb // 2 + 1, nb - 1}):
        kept = slim.slim_select_topk_blocks(torch.from_numpy(scores.copy()).cuda(), n_keep)
        np.testing.assert_array_equal(kept.cpu().numpy(), so.select_blocks(scores, n_keep))
