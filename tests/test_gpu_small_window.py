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


# The edges of csrc/window_plan.h: 64 (token, head of the group) pairs, 1024 elements of the window query, 16 MB of windows in a launch (8 MB from 33 pairs on), 4096
# waves at once, windows of half of a workgroup's keys, and workgroups that get more waves than units
@pytest.mark.parametrize("N,block,unit,w,Hq,Hkv,d,dtype", [
    (700, 64, 8, 8, 32, 8, 128, torch.bfloat16), (700, 64, 8, 9, 32, 8, 128, torch.bfloat16), (700, 64, 8, 1, 32, 8, 128, torch.bfloat16),
    (700, 64, 8, 4, 32, 8, 128, torch.float32), (700, 64, 8, 5, 32, 8, 128, torch.float32),
    (300, 16, 8, 32, 4, 2, 64, torch.float32), (45, 16, 16, 7, 6, 2, 32, torch.float32), (130, 128, 3, 5, 28, 4, 128, torch.bfloat16),
    (200, 16, 4, 3, 16, 16, 64, torch.bfloat16), (200, 16, 4, 3, 9, 9, 128, torch.bfloat16), (90, 8, 1, 2, 2, 1, 8, torch.bfloat16),
    (32768, 64, 8, 4, 32, 8, 128, torch.bfloat16), (32769, 64, 8, 4, 32, 8, 128, torch.bfloat16),
    (700, 64, 8, 16, 32, 8, 128, torch.bfloat16), (700, 64, 8, 17, 32, 8, 128, torch.bfloat16), (300, 16, 16, 4, 32, 8, 128, torch.bfloat16),
    (300, 64, 64, 2, 32, 8, 128, torch.float32), (4096, 8, 8, 4, 32, 8, 128, torch.bfloat16), (4104, 8, 8, 4, 32, 8, 128, torch.bfloat16),
    (600, 16, 8, 32, 4, 2, 64, torch.float32), (500, 20, 7, 3, 33, 3, 8, torch.float32), (100, 16, 4, 64, 1, 1, 8, torch.bfloat16),
    (16384, 32, 8, 8, 32, 8, 128, torch.bfloat16), (65536, 64, 8, 8, 32, 8, 128, torch.bfloat16), (40000, 128, 8, 2, 32, 1, 128, torch.float32),
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


@pytest.mark.parametrize("w,Hq,Hkv,d", [(32, 4, 2, 64), (32, 8, 1, 64), (8, 32, 1, 128), (2, 32, 1, 128), (32, 64, 1, 8), (16, 4, 1, 128), (5, 33, 3, 8)])
def test_float32_window_query_of_a_scoring_launch(slim, w, Hq, Hkv, d):
    """Keys of a block that are all one unit vector make the block's score an element of the window query, with no rounding but the query's own.  Its relative
    rms error against that of slim_window_query: no larger, with 8 % for the sample (over 2000 elements the rms of either is known to about 2 %)."""
    E = Hkv * d
    keys = torch.zeros(E, 64, E)
    keys[torch.arange(E), :, torch.arange(E)] = 1.0
    keys = keys.reshape(E * 64, Hkv, d).cuda()
    units = slim.slim_unit_keys(keys, 64, 8)
    err, n = {"keys": 0.0, "unit keys": 0.0, "own launch": 0.0}, max(20, 2000 // E)
    for seed in range(n):
        q = rand((w, Hq, d), torch.float32, seed)
        want = f64(q).reshape(w, Hkv, Hq // Hkv, d).sum((0, 2)).ravel() / (w * Hq)
        for name, got in (("keys", slim.slim_score_blocks(q.cuda(), keys, 64, 8)),
                          ("unit keys", slim.slim_score_blocks_from_unit_keys(q.cuda(), units, E * 64, Hkv, 64, 8)),
                          ("own launch", slim.slim_window_query(q.cuda(), Hkv))):
            err[name] += ((f64(got) - want) ** 2).sum() / (want ** 2).sum() / n
    rms = {k: v ** 0.5 for k, v in err.items()}
    print(f"   window {w}, heads {Hq}/{Hkv} of {d}: " + ", ".join(f"{k} {v:.3e}" for k, v in rms.items()), flush=True)
    assert max(rms["keys"], rms["unit keys"]) <= 1.08 * rms["own launch"]


@pytest.mark.parametrize("nb", [5, 256, 1000, 1024, 1025, 4096])
@pytest.mark.parametrize("kind", ["first digit", "second digit", "last digit", "equal"])
def test_selection_of_scores_that_differ_in_one_digit(slim, nb, kind):
    """Scores that differ in the sign and exponent, in a further digit, in the last, or not at all, at kept counts that end the search anywhere."""
    g = np.random.default_rng(nb)
    bits = {"first digit": np.where(np.arange(nb) % 3 == 0, 0x42000000, 0x3f800000), "second digit": 0x3f800000 + (g.permutation(nb) % 64 << 16),
            "last digit": 0x3f800000 + g.permutation(nb), "equal": np.full(nb, 0x3f800000)}[kind]
    scores = bits.astype(np.uint32).view(np.float32)
    for n_keep in sorted({2, max(2, (nb + 2) // 3), nb // 2 + 1, nb - 1}):
        kept = slim.slim_select_topk_blocks(torch.from_numpy(scores.copy()).cuda(), n_keep)
        np.testing.assert_array_equal(kept.cpu().numpy(), so.select_blocks(scores, n_keep))


def last_digit_of_the_search(keys, take):
    """Radix selection, eight bits at a time from the top: the digit at whose threshold every remaining candidate is taken; None: ties are left."""
    for p in range(4):
        digit = keys >> np.uint32(24 - 8 * p) & np.uint32(255)
        count = np.bincount(digit, minlength=256)[::-1].cumsum()[::-1]       # candidates with this digit or a larger one
        threshold = int(np.nonzero(count >= take)[0].max())
        if count[threshold] == take:
            return p
        take -= count[threshold + 1] if threshold < 255 else 0
        keys = keys[digit == threshold]
    return None


@pytest.mark.parametrize("flags", [0, 1, 2, 3])
@pytest.mark.parametrize("digit", [0, 1, 2, 3])
@pytest.mark.parametrize("nb", [5, 64, 65, 256, 257, 1000, 1024, 1025, 4096])
def test_selection_ends_at_a_digit(slim, nb, digit, flags):
    """A third of the blocks are above the others by the given digit, with anything in the digits below it: as many kept blocks end the search there; one fewer
    and one more do not."""
    g = np.random.default_rng(4 * nb + digit)
    forced = sorted({0} if flags & slim.FORCE_FIRST else set()) + ([nb - 1] if flags & slim.FORCE_LAST else [])
    free = np.setdiff1d(np.arange(nb), forced)
    high = g.choice(free, len(free) // 3 + 1, replace=False)
    shift = 24 - 8 * digit
    keys = np.full(nb, 0xbf8a9b00 if digit else 0, np.uint32) >> np.uint32(shift + 8) << np.uint32(shift + 8) if digit else np.zeros(nb, np.uint32)
    low_digit, high_digit = (0xbe, 0xc1) if digit == 0 else (0x21, 0x95)                # (a finite float in any case)
    keys |= np.uint32(low_digit << shift)
    keys[high] += np.uint32(high_digit - low_digit << shift)
    keys |= (g.integers(0, 1 << shift, nb) if shift else np.zeros(nb)).astype(np.uint32)
    scores = (keys & np.uint32(0x7fffffff)).view(np.float32)                             # keys of positive scores: their bits with the sign bit set
    assert np.isfinite(scores).all()
    ends = {take: last_digit_of_the_search(keys[free], take) for take in (len(high) - 1, len(high), len(high) + 1) if 0 < take < len(free)}
    assert ends[len(high)] == digit and all(e != digit or digit == 3 for t, e in ends.items() if t != len(high)), ends
    for take in ends:
        kept = slim.slim_select_topk_blocks(torch.from_numpy(scores.copy()).cuda(), take + len(forced), flags)
        np.testing.assert_array_equal(kept.cpu().numpy(), so.select_blocks(scores, take + len(forced), bool(flags & slim.FORCE_FIRST), bool(flags & slim.FORCE_LAST)))
