"""Prefill attention of few rows (bf16, 32 queries of four heads per workgroup): edges of query and key tiles, groups of three, four, seven and twelve heads, a softmax
reference that has to move, and row counts on both sides of its last one."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slim():
    import paper_2508_06447_amd as slim
    slim.load_library()
    return slim


def attention(q, k, v):
    """out, and what the magnitudes of the values would give: both [n, Hq, d] in float64."""
    n, Hq, d = q.shape
    out, mag = (torch.empty(n, Hq, d, dtype=torch.float64, device=q.device) for _ in range(2))
    above = torch.ones(n, n, dtype=torch.bool, device=q.device).triu(1)
    for h in range(Hq):
        g = h // (Hq // k.shape[1])
        p = torch.softmax((q[:, h].double() @ k[:, g].double().T / math.sqrt(d)).masked_fill(above, -math.inf), -1)
        out[:, h], mag[:, h] = p @ v[:, g].double(), p @ v[:, g].double().abs()
    return out, mag


def close(got, want, mag):
    """One rounding of the output and one of every P to bf16 (8 significant bits: half an ulp is at most 2^-8 of the value, each), and a tenth of them for the exponentials
    and float sums."""
    return bool(((got.double() - want).abs() <= 1.1 * 2.0 ** -8 * (want.abs() + mag)).all())


@pytest.mark.parametrize("heads", [(32, 8), (28, 4), (3, 1), (12, 1)])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 129, 255, 511])
def test_few_row_attention(slim, n, heads):
    print(f"attention {n} rows, heads {heads}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn(n, h, 128, generator=g, device="cuda").bfloat16() for h in (heads[0], heads[1], heads[1]))
    for grow in (0.0, 4.0):                               # 4: logits rise along the keys to some hundred, so that the reference moves again and again
        k_ = (k.float() * (1 + grow * torch.arange(n, device="cuda").view(-1, 1, 1) / n)).bfloat16()
        q_ = (q.float() * (1 + grow)).bfloat16()
        assert close(slim.slim_prefill_attn(q_, k_, v), *attention(q_, k_, v))


def test_few_row_attention_up_to_its_last_row(slim):
    """6 / 2 heads: the last row count of the kernel, and one more."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = cus * 32
    g = torch.Generator(device="cuda").manual_seed(5)
    for rows in (n, n + 1):
        q, k, v = (torch.randn(rows, h, 128, generator=g, device="cuda").bfloat16() for h in (6, 2, 2))
        got = slim.slim_prefill_attn(q, k, v)
        for lo in (0, 2000, rows - 40):                   # a few queries against all keys that they see
            for i in (lo, lo + 33):
                if i >= rows:
                    continue
                for h in (0, 5):
                    p = torch.softmax(k[:i + 1, h // 3].double() @ q[i, h].double() / math.sqrt(128), 0)
                    want, mag = p @ v[:i + 1, h // 3].double(), p @ v[:i + 1, h // 3].double().abs()
                    assert bool(((got[i, h].double() - want).abs() <= 2.0 ** -7 * (want.abs() + mag)).all())
