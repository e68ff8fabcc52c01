"""Large bf16 projections of one, two and three k-tiles: the generated loops leave before their loop, or enter it once."""
import numpy as np
import pytest
import torch

from tests.helpers import f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slim():
    import paper_2508_06447_amd as slim
    slim.load_library()
    return slim


# More than 2^23 outputs, which is what the few-row tiles take; rows that end in a tile of 256, of 128 and in none of theirs
@pytest.mark.parametrize("m,n", [(16640, 512), (16513, 512), (33001, 256), (8300, 1032)])
@pytest.mark.parametrize("k", [64, 128, 192])
@pytest.mark.parametrize("kind", ["plain", "residual", "bias", "norm", "swiglu"])
def test_projection(slim, m, n, k, kind):
    print(f"{kind} {m} x {n} from {k}", flush=True)
    g = np.random.default_rng(m + n + k)
    a, w, u = (torch.from_numpy(g.standard_normal(s).astype(np.float32)).bfloat16() for s in ((m, k), (n, k), (n, k)))
    r, b = torch.from_numpy(g.standard_normal((m, n)).astype(np.float32)).bfloat16(), torch.from_numpy(g.standard_normal(n).astype(np.float32)).bfloat16()
    ref, size = f64(a) @ f64(w).T, np.abs(f64(a)) @ np.abs(f64(w)).T
    tol = k * 2.0 ** -24 * size                              # k roundings of a float sum of such a size
    if kind == "plain":
        got = slim.slim_linear(a.cuda(), w.cuda())
    elif kind == "residual":
        got, ref = slim.slim_linear(a.cuda(), w.cuda(), residual=r.cuda()), ref + f64(r)
    elif kind == "bias":
        got, ref = slim.slim_linear_bias(a.cuda(), w.cuda(), b.cuda()), ref + f64(b)
    elif kind == "norm":
        rstd = slim.slim_row_rstd(a.cuda(), 1e-5)
        got, s = slim.slim_rmsnorm_linear(a.cuda(), w.cuda(), rstd), f64(rstd)[:, None]
        ref, tol = ref * s, tol * s
    else:
        up, up_size = f64(a) @ f64(u).T, np.abs(f64(a)) @ np.abs(f64(u)).T
        silu = ref / (1 + np.exp(-ref))
        got = slim.slim_swiglu_linear(a.cuda(), w.cuda(), u.cuda())
        # |silu'| <= 1.1; a few roundings (2^-21) of the exponential, the quotient and the products
        tol = 1.1 * tol * np.abs(up) + k * 2.0 ** -24 * up_size * np.abs(silu) + 2.0 ** -21 * np.abs(silu * up)
        ref = silu * up
    # Rounded to bf16 once: 8 significant bits, so half a unit of the last is up to 2^-8 of the value; what is added to the sum, in float.
    tol = tol + 2.0 ** -8 * (np.abs(ref) + tol) + 2.0 ** -21 * np.abs(ref) + 1e-30
    err = np.abs(f64(got) - ref)
    print(f"  max-abs {err.max():.2e}, largest error / bound {(err / tol).max():.2f}", flush=True)
    assert (err <= tol).all()
