"""float32 projections in tiles of 16 rows, at the edges of tiles, chunks and of the rule that takes them."""
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


# up to 128 tiles of 32 x 32 (32 x 16 for SwiGLU), more than 16 rows and more than 64 features in
@pytest.mark.parametrize("m,n,k", [(16, 40, 80), (17, 33, 65), (31, 1, 256), (32, 4096, 65), (32, 4097, 65), (33, 31, 257), (49, 66, 16 * 43), (100, 96, 300),
                                   (128, 1024, 128), (129, 1024, 128), (512, 256, 64)])
@pytest.mark.parametrize("kind", ["plain", "residual", "bias", "swiglu"])
def test_projection(slim, m, n, k, kind):
    print(f"{kind} {m} x {n} from {k}", flush=True)
    g = np.random.default_rng(m * 7 + n)
    a, w, u = (torch.from_numpy(g.standard_normal(s).astype(np.float32)) for s in ((m, k), (n, k), (n, k)))
    r, b = torch.from_numpy(g.standard_normal((m, n)).astype(np.float32)), torch.from_numpy(g.standard_normal(n).astype(np.float32))
    ref, size = f64(a) @ f64(w).T, np.abs(f64(a)) @ np.abs(f64(w)).T
    tol = k * 2.0 ** -24 * size + 2.0 ** -22                 # k roundings of a sum of such a size, and those of what is added to it
    if kind == "plain":
        got = slim.slim_linear(a.cuda(), w.cuda())
    elif kind == "residual":
        got, ref = slim.slim_linear(a.cuda(), w.cuda(), residual=r.cuda()), ref + f64(r)
    elif kind == "bias":
        got, ref = slim.slim_linear_bias(a.cuda(), w.cuda(), b.cuda()), ref + f64(b)
    else:
        up, up_size = f64(a) @ f64(u).T, np.abs(f64(a)) @ np.abs(f64(u)).T
        silu = ref / (1 + np.exp(-ref))
        got = slim.slim_swiglu_linear(a.cuda(), w.cuda(), u.cuda())
        # |silu'| <= 1.1; a few roundings (2^-21) of the exponential, the quotient and the products
        tol = 1.1 * tol * np.abs(up) + (k * 2.0 ** -24 * up_size) * np.abs(silu) + 2.0 ** -21 * np.abs(silu * up) + 2.0 ** -22
        ref = silu * up
    err = np.abs(f64(got) - ref)
    print(f"  max-abs {err.max():.2e}, largest error / bound {(err / tol).max():.2f}", flush=True)
    assert (err <= tol).all()
