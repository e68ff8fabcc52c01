"""Row counts at which a projection changes its kernel or its split, and what the first pass over the rows leaves behind."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import slim_oracle as so
from paper_2508_06447_amd import inputs
from tests.helpers import assert_residual_close, f64, oracle_shape, oracle_weights
from tests.test_gpu_layer import check_layer, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slim():
    import paper_2508_06447_amd as slim
    slim.load_library()
    return slim


@pytest.mark.parametrize("seq,hidden,ffn", [(2048, 4096, 8192), (2049, 4096, 8256), (2500, 3584, 8256)])   # 2 splits of 128 tiles, 3 of 144 and 140
def test_split_down_projection(slim, seq, hidden, ffn):
    print(f"down projection {seq} {hidden} {ffn}", flush=True)
    wl = inputs.scaled(inputs.WORKLOADS["cfg2"], seq=seq, hidden=hidden, n_q_heads=1, n_kv_heads=1, ffn=ffn, keep_ratio=1.0, planted=4)
    x, w, pos = inputs.hidden_states(wl), inputs.layer_weights(wl), inputs.positions(wl)
    z = run_gpu(slim, wl, x, w, pos, wl.n_blocks, fold=True)["x"]
    y = run_gpu(slim, wl, x, dict(w, w_down=torch.zeros_like(w["w_down"])), pos, wl.n_blocks, fold=True)["x"]
    rows = torch.tensor([0, 255, 256, 1023, 1792, seq - 2, seq - 1], device="cuda")
    want = so.ffn_residual(oracle_shape(wl), oracle_weights(w, np.float64), f64(y[rows]))
    assert_residual_close(z[rows], want, [want], f"down projection seq {seq} hidden {hidden} ffn {ffn}")


@pytest.mark.parametrize("m,n", [(1664, 4096), (1665, 4096), (2047, 4096), (1537, 4104), (1793, 3584), (2304, 3584)])
def test_projections_of_nearly_a_round(slim, m, n, k=320):
    """Products of bf16 numbers are exact in float and sums of 320 of them within 320 * 2^-24 of sum |a w|: the result is the exact one rounded to bf16."""
    print(f"projection {m} x {n} from {k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + n)
    a, w, r = (torch.randn(*s, generator=g, device="cuda").bfloat16() for s in ((m, k), (n, k), (m, n)))
    b = r[0].contiguous()
    prod, mag = a.double() @ w.double().T, a.double().abs() @ w.double().abs().T
    for want, got in ((prod, slim.slim_linear(a, w)), (prod + r.double(), slim.slim_linear(a, w, residual=r)), (prod + b.double(), slim.slim_linear_bias(a, w, b))):
        assert bool(((got.double() - want).abs() <= 2.0 ** -8 * want.abs() + 328 * 2.0 ** -24 * (mag + 8)).all())


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("seq,with_pos", [(1, True), (65, False), (259, True)])
def test_layer_that_drops_nothing_returns_blocks_and_positions(slim, seq, with_pos, fold):
    wl = inputs.scaled(inputs.WORKLOADS["cfg2"], seq=seq, hidden=128, n_q_heads=2, n_kv_heads=1, ffn=128, keep_ratio=1.0, planted=0)
    x, w = inputs.hidden_states(wl), inputs.layer_weights(wl)
    pos = torch.arange(seq, dtype=torch.int32) * 3 + 7 if with_pos else None
    res = run_gpu(slim, wl, x, w, pos, wl.n_blocks, fold=fold)
    assert torch.equal(res["kept"].cpu(), torch.arange(wl.n_blocks, dtype=torch.int32))
    assert torch.equal(res["pos"].cpu(), pos if with_pos else torch.arange(seq, dtype=torch.int32))


@pytest.mark.parametrize("nb,flags", [(nb, flags) for nb in (2, 3, 33, 63, 64, 65) for flags in (0, 1, 2, 3) if (nb, flags) != (2, 3)])
def test_layer_keeps_the_blocks_that_the_selection_keeps(slim, nb, flags):
    """Of up to 64 blocks a small compaction selects for itself (of 8 rows and 3 workgroups here, so that 63 of 64 kept are a small one): the same blocks and order as
    slim_select_topk_blocks on the layer's scores, whatever is forced, with distinct scores, many equal ones (a prompt that repeats) and scores that are not a number.  (Both forced of 2
    blocks leaves nothing to select.)"""
    wl = inputs.scaled(inputs.WORKLOADS["cfg1"], seq=nb * 8, planted=0)
    x, w = inputs.hidden_states(wl), {k: v.cuda() for k, v in inputs.layer_weights(wl).items()}
    shape = slim.make_shape(wl.hidden, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.ffn, 8, wl.unit, wl.window, x.dtype, wl.rope_theta, wl.rms_eps, flags)
    forced = bin(flags).count("1")
    alike = torch.zeros(nb * 8, dtype=torch.int32, device="cuda")                          # no rotation: equal rows have equal keys
    spread = 3 * torch.arange(nb * 8, dtype=torch.int32, device="cuda") + 5
    odd = x.clone()
    odd[8:16] = float("nan")
    counts = [n for n in sorted({max(1, forced), nb // 2 + 1, nb - 1}) if forced <= n < nb]
    assert counts
    for rows, pos in ((x, spread), (x[:8].repeat(nb, 1), alike), (odd, spread)):
        for n_keep in counts:
            res = slim.slim_pruned_layer(shape, w, rows.cuda(), pos, n_keep)
            want = slim.slim_select_topk_blocks(res["scores"], n_keep, flags)
            assert torch.equal(res["kept"], want), (nb, n_keep, flags)
            assert torch.equal(res["pos"], pos.view(nb, 8)[want.long()].flatten()), (nb, n_keep, flags)


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("seq,keep", [(1, 1.0), (64, 1.0), (65, 1.0), (128, 1.0), (256, 1.0), (257, 1.0), (1024, 1.0), (1025, 1.0), (600, 0.5)])
def test_split_output_projection(slim, seq, keep, fold):
    """4, 2, none, 2 and none again at the edges of their row counts and behind a pruning, against the oracle; and in a workspace of exactly the size asked for, whatever it holds."""
    print(f"output projection seq {seq} keep {keep} fold {fold}", flush=True)
    wl = inputs.scaled(inputs.WORKLOADS["cfg2"], seq=seq, keep_ratio=keep, hidden=2048, n_q_heads=16, n_kv_heads=4, ffn=256, planted=max(1, seq // 50))
    check_layer(slim, wl, np.float64, rows_count=64, label=f"output projection {seq} {keep} {fold}", fold=fold)
    x, w = inputs.hidden_states(wl).cuda(), {k: v.cuda() for k, v in inputs.layer_weights(wl).items() if not (fold and k.startswith("g_"))}
    shape = slim.make_shape(wl.hidden, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.ffn, wl.block, wl.unit, wl.window, x.dtype, wl.rope_theta, wl.rms_eps)
    size = slim.pruned_layer_workspace_bytes(shape, seq, wl.n_keep)
    buf, seen = torch.empty(size + 4096, dtype=torch.uint8, device="cuda"), []
    for fill in (0, 255):
        buf.fill_(fill)
        seen.append(slim.slim_pruned_layer(shape, w, x, None, wl.n_keep, workspace=buf[:size])["x"].clone())
        assert (buf[size:] == fill).all()
    assert torch.equal(*seen)


@pytest.mark.parametrize("seq", [64, 300])
def test_gains_that_are_not_aligned(slim, seq):
    """The pass that finishes a split output projection reads the gain in 16 bytes: one that is not aligned takes the projection and the norm as two launches."""
    print(f"gains not aligned, seq {seq}", flush=True)
    wl = inputs.scaled(inputs.WORKLOADS["cfg2"], seq=seq, keep_ratio=1.0, hidden=2048, n_q_heads=16, n_kv_heads=4, ffn=256, planted=max(1, seq // 50))
    g = torch.Generator(device="cuda").manual_seed(seq)
    gains = [(1 + 0.1 * torch.randn(wl.hidden + 1, generator=g, device="cuda")).bfloat16()[1:] for _ in range(2)]
    assert all(t.data_ptr() % 16 for t in gains)
    check_layer(slim, wl, np.float64, rows_count=64, label=f"gains not aligned {seq}", gains=gains)


@pytest.mark.parametrize("residual", [False, True])
def test_output_rows_that_lie_far_apart(slim, residual, m=64, n=54016, k=256, ldo=1 << 23):
    """Nearly a round of tiles whose rows are 2^23 elements apart (1 GB between first and last), against the same product in rows of n."""
    print(f"projection {m} x {n} from {k}, row stride {ldo}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    a, w, r = (torch.randn(*s, generator=g, device="cuda").bfloat16() for s in ((m, k), (n, k), (m, n)))
    far = torch.empty((m - 1) * ldo + n, dtype=torch.bfloat16, device="cuda").as_strided((m, n), (ldo, 1))
    far.copy_(r)                                          # (the residual is taken from the place that the result goes to)
    lib, p = slim.load_library(), lambda t: ctypes.c_void_p(t.data_ptr())
    rc = lib.slim_linear(p(a), k, p(w), p(far) if residual else None, m, n, k, ldo, 1, p(far), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, lib.slim_status_string(rc)
    prod, mag = a.double() @ w.double().T, a.double().abs() @ w.double().abs().T
    want = prod + r.double() if residual else prod
    assert bool(((far.double() - want).abs() <= 2.0 ** -8 * want.abs() + (k + 8) * 2.0 ** -24 * (mag + 8)).all())
