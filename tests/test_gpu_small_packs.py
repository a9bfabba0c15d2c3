"""Small packs: the 64 x 64 GEMM tiles give the results of the 128 x 128 ones, the one-stream step those of the step on
several streams, and the fused training head those of the oracle; evaluation in chunks, and inputs too wide for them."""
import numpy as np
import pytest

from oracle.pack import OraclePack
from paper_2607_05380_amd import configs, synth, tabpack
from parity import TOL, check_tensor, compare_member, make_inputs, oracle_cfg, oracle_hparams, to_dev

pytestmark = pytest.mark.gpu

# below, at and above the tile edges (32, 64, 128), and several tiles wide
WIDTHS = (1, 31, 64, 65, 129, 257)


def members(depths):
    return [dict(width=w, dropout=0.1 * (i % 3), lr=2e-3, wd=1e-3, depth=depths[i % len(depths)], muon_lr=2e-2)
            for i, w in enumerate(WIDTHS)]


def state(pk, grads):
    out = []
    for k in range(pk.K):
        parts = [pk.get_params(k), *pk.get_moments(k)] + ([pk.get_grads(k)] if grads else [])
        out += [x for p in parts for W, b in p for x in (W, b)]
    return out


@pytest.mark.parametrize("name,over", [
    ("regression_onehot", dict(B=300, d_in=37, features="normal")),
    ("regression_onehot", dict(B=65, d_in=64, keep_grads=0)),
    ("regression_onehot", dict(B=300, d_in=200, features="normal", optimizer="muon")),
    ("multiclass_lognormal", dict(B=300, d_in=37, precision="fp32")),
    ("binary_small", dict(B=256, L=3, optimizer="muon"))])
def test_mini_tiles_bit_identical(monkeypatch, name, over):
    # an output element is reduced over the full depth in one fixed order and
    # the bias partials over 64 rows in one order, whatever the tile: two
    # steps, an evaluation and a prediction must give the same bits
    cfg = configs.workload(name, K=len(WIDTHS), **over)
    mem = members((cfg["L"], 1, 2))
    Xtr, ytr, Xv, yv, _, idx = make_inputs(cfg, 900, 130)
    X, y, idx_d, Xv, yv = to_dev(Xtr, ytr, idx, Xv, yv)
    runs = []
    for tiles in ("small", "mini"):
        monkeypatch.setenv("TABPACK_GEMM_TILES", tiles)
        monkeypatch.setenv("TABPACK_NS_TILES", tiles)
        pk = tabpack.Pack(cfg, members=mem).bind()
        got = [pk.train_step(X, y, idx_d, s).cpu().numpy() for s in (1, 2)]
        got += [t.cpu().numpy() for t in pk.eval_members(Xv, yv)] + [pk.predict(Xv).cpu().numpy()]
        runs.append(got + state(pk, cfg.get("keep_grads", 1)))
    assert len(runs[0]) == len(runs[1])
    for a, b in zip(*runs):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("name,over", [
    ("regression_onehot", dict(B=300)),
    ("multiclass_lognormal", dict(B=200, d_in=24, L=1)),
    ("binary_small", dict(optimizer="muon", L=3)),
    ("binary_small", dict(emb_lo=8, emb_hi=16, emb_step=4))])
def test_one_stream_step_bit_identical(monkeypatch, name, over):
    # three steps (the second and third with keep words produced by the step
    # before) of a small pack on the caller's stream and split over two
    cfg = configs.workload(name, K=len(WIDTHS), **over)
    mem = [dict(m, d_emb=8 + 4 * (i % 3), sigma=1.0) for i, m in enumerate(members((cfg["L"], 1)))]
    Xtr, ytr, _, _, orders, _ = make_inputs(cfg, 1200, 10)
    X, y = to_dev(Xtr, ytr)
    runs = []
    for streams in ("1", "2"):
        monkeypatch.setenv("TABPACK_STREAMS", streams)
        monkeypatch.setenv("TABPACK_GEMM_TILES", "small")
        pk = tabpack.Pack(cfg, members=mem).bind()
        got = []
        for s in range(3):
            (idx,) = to_dev(synth.batch_indices(orders, s, cfg["B"]))
            got.append(pk.train_step(X, y, idx, s + 1).cpu().numpy())
        runs.append(got + [x for k in range(pk.K) for p in (pk.get_params(k), *pk.get_moments(k), pk.get_grads(k))
                           for part in p for x in (part.values() if isinstance(part, dict) else part)])
    for a, b in zip(*runs):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("d_out", [2, 3, 8, 16])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_fused_head_outputs(precision, d_out):
    # every output count's kernel, a batch that ends inside a 32-row block, and
    # widths of one to several column passes, against the oracle
    cfg = configs.workload("multiclass_lognormal", K=3, L=1, B=45, d_in=12, d_out=d_out, precision=precision)
    mem = [dict(width=w, dropout=0.0, lr=1e-3, wd=1e-3) for w in (7, 256, 530)]
    Xtr, ytr, _, _, _, idx = make_inputs(cfg, 400, 10)
    X, y, idx_d = to_dev(Xtr, ytr, idx)
    pk = tabpack.Pack(cfg, members=mem).bind()
    op = OraclePack(oracle_cfg(cfg), hparams=oracle_hparams(cfg, mem),
                    precision="bf16" if precision == "bf16" else "fp64")
    p0 = [[(W.copy(), b.copy()) for W, b in p] for p in op.params]
    loss = pk.train_step(X, y, idx_d, 1).cpu().numpy()
    check_tensor("loss", loss, op.train_step(Xtr, ytr, idx, 1), TOL[precision])
    for k in range(3):
        compare_member(pk, op, k, p0[k], TOL[precision])


def test_bad_index_of_removed_member_is_flagged():
    cfg = configs.workload("binary_small", K=3)
    Xtr, ytr, _, _, _, idx = make_inputs(cfg, 600, 10)
    idx = idx.copy()
    idx[1, 5] = 600
    X, y, idx_d = to_dev(Xtr, ytr, idx)
    pk = tabpack.Pack(cfg).bind()
    pk.set_active([1, 0, 1])
    pk.train_step(X, y, idx_d, 1)
    assert pk.status() == tabpack.STATUS_IDX_RANGE


def test_few_members_left_of_a_large_pack(monkeypatch):
    # a pack too large for the one-stream step, of which two members stay: one
    # stream with two gradient buffers against two streams
    cfg = configs.workload("regression_onehot", K=40, B=512, L=4, width_lo=300, width_hi=512)
    Xtr, ytr, _, _, orders, _ = make_inputs(cfg, 2000, 10)
    X, y = to_dev(Xtr, ytr)
    runs = []
    for streams in ("1", "2"):
        monkeypatch.setenv("TABPACK_STREAMS", streams)
        pk = tabpack.Pack(cfg).bind()
        (idx,) = to_dev(synth.batch_indices(orders, 0, cfg["B"]))
        got = [pk.train_step(X, y, idx, 1).cpu().numpy()]
        pk.set_active([k in (3, 17) for k in range(40)])
        for s in (1, 2):
            (idx,) = to_dev(synth.batch_indices(orders, s, cfg["B"]))
            got.append(pk.train_step(X, y, idx, s + 1).cpu().numpy()[[3, 17]])
        runs.append(got + [x for k in (0, 3, 17) for p in (pk.get_params(k), *pk.get_moments(k)) for part in p
                           for x in part])
    for a, b in zip(*runs):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("name,over", [
    ("regression_onehot", dict(B=300)),
    ("multiclass_lognormal", dict(B=700, d_in=24, L=2)),
    ("binary_small", dict(B=64, L=3)),
    ("binary_small", dict(emb_lo=8, emb_hi=16, emb_step=4)),
    ("regression_onehot", dict(B=300, d_in=20, features="normal", emb_lo=8, emb_hi=16, emb_step=4))])
def test_chunk_rows_do_not_change_predictions(name, over):
    # an activation row depends on its data row alone, reduced in one order by
    # every tile, so the rows of a short input have the bits they have in a long
    # one; 8,600 rows take a chunk of the largest size and a last one
    cfg = configs.workload(name, K=len(WIDTHS), **over)
    mem = [dict(m, d_emb=8 + 4 * (i % 3), sigma=0.3) for i, m in enumerate(members((cfg["L"], 1, 2)))]
    pk = tabpack.Pack(cfg, members=mem).bind()
    Xtr, ytr, Xv, yv, _, idx = make_inputs(cfg, 900, 8600)
    X, y, idx_d, Xv, yv = to_dev(Xtr, ytr, idx, Xv, yv)
    pk.train_step(X, y, idx_d, 1)
    whole = pk.predict(Xv, ensemble=False).cpu().numpy()
    mean = pk.predict(Xv, ensemble=True).cpu().numpy()
    pred = pk.eval_members(Xv, yv)[0].cpu().numpy()
    for n in (1, 33, 64, 65, 257, 2100, 8191):
        np.testing.assert_array_equal(pk.predict(Xv[:n], ensemble=False).cpu().numpy(), whole[:, :n])
        np.testing.assert_array_equal(pk.predict(Xv[:n], ensemble=True).cpu().numpy(), mean[:n])
        np.testing.assert_array_equal(pk.eval_members(Xv[:n], yv[:n])[0].cpu().numpy(), pred[:, :n])


@pytest.mark.parametrize("name,over", [
    ("regression_onehot", dict(B=300, d_in=8, features="normal")),
    ("regression_onehot", dict(B=257, d_in=37, features="normal")),
    ("multiclass_lognormal", dict(B=512, d_in=96)),
    ("binary_wide", dict(B=65, d_in=200))])
def test_huge_tiles_bit_identical(monkeypatch, name, over):
    # 256 x 256 tiles of 8 waves: column remainders from 32 to 256, depths of one
    # to ten 32-deep steps and ones that end inside a step, partly filled row
    # tiles; the accumulation order is the small tiles', so the bits are too
    cfg = configs.workload(name, K=6, L=3, **{k: v for k, v in over.items()})
    mem = [dict(width=w, dropout=0.1 * (i % 3), lr=2e-3, wd=1e-3, depth=(3, 1, 2)[i % 3])
           for i, w in enumerate((31, 65, 129, 257, 300, 420))]
    Xtr, ytr, Xv, yv, _, idx = make_inputs(cfg, 900, 530)
    X, y, idx_d, Xv, yv = to_dev(Xtr, ytr, idx, Xv, yv)
    runs = []
    for tiles in ("small", "huge"):
        monkeypatch.setenv("TABPACK_TILES_FWD", tiles)
        monkeypatch.setenv("TABPACK_TILES_DX", tiles)
        for bind in (False, True):
            pk = tabpack.Pack(cfg, members=mem).bind()
            if bind:
                pk.bind_data(X)
            got = [pk.train_step(X, y, idx_d, s).cpu().numpy() for s in (1, 2)]
            got += [t.cpu().numpy() for t in pk.eval_members(Xv, yv)] + [pk.predict(Xv).cpu().numpy()]
            runs.append(got + state(pk, cfg.get("keep_grads", 1)))
    for i in (0, 1):
        assert len(runs[i]) == len(runs[i + 2])
        for a, b in zip(runs[i], runs[i + 2]):
            np.testing.assert_array_equal(a, b)


def test_wide_inputs_predict_the_same_in_chunks():
    # 8,200 rows of 66,000 fp32 features are 2.02 GiB: chunks must end below the
    # loaders' 32-bit offsets.  The last rows of a long input are those of a
    # short one, and a block of rows agrees with the oracle's layer in fp64.
    import torch
    d_in, N = 66_000, 8_200
    cfg = configs.workload("regression_onehot", K=2, B=256, L=1, d_in=d_in, precision="fp32")
    pk = tabpack.Pack(cfg, members=[dict(width=w, dropout=0.0, lr=1e-3, wd=1e-3) for w in (16, 33)]).bind()
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn(N, d_in, device="cuda", generator=g)
    whole = pk.predict(X).cpu().numpy()
    for r0, r1 in ((0, 40), (4_050, 4_110), (8_100, 8_200)):
        np.testing.assert_array_equal(pk.predict(X[r0:r1].contiguous()).cpu().numpy(), whole[:, r0:r1])
    for k in range(2):
        (W1, b1), (W2, b2) = [(W.astype(np.float64), b.astype(np.float64)) for W, b in pk.get_params(k)]
        z = np.maximum(X[8_135:].cpu().numpy().astype(np.float64) @ W1.T + b1, 0.0) @ W2.T + b2
        # 66,000 fp32 products with weights of at most 66,000^-1/2 and normal
        # features: rounding of about 66,000^1/2 2^-24 per activation of size 0.6
        assert np.abs(whole[k, 8_135:] - z).max() < 1e-4


@pytest.mark.parametrize("rows", [1, 33, 200])
def test_debug_activation_past_a_short_input_is_zero(rows):
    # the rows a short evaluation does not compute hold the step's activations
    # in the workspace; the hook must not return them
    cfg = configs.workload("regression_onehot", K=3, B=300, d_in=24, features="normal")
    mem = [dict(width=w, dropout=0.0, lr=1e-3, wd=1e-3) for w in (40, 129, 70)]
    Xtr, ytr, Xv, yv, _, idx = make_inputs(cfg, 900, 300)
    X, y, idx_d, Xv = to_dev(Xtr, ytr, idx, Xv)
    pk = tabpack.Pack(cfg, members=mem).bind()
    pk.predict(Xv)
    full = {(l, k): pk.debug_activation(l, k) for l in (1, 2, 3) for k in range(3)}
    pk.train_step(X, y, idx_d, 1)
    fresh = tabpack.Pack(cfg, members=mem).bind()
    for p in (pk, fresh):
        p.predict(Xv[:rows].contiguous())
        for l in (1, 2, 3):
            for k in range(3):
                H = p.debug_activation(l, k)
                assert not H[rows:].any()
                if p is fresh:
                    np.testing.assert_array_equal(H[:rows], full[l, k][:rows])
    pk.set_active([1, 0, 1])
    pk.predict(Xv)
    assert not pk.debug_activation(1, 1).any() and pk.debug_activation(1, 2).any()


def test_batch_wider_than_an_operand():
    # a gathered batch of 600 x 2^20 fp32 features passes 2 GiB: the step is
    # refused, and evaluation takes the 511 rows of a chunk below the limit
    import torch
    cfg = configs.workload("regression_onehot", K=1, B=600, L=1, d_in=1 << 20, precision="fp32")
    pk = tabpack.Pack(cfg, members=[dict(width=9, dropout=0.0, lr=1e-3, wd=1e-3)]).bind()
    g = torch.Generator(device="cuda").manual_seed(5)
    X = torch.randn(600, 1 << 20, device="cuda", generator=g)
    y, idx = torch.zeros(600, device="cuda"), torch.zeros(1, 600, dtype=torch.int32, device="cuda")
    with pytest.raises(tabpack.PackError, match="operand limit"):
        pk.train_step(X, y, idx, 1)
    whole = pk.predict(X).cpu().numpy()
    for r0, r1 in ((0, 30), (500, 530), (570, 600)):
        np.testing.assert_array_equal(pk.predict(X[r0:r1].contiguous()).cpu().numpy(), whole[:, r0:r1])
    assert np.isfinite(whole).all() and np.unique(whole).size > 590
