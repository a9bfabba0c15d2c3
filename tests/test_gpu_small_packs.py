"""Small launches: the 64 x 64 GEMM tiles give the results of the 128 x 128 ones."""
import numpy as np
import pytest

from paper_2607_05380_amd import configs, tabpack
from parity import make_inputs, to_dev

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
