"""The planner's limits, on the host: GEMM operands stay inside the loaders' 32-bit offsets and the tile table holds
every launch.  No GPU and no parameters."""
import pytest

from paper_2607_05380_amd import configs, tabpack

OPERAND_MAX = (1 << 31) - 16  # a GEMM loader's offsets: bytes of an operand below 2 GiB, less one 16-byte vector


def members(K, w, **hp):
    return [dict(dict(width=w, dropout=0.1, lr=1e-3, wd=1e-3, muon_lr=1e-2, d_emb=16, sigma=0.3), **hp)] * K


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("d_in", [8, 4_000, 65_536, 65_537, 66_000, 131_072, 131_080, 262_144, 1 << 20])
@pytest.mark.parametrize("K,width,B", [(1, 32, 1), (4, 128, 256), (1, 128, 2048), (40, 480, 700), (1, 128, 65_536)])
def test_evaluation_operands_below_the_loaders_limit(K, width, B, d_in, precision):
    # rows past the limit read as zeros or as other rows: wrong predictions
    cfg = configs.workload("regression_onehot", K=K, B=B, L=1, d_in=d_in, precision=precision)
    p = tabpack.debug_plan(cfg, members=members(K, width))
    assert 0 < p["eval_operand"] <= OPERAND_MAX
    assert all(r >= 32 and r % 32 == 0 for r in p["eval_rows"])


@pytest.mark.parametrize("K,width,d_in,over", [
    (64, 512, 32_768, {}), (32, 512, 65_536, {}), (30, 128, 262_144, {}), (256, 128, 30_000, {}),
    (128, 256, 40_000, {}), (2, 16_384, 64, dict(L=2)), (256, 128, 30_000, dict(optimizer="muon")),
    (64, 512, 2_048, dict(emb_lo=16, emb_hi=16)), (4, 256, 256, dict(L=2)), (6, 130, 37, dict(L=3, B=300)),
    (40, 512, 512, dict(L=4, B=512))])
@pytest.mark.parametrize("tiles", [None, "mini", "small", "tall", "big", "huge"])
@pytest.mark.parametrize("streams", [None, "1", "3"])
def test_tile_table_holds_every_plan(monkeypatch, K, width, d_in, over, tiles, streams):
    # a bind fails when the launches' tiles outnumber the table's entries: packs
    # whose weight gradients have most of them, under every choice of tiles and
    # streams, with all members, one, or two thirds of them
    if tiles is not None:
        monkeypatch.setenv("TABPACK_GEMM_TILES", tiles)
        monkeypatch.setenv("TABPACK_NS_TILES", tiles)
    if streams is not None:
        monkeypatch.setenv("TABPACK_STREAMS", streams)
    cfg = configs.workload("regression_onehot", K=K, d_in=d_in, **dict(dict(L=1, B=256), **over))
    mem = members(K, width)
    for active in (None, [k == 0 for k in range(K)], [k % 3 > 0 or k == K - 1 for k in range(K)]):
        p = tabpack.debug_plan(cfg, members=mem, active=active)
        assert 0 < p["tiles"] <= p["tile_capacity"]


@pytest.mark.parametrize("K,width,B,over,groups,one", [
    # X' products of 128 x 128 tiles, on 64 features: K ((width / 128)^2 + width / 128)
    (16, 1024, 256, dict(), 2, False), (14, 1024, 256, dict(), 1, True),       # 1,152 and 1,008 of 1,024
    (2, 4096, 256, dict(), 2, False), (1, 4096, 256, dict(), 1, True),        # 2,112; one member cannot be split
    (5, 3072, 256, dict(), 1, True), (4, 3072, 256, dict(), 2, False),        # 3,000 and 2,400 of 2,560
    (4, 1024, 256, dict(precision="fp32"), 2, False), (3, 1024, 256, dict(precision="fp32"), 1, True),  # 288, 216 of 256
    (5, 3072, 256, dict(precision="fp32"), 2, False),
    # few symmetric tiles (of 144): wide first layers, whose products are shallow
    (90, 128, 256, dict(L=1, d_in=1500), 1, True), (40, 256, 256, dict(d_in=100, emb_lo=16, emb_hi=16), 2, False),
    (16, 256, 256, dict(precision="fp32", emb_lo=16, emb_hi=16), 1, True),
    (16, 1024, 256, dict(optimizer="adamw"), 1, True), (16, 1024, 2048, dict(), 3, False)])
def test_muon_split_rule(K, width, B, over, groups, one):
    cfg = configs.workload("regression_onehot", K=K, B=B, **dict(dict(optimizer="muon", L=2), **over))
    p = tabpack.debug_plan(cfg, members=members(K, width))
    assert (p["groups"], p["one_stream"]) == (groups, one)


SMALL, MINI = 1, 4  # tile sets


@pytest.mark.parametrize("K,width,B,over,sym,x", [
    # one stream: fewer than 256 tiles a launch -- K ((width / 128)^2 / 2 + ...) and X'
    (3, 1024, 256, dict(), MINI, MINI), (4, 1024, 256, dict(), MINI, SMALL), (8, 1024, 256, dict(), SMALL, SMALL),
    # groups in bf16: fewer than 400 tiles in all, or tiles times depth below 256 Ki (sym), 176 Ki (X')
    (16, 512, 2048, dict(), MINI, MINI), (32, 512, 1024, dict(), MINI, SMALL), (6, 1024, 4096, dict(), MINI, SMALL),
    (16, 512, 256, dict(d_in=2000), MINI, SMALL),  # (320 symmetric tiles in all, whatever their depth)
    (8, 1024, 2048, dict(), MINI, SMALL), (12, 1024, 2048, dict(), SMALL, SMALL), (4, 2048, 2048, dict(), SMALL, SMALL),
    # fp32: fewer than 256 tiles in the group with most
    (8, 1024, 2048, dict(precision="fp32"), MINI, MINI), (3, 2048, 4096, dict(precision="fp32"), MINI, SMALL),
    (4, 2048, 2048, dict(precision="fp32"), SMALL, SMALL)])
def test_newton_schulz_tile_rule(K, width, B, over, sym, x):
    cfg = configs.workload("regression_onehot", K=K, B=B, L=2, optimizer="muon", **over)
    p = tabpack.debug_plan(cfg, members=members(K, width))
    assert (p["ns_sym"], p["ns_x"]) == (sym, x)


@pytest.mark.parametrize("K,width,B", [(64, 2048, 256), (64, 2048, 2048), (200, 512, 256), (96, 1024, 1024)])
def test_huge_tiles_only_for_chunks_of_their_height(K, width, B):
    p = tabpack.debug_plan(configs.workload("regression_onehot", K=K, B=B, L=2), members=members(K, width))
    huge = 5
    assert [t == huge for t in p["eval_tiles"]] == [r >= 256 for r in p["eval_rows"]]
    assert p["eval_rows"][0] >= 256 > p["eval_rows"][-1]


@pytest.mark.parametrize("K,width,B,d_in,over,refused", [
    (1, 511, 256, 1 << 20, dict(precision="fp32"), False), (1, 512, 256, 1 << 20, dict(precision="fp32"), True),
    (2, 1023, 256, 1 << 20, dict(), False), (2, 1024, 256, 1 << 20, dict(), True),
    (1, 1000, 256, 65_536, dict(emb_lo=16, emb_hi=16), False), (1, 1025, 256, 65_536, dict(emb_lo=16, emb_hi=16), True),
    (1, 8_192, 65_535, 8, dict(precision="fp32"), False), (1, 8_192, 65_536, 8, dict(precision="fp32"), True),
    (1, 16_384, 65_536, 8, dict(), True)])
def test_operands_past_the_limit_are_refused(K, width, B, d_in, over, refused):
    # weights [width, d_in] or activations [B, width] of 2 GiB: their last rows would read as zeros
    cfg = configs.workload("regression_onehot", K=K, B=B, L=1, d_in=d_in, **over)
    if refused:
        with pytest.raises(tabpack.PackError, match="limited to 2 GiB"):
            tabpack.debug_plan(cfg, members=members(K, width))
    else:
        assert tabpack.debug_plan(cfg, members=members(K, width))["tiles"] > 0


@pytest.mark.parametrize("K,width,B,L,over,dw", [
    # two groups in bf16: fewer than 896 mini tiles (64 x 64) of both together, 512 in packs of one block
    (24, 384, 2304, 2, dict(), MINI), (26, 384, 2304, 2, dict(), SMALL),  # 864 and 936
    (62, 256, 2304, 1, dict(d_in=64), MINI), (130, 256, 2304, 1, dict(d_in=64), SMALL),  # 248 and 520
    (26, 384, 1024, 2, dict(K=60), SMALL), (30, 384, 1024, 2, dict(), MINI),  # short batches: the group's 135 of 256
    (26, 384, 2304, 2, dict(precision="fp32"), MINI), (60, 384, 2304, 2, dict(precision="fp32"), SMALL)])
def test_mini_weight_gradients_of_several_groups(K, width, B, L, over, dw):
    cfg = configs.workload("regression_onehot", B=B, L=L, **dict(dict(K=K), **over))
    p = tabpack.debug_plan(cfg, members=members(cfg["K"], width))
    assert p["groups"] == 2 and p["tiles_dw"] == dw


@pytest.mark.parametrize("K,width,B,over,fwd,dx", [
    # huge (5) from 640 small tiles of a mean depth of 512 on, data gradients from 2,048 of 768; else tall (2) from 1,024
    (40, 512, 2048, dict(), 5, 2), (40, 480, 2048, dict(), 2, 2),
    # (of 256 against small tiles of 16 members or more a launch)
    (32, 480, 1280, dict(), 5, 1), (30, 480, 1536, dict(), 1, 1), (64, 224, 1280, dict(), 1, 1), (44, 768, 2048, dict(), 5, 5), (44, 736, 2048, dict(), 5, 2),
    (24, 512, 1792, dict(), 5, 1), (22, 512, 1792, dict(), 1, 1),  # 672 and 616 small tiles a group
    (40, 512, 2048, dict(precision="fp32"), 1, 1)])
def test_huge_tiles_only_for_deep_launches(K, width, B, over, fwd, dx):
    p = tabpack.debug_plan(configs.workload("regression_onehot", K=K, B=B, L=2, **over), members=members(K, width))
    assert (p["tiles_fwd"], p["tiles_dx"]) == (fwd, dx)


@pytest.mark.parametrize("d_in,rows", [(16_000, 8_192), (65_528, 8_192), (65_536, 4_096), (262_144, 1_024)])
def test_wide_inputs_keep_the_chunks_that_fit(d_in, rows):
    # a chunk shrinks only where its rows would pass the loaders' limit: smaller
    # ones serve short requests by other tiles
    cfg = configs.workload("regression_onehot", K=4, B=256, L=1, d_in=d_in, precision="fp32")
    assert tabpack.debug_plan(cfg, members=members(4, 128))["eval_rows"][0] == rows


@pytest.mark.parametrize("width,tiles", [(128, 2), (160, 2), (192, 5), (512, 5)])
def test_huge_evaluation_tiles_by_depth(width, tiles):
    # tall (2) or huge (5) from 1,024 small tiles on: a depth of 192
    p = tabpack.debug_plan(configs.workload("regression_onehot", K=64, B=256, L=2), members=members(64, width))
    assert p["eval_tiles"][0] == tiles
