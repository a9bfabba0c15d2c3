"""The planner's limits, on the host: GEMM operands stay inside the loaders' 32-bit offsets and the tile table holds
every launch.  No GPU and no parameters."""
import pytest

from paper_2607_05380_amd import configs, tabpack

OPERAND_MAX = (1 << 31) - 16  # a GEMM loader's offsets: bytes of an operand below 2 GiB, less one 16-byte vector


def members(K, w, **hp):
    return [dict(dict(width=w, dropout=0.1, lr=1e-3, wd=1e-3, muon_lr=1e-2, d_emb=16, sigma=0.3), **hp)] * K


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("d_in", [8, 4_000, 65_536, 65_537, 66_000, 131_072, 131_080, 262_144, 1 << 20])
@pytest.mark.parametrize("K,width,B", [(1, 32, 1), (4, 128, 256), (1, 128, 2048), (40, 512, 700), (1, 128, 65_536)])
def test_evaluation_operands_below_the_loaders_limit(K, width, B, d_in, precision):
    # rows past the limit read as zeros or as other rows: wrong predictions
    cfg = configs.workload("regression_onehot", K=K, B=B, L=1, d_in=d_in, precision=precision)
    p = tabpack.debug_plan(cfg, members=members(K, width))
    assert 0 < p["eval_operand"] <= OPERAND_MAX
    assert all(r >= 32 and r % 32 == 0 for r in p["eval_rows"])
