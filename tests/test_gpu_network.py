"""The network over 64-row tiles in one kernel (batches of many rows) against
the checker and, bit for bit, against the layer-by-layer path that scores the
same requests alone."""
import numpy as np
import pytest

from paper_2007_16122_amd import synth
from tests.common import problem
from tests.gpu_common import (GpuScorer, compare_scores, device_table_from_numpy, log,
                              request_slice, run_oracle)

pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EDGE = [2000, 2000, 2000, 0, 193]      # 6,193 rows: 97 tiles, the last of 49 rows


@pytest.mark.parametrize("kw,cand", [
    (dict(), EDGE),                                               # 24 K steps
    (dict(), [2000, 2000, 2000, 144]),                            # 96 tiles exactly, the fewest
    (dict(dtype="f16", n_ad=23), EDGE),                           # D_in 752: half a K step of zeros
    (dict(dtype="f16", n_cross=14), EDGE),                        # 25 K steps
    (dict(dtype="f16", linear_log=True, n_user=16, n_ad=32, n_cross=16), EDGE),   # 1,024: the widest input
    (dict(dtype="f16", emb_dim=8, n_user=3, n_ad=4, n_cross=2), EDGE),            # 72: three K steps
    (dict(dtype="f16", n_user=16, n_ad=32, n_cross=17), EDGE),    # 1,040: past it, layer by layer
    (dict(), [1999] * 17 + [1]),                                  # three tiles per workgroup
    (dict(dtype="f16", widths=(768, 512, 256, 128, 64, 1)), EDGE),     # without the 1,024-wide layer
    (dict(dtype="f16", n_cross=14, widths=(800, 512, 256, 128, 64, 2)), [1999] * 17),
])
def test_row_tile_network(kw, cand):
    cfg = synth.config("serving_bf16", vocab=20_000, **kw)
    log(f"test_row_tile_network {kw} rows {sum(cand)} D_in {cfg.d_in}")
    tables, params, batch = problem(cfg, seed=61, cand=cand, model_seed=cfg.seed)
    run = GpuScorer(cfg, [device_table_from_numpy(t, cfg.dtype, "cuda") for t in tables], params, "cuda")
    qs = [0, len(cand) - 1]
    try:
        g = run.score(batch)["scores"]
        alone = [run.score(request_slice(cfg, batch, q))["scores"] for q in qs]
    finally:
        run.close()
    off = batch["req_off"]
    for q, a in zip(qs, alone):
        assert np.array_equal(a.view(np.uint32), g[off[q]:off[q + 1]].view(np.uint32)), f"request {q}"
    rng = np.random.default_rng(67)
    ends = [r for r in (0, 63, 64, 4095, 4096, batch["n_rows"] - 1)]
    sample = np.unique(np.concatenate([rng.choice(batch["n_rows"], 600, replace=False), ends]))
    o = run_oracle(cfg, tables, params, batch, sample=sample)
    compare_scores(cfg, g[sample], o["scores"], f"row-tile network {kw}")
