"""The fp32 model in one kernel against the checker, over the shapes where a
tile, a group slot, a K chunk or a width ends."""
import numpy as np
import pytest

from paper_2007_16122_amd import synth
from tests.common import assert_se_weights_close, problem
from tests.gpu_common import (GpuScorer, compare_scores, device_table_from_numpy, log,
                              request_slice, run_oracle)

pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw,hidden,n_out,cand", [
    (dict(n_user=1, n_ad=1, n_cross=0), (4, 1), 1, [1]),              # the smallest
    (dict(n_user=4, n_ad=8, n_cross=4), (64, 64), 2, [15, 0, 1, 17]),  # 16 groups, a slot each
    (dict(n_user=4, n_ad=8, n_cross=5), (64, 32), 1, [300, 16]),      # 17: a second slot
    (dict(n_user=8, n_ad=16, n_cross=8, linear_log=True), (60, 33), 1, [33, 64, 1]),   # 32 groups
    (dict(n_user=9, n_ad=16, n_cross=8, hashed=True), (20, 17), 2, [33, 64, 1]),       # 33
    (dict(n_user=16, n_ad=32, n_cross=16, hashed=True, cross_pairs=tuple((f, 2 * f) for f in range(16))),
     (64, 64), 1, [9000, 7, 3]),                                      # 64 groups, many tiles a workgroup
    (dict(n_user=0, n_ad=5, n_cross=3), (8, 8), 1, [40, 41]),         # no user side
    (dict(), (64, 32), 1, [3] * 1500),                                # offsets past the LDS copy
    (dict(), (68, 32), 1, [100, 12]),                                 # wider than 64: layer by layer
])
def test_net_f32(kw, hidden, n_out, cand):
    cfg = synth.config("tiny_fp32", vocab=5000, **kw)
    cfg = synth.config("tiny_fp32", vocab=5000, **kw, widths=(cfg.d_in,) + hidden + (n_out,))
    log(f"test_net_f32 {kw} {cfg.widths} rows {sum(cand)}")
    tables, params, batch = problem(cfg, seed=71, cand=cand)
    run = GpuScorer(cfg, [device_table_from_numpy(t, cfg.dtype, "cuda") for t in tables], params, "cuda")
    q = len(cand) - 1
    try:
        g = run.score(batch, want_rows=True, want_s=True, want_x=True)
        plain = run.score(batch)["scores"]
        alone = run.score(request_slice(cfg, batch, q))["scores"]
    finally:
        run.close()
    off = batch["req_off"]
    assert np.array_equal(plain.view(np.uint32), g["scores"].view(np.uint32))
    assert np.array_equal(alone.view(np.uint32), plain[off[q]:off[q + 1]].view(np.uint32))
    o = run_oracle(cfg, tables, params, batch, want_rows=True, want_s=True, want_z=True, want_x=True)
    assert np.array_equal(g["rows"], o["rows"].T.astype(np.int32))
    assert_se_weights_close(params, g["s"], o)
    # two fp32 roundings of a weight within 3e-6 and one of the product (and
    # the logarithm's 2^-22) on values below 1
    assert np.max(np.abs(g["x"].astype(np.float64) - o["x"])) <= 4e-6
    compare_scores(cfg, g["scores"], o["scores"], f"net_f32 {kw}")
