"""The literal SE layer on the half-precision matrix cores (three-part
weights) against the checker, where a row tile, a K step, a feature block or
the LDS rows end, and its two reweightings (in place, and as the network over
row tiles reads the rows) against each other bit for bit."""
import numpy as np
import pytest

from paper_2007_16122_amd import synth
from tests.common import problem
from tests.gpu_common import (GpuScorer, compare_scores, device_table_from_numpy, log,
                              request_slice, run_oracle)

pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw,cand", [
    (dict(), [2000, 2000, 2000, 145]),                          # weighted by the network kernel
    (dict(dtype="f16", linear_log=True), [2000] * 8 + [401]),   # 32-row tiles of the layer
    (dict(n_ad=23), [1, 0, 15, 17]),                            # 47 groups: a half K step, a partial block
    (dict(dtype="f16", emb_dim=8, n_user=3, n_ad=5, n_cross=1), [33, 6200]),   # 9 groups of 8
    (dict(dtype="f16", n_user=16, n_ad=32, n_cross=16), [100, 6100]),          # 1,024 values: the longest LDS row
    (dict(dtype="f16", n_user=16, n_ad=32, n_cross=17), [100, 63]),            # past it
    (dict(dtype="f16", emb_dim=32, n_user=4, n_ad=8, n_cross=5, hashed=True), [70, 6100]),
])
def test_literal_split(kw, cand):
    cfg = synth.config("serving_bf16", vocab=20_000, se_form="literal", **kw)
    log(f"test_literal_split {kw} rows {sum(cand)} D_in {cfg.d_in}")
    tables, params, batch = problem(cfg, seed=73, cand=cand, model_seed=cfg.seed)
    # one feature's weights span the fp32 exponents an SE layer could hold
    params = dict(params)
    w = params["se_w1"].copy()
    w[1] *= np.float32(2.0) ** -20
    w[2, ::3] *= np.float32(2.0) ** -12
    params["se_w1"] = w
    run = GpuScorer(cfg, [device_table_from_numpy(t, cfg.dtype, "cuda") for t in tables], params, "cuda")
    q = len(cand) - 1
    try:
        g = run.score(batch, want_s=True)
        alone = run.score(request_slice(cfg, batch, q), want_s=True)
        x = run.score(batch, want_x=True)
    finally:
        run.close()
    off = batch["req_off"]
    for a, b in ((alone["s"], g["s"][off[q]:off[q + 1]]), (alone["scores"], g["scores"][off[q]:off[q + 1]]),
                 (x["scores"], g["scores"])):
        assert np.array_equal(a, b)
    rng = np.random.default_rng(79)
    n = batch["n_rows"]
    sample = np.unique(np.concatenate([rng.choice(n, min(n, 500), replace=False), [0, n - 1]]))
    o = run_oracle(cfg, tables, params, batch, sample=sample, want_s=True, want_x=True)
    # the layer's sum of D_in products in fp32, through a sigmoid of slope 1/4
    bound = 2.0 ** -24 * 4 + 0.25 * 2.0 ** -24 * (cfg.d_in / 32 * 3 + 4) * np.max(
        np.abs(o["x"]).sum(axis=1)) * 2 * np.max(np.abs(params["se_w1"]))
    assert np.max(np.abs(g["s"][sample] - o["s"])) <= min(bound, 1e-5)
    compare_scores(cfg, g["scores"][sample], o["scores"], f"literal split {kw}")


@pytest.mark.parametrize("n_cross", [5, 46])     # rows held in LDS; longer ones
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_literal_infinite_value(dtype, n_cross):
    """An infinite embedding value saturates its rows' weights by the sign of
    its column of W, also where a weight needs fewer than three parts, and
    leaves the other rows as they are."""
    cfg = synth.config("serving_bf16", vocab=50, se_form="literal", dtype=dtype, n_user=4, n_ad=16,
                       n_cross=n_cross)
    log(f"test_literal_infinite_value {dtype} D_in {cfg.d_in}")
    tables, params, batch = problem(cfg, seed=83, cand=[70, 19], model_seed=cfg.seed)
    params = dict(params)
    w = params["se_w1"].copy()
    col = cfg.n_user * cfg.emb_dim
    w[:, col] = np.where(np.arange(cfg.n_groups) % 2, np.float32(-0.1), np.float32(0.5))
    params["se_w1"] = w
    scores = []
    for inf in (False, True):
        if inf:
            tables = list(tables)
            t = tables[cfg.n_user].copy()
            t[7, 0] = 0x7F80 if dtype == "bf16" else np.inf
            tables[cfg.n_user] = t
        run = GpuScorer(cfg, [device_table_from_numpy(t, cfg.dtype, "cuda") for t in tables], params, "cuda")
        try:
            scores.append(run.score(batch, want_s=True))
        finally:
            run.close()
    hit = batch["ad_ids"][0] == 7
    assert hit.any() and not hit.all()
    want = (w[:, col] > 0).astype(np.float32)
    assert np.array_equal(scores[1]["s"][hit], np.broadcast_to(want, (hit.sum(), cfg.n_groups)))
    for k in ("s", "scores"):
        assert np.array_equal(scores[1][k][~hit], scores[0][k][~hit])
