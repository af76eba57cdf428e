"""The gather with one wave per 16 groups against the checker: pooled groups
at the ends of a wave's slots, 16-byte group rows, row counts around a tile
and around the sizes where the form changes."""
import numpy as np
import pytest

from paper_2007_16122_amd import synth
from tests.common import assert_se_weights_close, problem
from tests.gpu_common import (GpuScorer, compare_scores, device_table_from_numpy, log,
                              request_slice, run_oracle, with_empty_sequences)

pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,kw,cand", [
    ("multivalued_fp16_ll", dict(), [1, 15, 0, 17]),                        # 54 groups, groups 12..17 pooled
    ("multivalued_fp16_ll", dict(n_user=0, n_seq=1, n_ad=3, n_cross=0), [33]),        # one wave, no user rows
    ("multivalued_fp16_ll", dict(n_user=16, n_seq=16, n_ad=16, n_cross=16), [40, 7]),  # a wave all pooled
    ("multivalued_fp16_ll", dict(n_user=6, n_seq=8, n_ad=12, n_cross=7, hashed=True), [300, 90]),
    ("multivalued_fp16_ll", dict(emb_dim=8), [64, 31, 5]),
    ("serving_bf16", dict(emb_dim=8, n_ad=23), [100, 0, 29]),               # 16-byte rows, 47 groups
    ("serving_bf16", dict(emb_dim=8, cross_pairs=tuple((f, f) for f in range(12))), [50] * 30),
    ("serving_bf16", dict(), [8192]),                                       # the most tiles of the chained form
    ("serving_bf16", dict(), [4000, 4000, 193]),                            # the fewest of this one
    ("serving_bf16", dict(linear_log=True), [12800, 12800]),                # the most
    ("serving_bf16", dict(), [12800, 12801]),                               # past it: one wave per tile
])
def test_gather_split(name, kw, cand):
    cfg = synth.config(name, vocab=20_000, **kw)
    log(f"test_gather_split {name} {kw} rows {sum(cand)}")
    tables, params, batch = problem(cfg, seed=83, cand=cand, model_seed=cfg.seed)
    if cfg.n_seq:
        batch = with_empty_sequences(cfg, batch, {(0, 0), (cfg.n_seq - 1, len(cand) - 1)})
    run = GpuScorer(cfg, [device_table_from_numpy(t, cfg.dtype, "cuda") for t in tables], params, "cuda")
    q = len(cand) - 1
    try:
        g = run.score(batch, want_rows=True, want_s=True)
        alone = run.score(request_slice(cfg, batch, q), want_s=True)
    finally:
        run.close()
    lo, hi = (int(v) for v in batch["req_off"][q:q + 2])
    assert np.array_equal(alone["s"].view(np.uint32), g["s"][lo:hi].view(np.uint32))
    assert np.array_equal(alone["scores"], g["scores"][lo:hi])
    rng = np.random.default_rng(89)
    n = batch["n_rows"]
    sample = np.unique(np.concatenate([rng.choice(n, min(n, 400), replace=False), [0, n - 1]]))
    o = run_oracle(cfg, tables, params, batch, sample=sample, want_rows=True, want_s=True, want_z=True)
    assert np.array_equal(g["rows"][:, sample], o["rows"].T.astype(np.int32)), "gather indices differ"
    assert_se_weights_close(params, g["s"][sample], o)
    compare_scores(cfg, g["scores"][sample], o["scores"], f"gather split {name} {kw}")
