"""The statistics of a step on both sides of the rule that merges a row's partials
before the decision (more than 6000 partials per sequence: block length times
vocabulary tiles of 256 ids), around one pass of a merging wave's lanes (512 partials),
against the logits that the same kernels give."""
import numpy as np
import pytest
import torch

import wino_inputs as wi
from helpers import STATS_DT, batch_tokens

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab,lb,B", [
    (256 * 250, 24, 3), (256 * 251, 24, 3), (256 * 100, 61, 2), (256 * 7, 1, 1), (256 * 512, 12, 1),
    (256 * 513, 12, 2), (256 * 526, 12, 1),
])
def test_step_statistics(vocab, lb, B, monkeypatch):
    import paper_2605_16941_amd as P
    # one tile, no K-slices: the step's gathered block rows and the full forward of
    # the logits then go through the same additions, so the logits are the same bits
    monkeypatch.setenv("WINO_GEMM_TILE", "0")
    monkeypatch.setenv("WINO_GEMM_TAIL", "0")
    cfg = wi.preset("tiny", n_layers=1, vocab=vocab, mask_id=700)
    wd = wi.model_weights(cfg, seed=4, device="cuda", gain_std=0.1)
    wd["lm_bias"] = None  # (a flat distribution: every partial carries its share of the sum)
    p, g = 7, 2 * lb
    model = P.WinoModel(cfg, wd, B, p + g + lb)
    tok = batch_tokens(cfg, B, p, g, seed=6, fill=[(0, lb, 0.5)] if lb > 1 else None)
    prm = P.make_params(B, p, g, lb, cfg.mask_id)
    tok_d = torch.tensor(tok, dtype=torch.int32, device="cuda")
    bs = torch.zeros(B, dtype=torch.int32, device="cuda")
    logits = torch.empty(B, 2 * lb, vocab, device="cuda")
    P.wino_debug_logits(model.ctx, prm, tok_d, bs, logits)
    stats = torch.empty(B, lb, 6, dtype=torch.int32, device="cuda")
    P.wino_step(model.ctx, prm, tok_d, bs, None, None, None, stats)
    torch.cuda.synchronize()
    model.close()
    st = stats.cpu().numpy().view(STATS_DT)[..., 0]
    z = logits.cpu().numpy()
    for b in range(B):
        for j in range(lb):
            t = tok[b, p + j]
            row = z[b, j if t == cfg.mask_id else lb + j]
            s = st[b, j]
            assert s["m_all"] == row.max()
            e = np.exp(row.astype(np.float64) - row.max())
            # one exponential per id and per merge level, each good to (2 + |z - m|) 2^-23,
            # and about ten levels of fp32 sums; a 256-id tile is more than 1e-4 of it
            n = vocab // 256
            assert e.reshape(n, 256).sum(-1).min() > 1e-4 * e.sum()
            assert abs(s["sumexp"] / e.sum() - 1) < (12 + float(row.max() - row.min())) * 2.0 ** -23
            best = np.where(np.arange(vocab) == cfg.mask_id, -np.inf, row)
            assert s["z_best"] == best.max() and s["argmax"] == int(np.argmax(best))
            if t != cfg.mask_id:
                assert s["z_target"] == row[t]
