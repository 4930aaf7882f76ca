"""The statistics of a step on both sides of the rule that merges a row's partials
before the decision (more than 6000 partials per sequence: block length times
vocabulary tiles of 256 ids), against the logits of the same kernels."""
import numpy as np
import pytest
import torch

import wino_inputs as wi
from helpers import STATS_DT, batch_tokens

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab,lb,B", [(256 * 250, 24, 3), (256 * 251, 24, 3), (256 * 100, 61, 2), (256 * 7, 1, 1)])
def test_step_statistics(vocab, lb, B):
    import paper_2605_16941_amd as P
    cfg = wi.preset("tiny", n_layers=1, vocab=vocab, mask_id=700)
    wd = wi.model_weights(cfg, seed=4, device="cuda", gain_std=0.1)
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
    z = logits.double().cpu().numpy()
    for b in range(B):
        for j in range(lb):
            t = tok[b, p + j]
            row = z[b, j if t == cfg.mask_id else lb + j]
            # the step runs its last layer's block rows in other tiles than the
            # full forward of the logits: fp32 sums in another order, at most a bf16
            # flip upstream
            s = st[b, j]
            assert abs(s["m_all"] - row.max()) < 1e-2
            want = np.exp(row - row.max()).sum()
            assert abs(s["sumexp"] * np.exp(s["m_all"] - row.max()) / want - 1) < 1e-2
            best = np.where(np.arange(vocab) == cfg.mask_id, -np.inf, row)
            assert abs(s["z_best"] - best.max()) < 1e-2 and best[s["argmax"]] > best.max() - 2e-2
            if t != cfg.mask_id:
                assert abs(s["z_target"] - row[t]) < 1e-2
